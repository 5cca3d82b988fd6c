// Deposit (Eq. smooth) and smoothed-force gather (Eq. gi) by tile pieces, for
// every kernel ball that reaches at most 8 cells.
//
// Weights.  A particle at u = x / s has the central pixel c = floor(u + 1/2)
// and the sub-pixel offset f = c - u.  Its Gaussian weight on ball cell d is
// exp(-|d + f|^2 / (2 sigma^2)) = wx[dx] wy[dy] wz[dz], so a lane evaluates
// 3 (2 EXT + 1) exponentials and forms the products; for the balls of radius 4
// sigma at sigma = 1, 1.5 and 2 cells which cells are in it is known at compile
// time, so every cell's LDS address is the lane's base address plus an
// immediate.  The normalisation S = sum_B w is
// summed in FP64 row by row: for the row (dy, dz) of half-width h,
// wy[dy] wz[dz] sum_{|dx| <= h} wx[dx].
//
// Work split.  After the tile sort (8^3-cell tiles), each tile's particles are
// cut into pieces of at most kPiece; blocks take pieces from a work counter.
//  - Deposit: a piece accumulates its balls in an LDS copy of the tile plus a
//    halo of EXT cells, as exact 64-bit fixed-point sums at its tile's scale
//    (below), and stores the piece's halo box to a staging slot: as integers
//    if the tile has several pieces, else as FP32 (one rounding of the exact
//    sum).  A second kernel gives every tile near matter one owner block,
//    which sums each of the 27 neighbouring tiles' staged boxes exactly
//    (integers, at that neighbour's scale), converts the 27 sums and adds
//    them in a fixed order into rho.  No cell is written with global atomics and no rounding
//    depends on how a tile's particles fall into pieces, so the density does
//    not depend on the order in which the particles arrive (the sort ranks
//    them within a tile with atomics).  Pieces beyond the staging capacity
//    (and particles whose mass or position is not finite) add their cells with
//    FP32 global atomics.
//  - Gather: a piece loads its tile plus a halo of EXT + 1 cells of phi into
//    LDS once; each lane then sums its particle's ball with the central
//    difference folded into the weights, g = -(1/(2 s S)) sum_e phi(c + e) W(e)
//    with W_x(e) = w(e - e_x) - w(e + e_x) (w = 0 outside the ball), so every
//    cell of the dilated ball is read once; phi is taken relative to phi(c),
//    which the zero sum of W allows and which keeps the FP32 products small.
#include <type_traits>

#include "pm_device.h"
#include "pm_internal.h"

namespace pm {

namespace {
constexpr int kTile = 8;
constexpr int kNT = 256;
// Block sizes of the deposit and of the gather (a piece per block).  Pieces
// average about 70 particles on the isothermal sphere, so a block of the narrow
// ball's gather is two waves, which keeps more pieces in flight per CU.
constexpr int kDepNT = 256;
// Particles up to which a pass goes by rows of the ball, one particle per wave,
// and not by one particle per lane.
constexpr int kRowMost = 16;
#ifndef PM_GATHER_NT
#define PM_GATHER_NT 128
#endif
#ifndef PM_GATHER_NT_WIDE
#define PM_GATHER_NT_WIDE 256
#endif
constexpr int gather_nt(int ext) { return ext <= 3 ? PM_GATHER_NT : PM_GATHER_NT_WIDE; }

__device__ __forceinline__ int wrapi(int i, int N) { return i & (N - 1); }

constexpr bool in_ball(int x, int y, int z, int R2, int EXT) {
  return x >= -EXT && x <= EXT && y >= -EXT && y <= EXT && z >= -EXT && z <= EXT && x * x + y * y + z * z < R2;
}
// half-width of row (dy, dz) of the ball, -1 if the row is empty
constexpr int row_half(int dy, int dz, int R2, int EXT) {
  int h = -1;
  for (int x = 0; x <= EXT; ++x)
    if (in_ball(x, dy, dz, R2, EXT)) h = x;
  return h;
}

// Compile-time loops.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Per-lane particle state.
template <int EXT>
struct Lane {
  int cx, cy, cz;              // central pixel (wrapped grid index)
  float wx[2 * EXT + 1], wy[2 * EXT + 1], wz[2 * EXT + 1];
  double sx[EXT + 1];          // sum of wx over |dx| <= h
};

template <int EXT>
__device__ __forceinline__ void lane_setup(Lane<EXT>& L, const KernelGeom& kg, float px, float py, float pz) {
  const int half = kg.N / 2;
  float fx, fy, fz;
  L.cx = wrapi(central_pixel(px, kg.inv_s, &fx) + half, kg.N);
  L.cy = wrapi(central_pixel(py, kg.inv_s, &fy) + half, kg.N);
  L.cz = wrapi(central_pixel(pz, kg.inv_s, &fz) + half, kg.N);
#pragma unroll
  for (int d = -EXT; d <= EXT; ++d) {
    const float ex = (float)d + fx, ey = (float)d + fy, ez = (float)d + fz;
    L.wx[d + EXT] = expf(-ex * ex * kg.inv2sig2);
    L.wy[d + EXT] = expf(-ey * ey * kg.inv2sig2);
    L.wz[d + EXT] = expf(-ez * ez * kg.inv2sig2);
  }
  L.sx[0] = (double)L.wx[EXT];
#pragma unroll
  for (int h = 1; h <= EXT; ++h) L.sx[h] = L.sx[h - 1] + ((double)L.wx[EXT - h] + (double)L.wx[EXT + h]);
}

// Blocks take pieces from a work counter (pieces differ in size by three
// orders of magnitude); the tile of a piece is one load from the map.
__device__ __forceinline__ int next_piece(int* counter, int* slot) {
  __syncthreads();
  if (threadIdx.x == 0) *slot = atomicAdd(counter, 1);
  __syncthreads();
  return *slot;
}

// ---------------------------------------------------------------------------
// weights of a batch of particles
// ---------------------------------------------------------------------------
// Weights of up to NT / 4 particles into w[p][3 W] (x, y, z), four threads per
// particle, and their normalisations into norm[p].  index(p): the particle of
// batch entry p.  base[p]: its central cell in the LDS tile (row pitch RP, plane
// pitch PP, halo HE).  Ends with a barrier.
template <int EXT, int NT, typename T, typename F>
__device__ __forceinline__ void weights_to_lds(const KernelGeom& kg, const float* __restrict__ pos, int count, int HE,
                                               int RP, int PP, const int* hrow, T* w, double* norm, int* base,
                                               F&& index) {
  constexpr int W = 2 * EXT + 1, WS = 3 * W + 1;
  const int p = threadIdx.x >> 2, q = threadIdx.x & 3;
  const bool on = p < count;
  T* wp = w + p * WS;
  if (on) {
    const int64_t i = index(p);
    const int half = kg.N / 2;
    float f[3];
    int c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
      c[a] = wrapi(central_pixel(pos[3 * i + a], kg.inv_s, &f[a]) + half, kg.N) & (kTile - 1);
    for (int d = q; d < 3 * W; d += 4) {
      const int a = d / W;
      const float e = (float)(d - a * W - EXT) + (a == 0 ? f[0] : a == 1 ? f[1] : f[2]);
      wp[d] = (T)expf(-e * e * kg.inv2sig2);
    }
    if (q == 0) base[p] = (c[2] + HE) * PP + (c[1] + HE) * RP + c[0] + HE;
  }
  __syncthreads();
  double S = 0.0;
  if (on && !kg.analytic) {
    // sum over the ball, row by row: wy wz sum_{|dx| <= h} wx in FP64
    double sx[EXT + 1];
    sx[0] = (double)wp[EXT];
#pragma unroll
    for (int h = 1; h <= EXT; ++h) sx[h] = sx[h - 1] + ((double)wp[EXT - h] + (double)wp[EXT + h]);
    for (int z = q; z < W; z += 4) {
      double t = 0.0;
      for (int y = 0; y < W; ++y) {
        const int h = hrow[z * W + y];
        double v = 0.0;
#pragma unroll
        for (int k = 0; k <= EXT; ++k) v = (h == k) ? sx[k] : v;
        t = fma((double)wp[W + y], v, t);
      }
      S = fma((double)wp[2 * W + z], t, S);
    }
  }
  S += __shfl_xor(S, 1, 64);
  S += __shfl_xor(S, 2, 64);
  if (on && q == 0) norm[p] = kg.analytic ? kg.analytic_norm : S;
  __syncthreads();
}

// The ball's rows from the context's table: half-widths by (dz, dy) into
// hrow[W][W] (-1: no row; block-wide, no barrier at the end), and the lane's own
// rows lane + 64 u.
template <int EXT, int RU>
__device__ __forceinline__ void ball_rows(const KernelGeom& kg, int NT, int RP, int PP, int* hrow, int* roff, int* rh,
                                          int* ry, int* rz) {
  constexpr int W = 2 * EXT + 1;
  for (int j = threadIdx.x; j < W * W; j += NT) hrow[j] = -1;
  __syncthreads();
  for (int j = threadIdx.x; j < kg.nrows; j += NT) {
    const int r = kg.rows[j];
    hrow[(((r >> 8) & 255) - 16 + EXT) * W + (r & 255) - 16 + EXT] = r >> 16;
  }
#pragma unroll
  for (int u = 0; u < RU; ++u) {
    const int k = (threadIdx.x & 63) + 64 * u;
    const int r = k < kg.nrows ? kg.rows[k] : (16 | 16 << 8);
    ry[u] = (r & 255) - 16;
    rz[u] = ((r >> 8) & 255) - 16;
    rh[u] = k < kg.nrows ? r >> 16 : -1;
    roff[u] = rz[u] * PP + ry[u] * RP;
  }
}

// ---------------------------------------------------------------------------
// deposit
// ---------------------------------------------------------------------------
// Fixed-point cell sums.  LDS adds of 64-bit integers are native and an order
// of magnitude faster than LDS adds of FP32 on this chip (those take a slow
// path), and integer sums are exact, so a piece accumulates its balls as
// integers: each contribution c becomes round(c 2^k) with one power-of-two
// scale per tile, shared by the tile's pieces, chosen so that no cell sum over
// all the tile's particles can overflow; the cell's FP32 value is the integer
// sum times 2^-k.  The product of the three normalised 1D weights is at most 1,
// so every contribution of particle i is at most A_i = |m_i| / (S_i s^3) <=
// |m_i| / (w0 s^3), w0 being the smallest possible central-cell weight; a tile of
// n_t particles adds at most n_t contributions to a cell.  With A < 2^e for the
// tile's largest |m|, k = 51 - ceil(log2 n_t) - e keeps every sum below 2^51,
// where round(c 2^k) is the low part of the FP64 number c 2^k + 3 2^51: one
// multiply-add makes it from the weights.
//
// Work split.  The piece's particles are ordered by cell and go in batches of
// 64, whose weights four threads per particle put into LDS.
//  - By rows: lanes own rows (dy, dz) of the ball and a wave takes one particle
//    at a time, so a wave's adds go to distinct cells however the particles
//    crowd; a lane keeps its row's sums in registers, with LDS adds only when
//    the cell changes.  Three instructions per dx and lane.
//  - One particle per lane (the 251 cells of radius 4, batches of more than
//    kRowMost particles): the ball's slices dz are dealt to the four waves, two
//    instructions and an LDS add per cell at compile-time offsets.  Neighbouring
//    lanes take particles far apart in the cell order, so that few of a wave's
//    adds meet at one address.
// Bound: vector instructions by rows, LDS adds by lanes.  Measured, tile kernel:
// the ring's 4097 particles (sigma = 1.5) 48 us, 425 us with a lane per particle
// in the sort's order, whose adds ran up to 64 deep on one address; 300 001
// particles of a mixture (sigma = 1) 103 us, 134 us that way, 126 us all by
// rows; the isothermal sphere's 2^20, about 70 to a piece, 302 us (265 us with
// each wave taking particles of its own and no ordering).
__device__ __forceinline__ int tile_scale_exp(const KernelGeom& kg, unsigned mbits, int count) {
  const double s3 = (double)kg.s * kg.s * kg.s;
  // the normalisation is at least the central cell's weight, whose offset is
  // at most 1/2 cell per axis (or the analytic prefactor)
  const double norm_lo = kg.analytic ? kg.analytic_norm : (double)expf(-0.75f * kg.inv2sig2);
  const double A = (double)__uint_as_float(mbits) / (norm_lo * s3);
  int e = 0;
  frexp(A > 0.0 ? A : 1.0, &e);                   // A < 2^e
  const int cb = count > 1 ? 32 - __clz(count - 1) : 0;      // ceil(log2 count)
  return 51 - cb - e;
}

// Largest |m| of each tile's particles, tmax[t] (float bits; zeroed before),
// from the pieces: a block reduces a piece and adds one atomic max per wave.
// Values that are not finite set no scale.
__global__ __launch_bounds__(kNT) void k_tile_mass_max(const int* __restrict__ perm, const int* __restrict__ offsets,
                                                      const int* __restrict__ pc_off, const int* __restrict__ ptile,
                                                      int ntiles, int piece, const float* __restrict__ mass,
                                                      unsigned* tmax) {
  const int total = pc_off[ntiles];
  for (int p = blockIdx.x; p < total; p += gridDim.x) {
    const int t = ptile[p];
    const int a = offsets[t] + (p - pc_off[t]) * piece;
    const int b = min(a + piece, offsets[t + 1]);
    float m = 0.0f;
    for (int j = a + (int)threadIdx.x; j < b; j += kNT) {
      const float v = fabsf(mass[perm[j]]);
      m = v < INFINITY ? fmaxf(m, v) : m;
    }
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63) == 0 && m > 0.0f) atomicMax(&tmax[t], __float_as_uint(m));   // non-negative floats order as their bits
  }
}

constexpr double kFixMagic = 6755399441055744.0;           // 3 2^51
constexpr unsigned kFixMagicHi = 0x43380000u;               // its high word; the low word is 0

// Pitches of the deposit's LDS tile: odd, so that a wave's rows spread over
// the banks.
template <int EXT>
struct DepTile {
  static constexpr int TE = kTile + 2 * EXT, RP = TE | 1, PP = RP * TE + 2;
  static constexpr size_t cells = (size_t)PP * TE;
};
constexpr int kDepBatch = kDepNT / 4;

// R2: the compiled shape of the lane path, 0 without one.
template <int EXT, int R2>
__global__ __launch_bounds__(kDepNT) void k_deposit_pieces(KernelGeom kg, const int* __restrict__ perm,
                                                           const int* __restrict__ offsets,
                                                           const int* __restrict__ pc_off,
                                                           const int* __restrict__ ptile, int ntiles, int* counter,
                                                           const float* __restrict__ pos,
                                                           const float* __restrict__ mass,
                                                           const unsigned* __restrict__ tmax, long long* stage,
                                                           int cap, float* rho) {
  using D = DepTile<EXT>;
  constexpr int TE = D::TE, RP = D::RP, PP = D::PP, TE3 = TE * TE * TE;
  constexpr int W = 2 * EXT + 1, WS = 3 * W + 1, RU = (W * W + 63) / 64;
  extern __shared__ unsigned long long tile64[];
  double* wb = reinterpret_cast<double*>(tile64 + D::cells);      // [kDepBatch][WS]
  __shared__ double norm[kDepBatch], amp[kDepBatch];
  __shared__ int cell[kDepBatch], bins[512], wsum[kDepNT / 64];
  __shared__ unsigned short order[kMaxPiece];
  __shared__ int hrow[W * W];
  __shared__ int slot;
  const int N = kg.N, nt = N / kTile, piece = kg.piece;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double s3 = (double)kg.s * kg.s * kg.s;
  const int total = pc_off[ntiles];
  int roff[RU], rh[RU], ry[RU], rz[RU];
  ball_rows<EXT, RU>(kg, kDepNT, RP, PP, hrow, roff, rh, ry, rz);
  for (int p = next_piece(counter, &slot); p < total; p = next_piece(counter, &slot)) {
    const int t = ptile[p];
    const int a = offsets[t] + (p - pc_off[t]) * piece;
    const int n = min(piece, offsets[t + 1] - a);
    const int tx = t % nt, ty = (t / nt) % nt, tz = t / (nt * nt);
    const bool staged = p < cap;
    const int k = staged ? tile_scale_exp(kg, tmax[t], offsets[t + 1] - offsets[t]) : 0;
    // particles in the order of their cells (few particles: as they come)
    const bool sorted = n > 32;
    for (int j = threadIdx.x; j < (int)D::cells; j += kDepNT) tile64[j] = 0ull;
    if (sorted) {
      bins[threadIdx.x] = bins[threadIdx.x + 256] = 0;
      __syncthreads();
      int key[kMaxPiece / kDepNT], rank[kMaxPiece / kDepNT];
#pragma unroll
      for (int u = 0; u < kMaxPiece / kDepNT; ++u) {
        const int j = threadIdx.x + u * kDepNT;
        if (j < n) {
          const int64_t i = perm[a + j];
          int c[3];
          for (int x = 0; x < 3; ++x)
            c[x] = (central_pixel(pos[3 * i + x], kg.inv_s, nullptr) + N / 2) & (kTile - 1);
          key[u] = (c[2] * kTile + c[1]) * kTile + c[0];
          rank[u] = atomicAdd(&bins[key[u]], 1);
        }
      }
      __syncthreads();
      const int b0 = bins[2 * threadIdx.x], b1 = bins[2 * threadIdx.x + 1];
      int x = b0 + b1;
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
      }
      if (lane == 63) wsum[wave] = x;
      __syncthreads();
      for (int w = 0; w < wave; ++w) x += wsum[w];
      bins[2 * threadIdx.x] = x - b0 - b1;
      bins[2 * threadIdx.x + 1] = x - b1;
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kMaxPiece / kDepNT; ++u) {
        const int j = threadIdx.x + u * kDepNT;
        if (j < n) order[bins[key[u]] + rank[u]] = (unsigned short)j;
      }
    }
    __syncthreads();
    for (int j0 = 0; j0 < n; j0 += kDepBatch) {
      const int count = min(kDepBatch, n - j0);
      // (by lanes, entry q of batch b is the particle q nb + b of the cell order)
      const int nb = n / kDepBatch, b = j0 / kDepBatch;
      const bool spread = R2 > 0 && b < nb;
      auto at = [&](int q) { return perm[a + (sorted ? (int)order[spread ? q * nb + b : j0 + q] : j0 + q)]; };
      weights_to_lds<EXT, kDepNT>(kg, pos, count, EXT, RP, PP, hrow, wb, norm, cell, at);
      if (threadIdx.x < count) amp[threadIdx.x] = ldexp((double)mass[at(threadIdx.x)] / (norm[threadIdx.x] * s3), k);
      __syncthreads();
      if constexpr (R2 > 0) {
        bool lanes = staged && count > kRowMost;
        for (int q = 0; q < count && lanes; q += 64) lanes = __all(q + lane >= count || fabs(amp[q + lane]) < INFINITY);
        if (lanes) {
          if (lane < count) {
            const double* wp = wb + lane * WS;
            const double m = amp[lane];
            double wx[W];
#pragma unroll
            for (int d = 0; d < W; ++d) wx[d] = wp[d];
            unsigned long long* c0 = tile64 + cell[lane];
            static_for<-EXT, EXT + 1>([&](auto DZc) {
              constexpr int dz = decltype(DZc)::value;
              if ((dz + EXT) % (kDepNT / 64) != wave) return;
              const double mz = m * wp[2 * W + dz + EXT];
              static_for<-EXT, EXT + 1>([&](auto DYc) {
                constexpr int dy = decltype(DYc)::value;
                constexpr int h = row_half(dy, dz, R2, EXT);
                if constexpr (h >= 0) {
                  const double ayz = mz * wp[W + dy + EXT];
                  static_for<-h, h + 1>([&](auto DXc) {
                    constexpr int dx = decltype(DXc)::value;
                    const unsigned long long v = (unsigned long long)__double_as_longlong(fma(ayz, wx[dx + EXT], kFixMagic)) -
                                                 ((unsigned long long)kFixMagicHi << 32);
                    __hip_atomic_fetch_add(c0 + dz * PP + dy * RP + dx, v, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                  });
                }
              });
            });
          }
          __syncthreads();
          continue;
        }
      }
      // a run of the batch per wave
      const int per = (count + kDepNT / 64 - 1) / (kDepNT / 64);
      const int q0 = wave * per, q1 = min(q0 + per, count);
#pragma unroll 1
      for (int u = 0; u < RU; ++u) {
        if (64 * u >= kg.nrows) break;
        const int h = rh[u], yo = W + ry[u] + EXT, zo = 2 * W + rz[u] + EXT;
        unsigned long long acc[W];
        int run = 0, cur = -1;
        auto flush = [&]() {
          if (run == 0) return;
          unsigned long long* c0 = tile64 + cur + roff[u];
          const unsigned long long off = (unsigned long long)(kFixMagicHi * (unsigned)run) << 32;
#pragma unroll
          for (int d = -EXT; d <= EXT; ++d)
            if ((d < 0 ? -d : d) <= h)
              __hip_atomic_fetch_add(c0 + d, acc[d + EXT] - off, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          run = 0;
        };
        for (int q = q0; q < q1; ++q) {
          const double* wp = wb + q * WS;
          const double m = amp[q];
          const int c = __builtin_amdgcn_readfirstlane(cell[q]);
          if (staged && fabs(m) < INFINITY) {
            if (c != cur || run == 0) {
              flush();
              cur = c;
#pragma unroll
              for (int d = 0; d < W; ++d) acc[d] = 0ull;
            }
            const double ayz = m * wp[yo] * wp[zo];
#pragma unroll
            for (int d = 0; d < W; ++d)
              acc[d] += (unsigned long long)__double_as_longlong(fma(ayz, wp[d], kFixMagic));
            ++run;
          } else if (h >= 0) {
            // no staging slot left (or a value that is not finite): FP32 adds to rho
            const double ayz = ldexp(m, -k) * wp[yo] * wp[zo];
            const int lz = c / PP, ly = (c - lz * PP) / RP, lx = c - lz * PP - ly * RP;
            const long long r = ((long long)wrapi(tz * kTile + lz - EXT + rz[u], N) * N +
                                 wrapi(ty * kTile + ly - EXT + ry[u], N)) * N;
            for (int d = -h; d <= h; ++d)
              unsafeAtomicAdd(&rho[r + wrapi(tx * kTile + lx - EXT + d, N)], (float)(ayz * wp[d + EXT]));
          }
        }
        flush();
      }
      __syncthreads();
    }
    if (staged) {
      // a tile of several pieces stages integers, summed exactly by the
      // reduction; a lone piece's box is already its tile's exact sum and is
      // staged as FP32 (the slot's first half), half the bytes
      const bool multi = pc_off[t + 1] - pc_off[t] > 1;
      long long* dst = stage + (size_t)p * TE3;
      float* dstf = reinterpret_cast<float*>(dst);
      for (int j = threadIdx.x; j < TE3; j += kDepNT) {
        const int lx = j % TE, ly = (j / TE) % TE, lz = j / (TE * TE);
        const long long v = (long long)tile64[lz * PP + ly * RP + lx];
        if (multi) dst[j] = v;
        else dstf[j] = (float)ldexp((double)v, -k);
      }
    }
  }
}

// Each listed tile: rho += the staged halo boxes of the pieces of its 27
// neighbouring tiles, one cell per thread.  A neighbour's pieces are summed
// exactly as integers (a lone piece read with the others' at once, 27
// independent loads with those outside a neighbour's box predicated off; the
// pieces of a dense neighbour eight loads at a time), each neighbour's sum is
// converted at its tile's scale, and the 27 values are added in a fixed
// order.  The
// owners of the densest tiles set the kernel's length, so a block keeps as
// many of their loads in flight as it can.
#ifndef PM_RED_NT
#define PM_RED_NT 512
#endif
constexpr int kRedNT = PM_RED_NT;
#ifndef PM_RED_LOADS
#define PM_RED_LOADS 8
#endif
constexpr int kRedLoads = PM_RED_LOADS;       // loads in flight per dense neighbour
static_assert(512 % kRedNT == 0, "a reduce block covers the 512 cells of a tile");
template <int EXT>
__global__ __launch_bounds__(kRedNT) void k_deposit_reduce(KernelGeom kg, const int* __restrict__ list,
                                                           const int* __restrict__ nlist,
                                                           const int* __restrict__ offsets,
                                                           const int* __restrict__ pc_off,
                                                           const unsigned* __restrict__ tmax, int nt, int N,
                                                           const long long* __restrict__ stage, int cap, float* rho) {
  constexpr int TE = kTile + 2 * EXT;
  constexpr int TE3 = TE * TE * TE;
  __shared__ int sq0[27], sq1[27], sk[27], smulti[27];
  const int n = *nlist;
  for (int li = blockIdx.x; li < n; li += gridDim.x) {
    const int t = list[li];
    const int tx = t % nt, ty = (t / nt) % nt, tz = t / (nt * nt);
    __syncthreads();                                // the previous tile's piece ranges are done with
    if (threadIdx.x < 27) {
      const int nb = threadIdx.x;
      const int dx = nb % 3 - 1, dy = (nb / 3) % 3 - 1, dz = nb / 9 - 1;
      const int u = ((((tz + dz) + nt) % nt) * nt + ((ty + dy) + nt) % nt) * nt + ((tx + dx) + nt) % nt;
      sq0[nb] = pc_off[u];
      sq1[nb] = min(pc_off[u + 1], cap);
      sk[nb] = tile_scale_exp(kg, tmax[u], offsets[u + 1] - offsets[u]);
      smulti[nb] = pc_off[u + 1] - pc_off[u] > 1;   // staged as integers
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 512 / kRedNT; ++h) {
      const int cell = threadIdx.x + h * kRedNT;    // 512 cells of the tile
      const int cx = cell & 7, cy = (cell >> 3) & 7, cz = cell >> 6;
      float v[27];
      static_for<0, 27>([&](auto NBc) {
        constexpr int nb = decltype(NBc)::value;
        constexpr int dx = nb % 3 - 1, dy = (nb / 3) % 3 - 1, dz = nb / 9 - 1;
        // this cell in the halo box of neighbour nb (origin at its corner minus EXT)
        const int lx = cx - dx * kTile + EXT, ly = cy - dy * kTile + EXT, lz = cz - dz * kTile + EXT;
        const bool in = lx >= 0 && lx < TE && ly >= 0 && ly < TE && lz >= 0 && lz < TE && sq0[nb] < sq1[nb] &&
                        !smulti[nb];
        v[nb] = in ? reinterpret_cast<const float*>(stage + (size_t)sq0[nb] * TE3)[(lz * TE + ly) * TE + lx] : 0.0f;
      });
      const long long g = ((long long)(tz * kTile + cz) * N + (ty * kTile + cy)) * N + (tx * kTile + cx);
      const float r0 = rho[g];
      // neighbours of one piece, from the loads above, in order; then those of
      // several pieces, whose integer boxes are summed here.  Which neighbours
      // have several pieces depends only on the tiles' particle counts, so the
      // order of the additions is fixed.
      float sum = 0.0f;
#pragma unroll
      for (int nb = 0; nb < 27; ++nb) sum += v[nb];
      for (int nb = 0; nb < 27; ++nb) {
        const int q1 = sq1[nb];
        int q = sq0[nb];
        if (!smulti[nb] || q >= q1) continue;
        const int dx = nb % 3 - 1, dy = (nb / 3) % 3 - 1, dz = nb / 9 - 1;
        const int lx = cx - dx * kTile + EXT, ly = cy - dy * kTile + EXT, lz = cz - dz * kTile + EXT;
        if (lx < 0 || lx >= TE || ly < 0 || ly >= TE || lz < 0 || lz >= TE) continue;
        // kRedLoads independent loads in flight; integer sums are exact in any order
        const long long* src = stage + (lz * TE + ly) * TE + lx;
        long long a[kRedLoads];
#pragma unroll
        for (int i = 0; i < kRedLoads; ++i) a[i] = 0;
        for (; q + kRedLoads - 1 < q1; q += kRedLoads) {
#pragma unroll
          for (int i = 0; i < kRedLoads; ++i) a[i] += src[(size_t)(q + i) * TE3];
        }
        for (; q < q1; ++q) a[0] += src[(size_t)q * TE3];
        long long tot = 0;
#pragma unroll
        for (int i = 0; i < kRedLoads; ++i) tot += a[i];
        sum += (float)ldexp((double)tot, -sk[nb]);
      }
      if (sum != 0.0f) rho[g] = r0 + sum;
    }
  }
}

// ---------------------------------------------------------------------------
// gather + push
// ---------------------------------------------------------------------------
// A piece loads its tile plus a halo of EXT + 1 cells of phi into LDS once.
// Its particles are then summed in one of two ways.
//  - One particle per lane (balls with a compiled shape R2): the dilated ball
//    is walked row by row (each wave takes every NW-th slice ez of the same 64
//    particles, so that a piece's time falls with the block's waves), v_e = phi(c + e) - phi(c).  With S_h = sum_{|e| <= h}
//    wx(e) v_e a row adds
//       x:  wy wz (sum_e v_e (wx(e - 1) - wx(e + 1)))
//       y:  wz (wy(ey - 1) S_{h(ey-1,ez)} - wy(ey + 1) S_{h(ey+1,ez)})
//       z:  wy (wz(ez - 1) S_{h(ey,ez-1)} - wz(ez + 1) S_{h(ey,ez+1)})
//    with w = 0 and h = -1 outside the ball: three FP32 instructions per cell
//    (the subtraction and two multiply-adds) and some twenty per row, where
//    products of three weights per cell take nine.
//  - One particle per wave (the last few particles of a piece, and the other
//    balls): lanes own the ball's rows (dy, dz) and step along dx together,
//       x: phi(dx + 1) - phi(dx - 1), and the differences of the rows next to
//    it in y and z, each times wx(dx); the rows are then summed over the wave.
//    Four threads per particle have put its weights into LDS before.
// A lane-per-particle pass over a compiled ball costs as much for one particle
// as for 64, so the remainder of a piece goes by rows up to kRowMost particles
// (the costs cross near 14 to 18 particles for the three compiled balls).
// Bound: vector instructions at full waves, the serial length of a ball at few
// particles.  65 537 particles of a mixture at sigma = 2 in a 256^3 box: a
// smooth_accel call takes 134 us, 3000 us with one wave per particle reading
// six neighbours per cell from memory; the ring (4097 particles, sigma = 1.5)
// gathers and pushes in 47 us instead of 115 with a lane per particle alone.

// Acceleration from the summed differences, then the store or the push.
__device__ __forceinline__ void gather_out(const KernelGeom& kg, int64_t i, double norm, float gx, float gy, float gz,
                                           float* pos, float* vel, float* acc, float dt_kick, float dt_drift,
                                           int mode) {
  const float f = (float)(-1.0 / (2.0 * (double)kg.s * norm));
  const float ax = gx * f, ay = gy * f, az = gz * f;
  if (mode == 0) {
    acc[3 * i] = ax;
    acc[3 * i + 1] = ay;
    acc[3 * i + 2] = az;
  } else {
    const float vx = fmaf(ax, dt_kick, vel[3 * i]);
    const float vy = fmaf(ay, dt_kick, vel[3 * i + 1]);
    const float vz = fmaf(az, dt_kick, vel[3 * i + 2]);
    vel[3 * i] = vx; vel[3 * i + 1] = vy; vel[3 * i + 2] = vz;
    pos[3 * i] = fmaf(vx, dt_drift, pos[3 * i]);
    pos[3 * i + 1] = fmaf(vy, dt_drift, pos[3 * i + 1]);
    pos[3 * i + 2] = fmaf(vz, dt_drift, pos[3 * i + 2]);
  }
}

// Sums the lane's particle over the dilated ball (compiled shape), base: its
// central cell in the LDS tile: g = the three sums and the ball sum S of the
// weights over the slices ez this wave owns (every NW-th).  The weights of the differences sum to zero
// over the ball, so phi is taken relative to its value at the central pixel.
// A row is summed in FP32 relative to its own middle cell, whose offset from
// the centre enters with the row's weight sum in FP64, and the rows are added
// in FP64: FP32 throughout loses two bits to the offsets that cancel between
// rows (1.9e-7 against 5e-8 of the force at sigma = 2), this form none (8e-9).
template <int EXT, int R2, int RP, int PP, int NW>
__device__ __forceinline__ void lane_gather(const Lane<EXT>& L, const float* base, int wave, double* g) {
  constexpr int HE = EXT + 1;
  const float phc = base[0];
  float wd[2 * EXT + 1];                          // wx(e - 1) - wx(e + 1), |e| < EXT
#pragma unroll
  for (int e = 1; e < 2 * EXT; ++e) wd[e] = L.wx[e - 1] - L.wx[e + 1];
  double gx = 0.0, gy = 0.0, gz = 0.0, S = 0.0;
  static_for<-HE, HE + 1>([&](auto EZc) {
    constexpr int ez = decltype(EZc)::value;
    if ((ez + HE) % NW != wave) return;
    // weights of the slices ez, ez - 1 and ez + 1 (0 outside the ball)
    const double wz = ez >= -EXT && ez <= EXT ? (double)L.wz[ez >= -EXT && ez <= EXT ? ez + EXT : 0] : 0.0;
    const double wzm = ez - 1 >= -EXT ? (double)L.wz[ez - 1 >= -EXT ? ez - 1 + EXT : 0] : 0.0;
    const double wzp = ez + 1 <= EXT ? (double)L.wz[ez + 1 <= EXT ? ez + 1 + EXT : 0] : 0.0;
    double sx = 0.0, sy = 0.0, sw = 0.0;          // the slice's sums of x, y and the weights
    static_for<-HE, HE + 1>([&](auto EYc) {
      constexpr int ey = decltype(EYc)::value;
      constexpr auto half = [](int y, int z) constexpr {
        return y < -EXT || y > EXT || z < -EXT || z > EXT ? -1 : row_half(y, z, R2, EXT);
      };
      constexpr int h = half(ey, ez);
      constexpr int hym = half(ey - 1, ez), hyp = half(ey + 1, ez), hzm = half(ey, ez - 1), hzp = half(ey, ez + 1);
      constexpr int hy = hym > hyp ? hym : hyp, hz = hzm > hzp ? hzm : hzp;
      constexpr int hs = hy > hz ? hy : hz;                     // cells the sums S need
      constexpr int m = h >= 0 && h + 1 > hs ? h + 1 : hs;      // cells read
      if constexpr (m >= 0) {
        const float* row = base + ez * PP + ey * RP;
        const float r0 = row[0];
        float v[2 * m + 1];
        v[m] = 0.0f;
        static_for<1, m + 1>([&](auto Ec) {
          constexpr int e = decltype(Ec)::value;
          v[m - e] = row[-e] - r0;
          v[m + e] = row[e] - r0;
        });
        if constexpr (h >= 0) {
          float t = 0.0f;
          static_for<-h - 1, h + 2>([&](auto Ec) {
            constexpr int e = decltype(Ec)::value;
            // wx(e - 1) and wx(e + 1) where they lie in the row
            if constexpr (e == 0) {}
            else if constexpr (e - 1 >= -h && e + 1 <= h) t = fmaf(v[e + m], wd[e + EXT], t);
            else if constexpr (e - 1 >= -h && e - 1 <= h) t = fmaf(v[e + m], L.wx[e - 1 + EXT], t);
            else if constexpr (e + 1 >= -h && e + 1 <= h) t = fmaf(v[e + m], -L.wx[e + 1 + EXT], t);
          });
          sx = fma((double)t, (double)L.wy[h >= 0 ? ey + EXT : 0], sx);
          sw = fma((double)L.wy[h >= 0 ? ey + EXT : 0], L.sx[h >= 0 ? h : 0], sw);
        }
        if constexpr (hs >= 0) {
          float s[hs + 1];
          s[0] = 0.0f;
          static_for<1, hs + 1>([&](auto Ec) {
            constexpr int e = decltype(Ec)::value;
            s[e] = fmaf(v[m - e], L.wx[EXT - e], fmaf(v[m + e], L.wx[EXT + e], s[e - 1]));
          });
          const double off = (double)(r0 - phc);
          auto Sh = [&](auto Hc) {
            constexpr int k = decltype(Hc)::value;
            return fma(off, L.sx[k], (double)s[k]);
          };
          if constexpr (hym >= 0) sy = fma((double)L.wy[hym >= 0 ? ey - 1 + EXT : 0], Sh(std::integral_constant<int, hym >= 0 ? hym : 0>{}), sy);
          if constexpr (hyp >= 0) sy = fma(-(double)L.wy[hyp >= 0 ? ey + 1 + EXT : 0], Sh(std::integral_constant<int, hyp >= 0 ? hyp : 0>{}), sy);
          if constexpr (hz >= 0) {
            double t = 0.0;
            if constexpr (hzm >= 0) t = wzm * Sh(std::integral_constant<int, hzm >= 0 ? hzm : 0>{});
            if constexpr (hzp >= 0) t = fma(-wzp, Sh(std::integral_constant<int, hzp >= 0 ? hzp : 0>{}), t);
            gz = fma(t, (double)L.wy[hz >= 0 ? ey + EXT : 0], gz);
          }
        }
      }
    });
    gx = fma(sx, wz, gx);
    gy = fma(sy, wz, gy);
    S = fma(sw, wz, S);
  });
  g[0] = gx;
  g[1] = gy;
  g[2] = gz;
  g[3] = S;
}

// Floats of LDS before the tile: the lane pass's sums or the row pass's weights.
template <int EXT>
constexpr int gather_scratch() {
  constexpr int nt = gather_nt(EXT);
  constexpr int a = nt / 64 * 4 * 64 * 2, b = nt / 4 * (3 * (2 * EXT + 1) + 1);
  return (a > b ? a : b) + 1 & ~1;
}

// R2 = 0: a ball without a compiled shape, all particles by rows.
template <int EXT, int R2>
__global__ __launch_bounds__(gather_nt(EXT)) void k_gather_pieces(KernelGeom kg, const int* __restrict__ perm,
                                                       const int* __restrict__ offsets,
                                                       const int* __restrict__ pc_off,
                                                       const int* __restrict__ ptile, int ntiles, int piece,
                                                       int* counter, const float* __restrict__ phi, float* pos,
                                                       float* vel, float* acc, float dt_kick, float dt_drift,
                                                       int mode) {
  constexpr int HE = EXT + 1;                      // ball plus the difference stencil
  constexpr int TE = kTile + 2 * HE;
  constexpr int RP = TE + 1, PP = RP * TE + 1;     // padded row and plane pitches
  constexpr int W = 2 * EXT + 1, WS = 3 * W + 1;
  constexpr int RU = (W * W + 63) / 64;            // rows per lane, at most
  constexpr int kGatNT = gather_nt(EXT), NW = kGatNT / 64;
  constexpr int kRowBatch = kGatNT / 4;            // particles whose weights LDS holds at once
  extern __shared__ double gsm[];
  double* red = gsm;                               // [NW][4][64] sums of the lane pass, or
  float* wbuf = reinterpret_cast<float*>(gsm);     // [kRowBatch][WS] weights of the row pass
  float* tile = reinterpret_cast<float*>(gsm) + gather_scratch<EXT>();
  __shared__ double norm[kRowBatch];
  __shared__ int cell[kRowBatch];
  __shared__ int hrow[W * W];
  __shared__ int slot;
  const int N = kg.N, nt = N / kTile;
  const int total = pc_off[ntiles];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int roff[RU], rh[RU], ry[RU], rz[RU];
  ball_rows<EXT, RU>(kg, kGatNT, RP, PP, hrow, roff, rh, ry, rz);
  for (int p = next_piece(counter, &slot); p < total; p = next_piece(counter, &slot)) {
    const int t = ptile[p];
    const int a = offsets[t] + (p - pc_off[t]) * piece;
    const int b = min(a + piece, offsets[t + 1]);
    const int tx = t % nt, ty = (t / nt) % nt, tz = t / (nt * nt);
    const int ox = tx * kTile - HE, oy = ty * kTile - HE, oz = tz * kTile - HE;
#pragma unroll 8
    for (int j = threadIdx.x; j < TE * TE * TE; j += kGatNT) {
      const int lx = j % TE, ly = (j / TE) % TE, lz = j / (TE * TE);
      tile[lz * PP + ly * RP + lx] =
          phi[((long long)wrapi(oz + lz, N) * N + wrapi(oy + ly, N)) * N + wrapi(ox + lx, N)];
    }
    __syncthreads();
    const int tail = (b - a) & 63;
    const int mid = R2 == 0 ? a : (tail > kRowMost ? b : b - tail);
    if constexpr (R2 > 0) {
      // 64 particles at a time, one per lane, the ball's slices dealt to the waves
      for (int j0 = a; j0 < mid; j0 += 64) {
        const int64_t i = perm[min(j0 + lane, mid - 1)];
        Lane<EXT> L;
        lane_setup<EXT>(L, kg, pos[3 * i], pos[3 * i + 1], pos[3 * i + 2]);
        const int lx = (L.cx & (kTile - 1)) + HE, ly = (L.cy & (kTile - 1)) + HE, lz = (L.cz & (kTile - 1)) + HE;
        double g[4];
        lane_gather<EXT, R2, RP, PP, NW>(L, tile + lz * PP + ly * RP + lx, wave, g);
#pragma unroll
        for (int c = 0; c < 4; ++c) red[(wave * 4 + c) * 64 + lane] = g[c];
        __syncthreads();
        if (wave == 0 && j0 + lane < mid) {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            for (int w = 1; w < NW; ++w) g[c] += red[(w * 4 + c) * 64 + lane];
          gather_out(kg, i, kg.analytic ? kg.analytic_norm : g[3], (float)g[0], (float)g[1], (float)g[2], pos, vel, acc,
                     dt_kick, dt_drift, mode);
        }
        __syncthreads();
      }
    }
    for (int j0 = mid; j0 < b; j0 += kRowBatch) {
      const int count = min(kRowBatch, b - j0);
      weights_to_lds<EXT, kGatNT>(kg, pos, count, HE, RP, PP, hrow, wbuf, norm, cell, [&](int q) { return perm[j0 + q]; });
      for (int k = wave; k < count; k += kGatNT / 64) {
        const float* wp = wbuf + k * WS;
        const float* c0 = tile + cell[k];
        float gx = 0.0f, gy = 0.0f, gz = 0.0f;
#pragma unroll
        for (int u = 0; u < RU; ++u) {
          if (64 * u >= kg.nrows) break;
          const float* r = c0 + roff[u];
          float sx = 0.0f, sy = 0.0f, sz = 0.0f;
          float vm = r[-EXT - 1], v0 = r[-EXT];
#pragma unroll
          for (int dx = -EXT; dx <= EXT; ++dx) {
            const float vp = r[dx + 1];
            const float w = (dx < 0 ? -dx : dx) <= rh[u] ? wp[dx + EXT] : 0.0f;
            sx = fmaf(w, vp - vm, sx);
            sy = fmaf(w, r[dx + RP] - r[dx - RP], sy);
            sz = fmaf(w, r[dx + PP] - r[dx - PP], sz);
            vm = v0;
            v0 = vp;
          }
          const float wyz = wp[W + ry[u] + EXT] * wp[2 * W + rz[u] + EXT];
          gx = fmaf(wyz, sx, gx);
          gy = fmaf(wyz, sy, gy);
          gz = fmaf(wyz, sz, gz);
        }
        for (int o = 32; o > 0; o >>= 1) {
          gx += __shfl_xor(gx, o, 64);
          gy += __shfl_xor(gy, o, 64);
          gz += __shfl_xor(gz, o, 64);
        }
        if (lane == 0) gather_out(kg, perm[j0 + k], norm[k], gx, gy, gz, pos, vel, acc, dt_kick, dt_drift, mode);
      }
      __syncthreads();
    }
  }
}

// Grid sizes of the persistent kernels.
constexpr int kPersistBlocks = 2048;
}  // namespace

template <int EXT>
static constexpr size_t deposit_lds() {
  return sizeof(double) * (DepTile<EXT>::cells + (size_t)kDepBatch * (3 * (2 * EXT + 1) + 1));
}
template <int EXT>
static constexpr size_t gather_lds() {
  constexpr int TE = kTile + 2 * (EXT + 1);
  return sizeof(float) * ((size_t)TE * ((TE + 1) * TE + 1) + gather_scratch<EXT>());
}

size_t piece_stage_cells(int ext, int cap) {
  const size_t te = kTile + 2 * (size_t)ext;
  return (size_t)cap * te * te * te;
}

hipError_t deposit_pieces(const KernelGeom& kg, const SortBufs& sb, const PieceBufs& pb, const float* pos,
                          const float* mass, int64_t n, float* rho, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (kg.piece > kMaxPiece) return hipErrorInvalidValue;
  const int nt = kg.N / kTile;
  hipLaunchKernelGGL(k_tile_mass_max, dim3(kPersistBlocks), dim3(kNT), 0, st, sb.perm, sb.offsets, pb.pc_off, pb.ptile,
                     sb.ntiles, kg.piece, mass, pb.tmax);
#define DEPOSIT(EXT, R2)                                                                                            \
  hipLaunchKernelGGL((k_deposit_pieces<EXT, R2>), dim3(kPersistBlocks), dim3(kDepNT), deposit_lds<EXT>(), st, kg,      \
                     sb.perm, sb.offsets, pb.pc_off, pb.ptile, sb.ntiles, pb.counter, pos, mass, pb.tmax, pb.stage, \
                     pb.cap, rho);                                                                                 \
  hipLaunchKernelGGL((k_deposit_reduce<EXT>), dim3(kPersistBlocks), dim3(kRedNT), 0, st, kg, pb.list,              \
                     pb.list_off + sb.ntiles, sb.offsets, pb.pc_off, pb.tmax, nt, kg.N, pb.stage, pb.cap, rho)
  switch (kg.plan_ext) {
    case 1: DEPOSIT(1, 0); break;
    case 2: DEPOSIT(2, 0); break;
    case 3:
      if (kg.nball == 251) { DEPOSIT(3, 16); } else { DEPOSIT(3, 0); }
      break;
    case 4: DEPOSIT(4, 0); break;
    case 5: DEPOSIT(5, 0); break;
    case 6: DEPOSIT(6, 0); break;
    case 7: DEPOSIT(7, 0); break;
    case 8: DEPOSIT(8, 0); break;
    default: return hipErrorInvalidValue;
  }
#undef DEPOSIT
  return hipGetLastError();
}

hipError_t gather_pieces(const KernelGeom& kg, const SortBufs& sb, const PieceBufs& pb, const float* phi,
                         float* pos, float* vel, float* acc, int64_t n, float dt_kick, float dt_drift, int mode,
                         hipStream_t st) {
  if (n <= 0) return hipSuccess;
#define GATHER(EXT, R2)                                                                                            \
  hipLaunchKernelGGL((k_gather_pieces<EXT, R2>), dim3(kPersistBlocks), dim3(gather_nt(EXT)), gather_lds<EXT>(), st, kg,    \
                     sb.perm, sb.offsets, pb.pc_off, pb.ptile, sb.ntiles, kg.piece, pb.counter + 1, phi, pos, vel, \
                     acc, dt_kick, dt_drift, mode)
  switch (kg.plan_ext) {
    case 1: GATHER(1, 0); break;
    case 2: GATHER(2, 0); break;
    case 3: if (kg.nball == 251) GATHER(3, 16); else GATHER(3, 0); break;
    case 4: GATHER(4, 0); break;
    case 5: if (kg.nball == 895) GATHER(5, 36); else GATHER(5, 0); break;
    case 6: GATHER(6, 0); break;
    case 7: if (kg.nball == 2103) GATHER(7, 64); else GATHER(7, 0); break;
    case 8: GATHER(8, 0); break;
    default: return hipErrorInvalidValue;
  }
#undef GATHER
  return hipGetLastError();
}

}  // namespace pm
