"""Solves in potential form (two spectra through the z passes) at every box
size with a thread layout of its own, and the warm start from the kept
spectrum of F, against the FP64 oracle on the same FP32 inputs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pm as orc  # noqa: E402
import workloads as W  # noqa: E402
from tests.gpu_util import dev, grid, host, oparams, rel_l2, rel_max  # noqa: E402

pytestmark = pytest.mark.gpu

# the stated target of the potential and the force in FP32
TOL = 1e-5


@pytest.fixture(scope="module")
def M():
    from paper_2312_02968_amd import mondpm
    return mondpm


def _case(N, K, flags=0, n=None):
    w = W.random_cloud(N, n or N // 2, 200, iters=K, radius_frac=0.25, n_pad=N)
    p = dict(w["params"], flags=flags)
    rho = orc.deposit(oparams(p), w["pos"].astype(np.float64), w["mass"].astype(np.float64)).astype(np.float32)
    return p, rho


@pytest.mark.parametrize("N,K", [(16, 3), (32, 1), (32, 3), (64, 2), (128, 2), (256, 2)])
def test_solve_every_layout(M, N, K):
    print("solve", N, K, flush=True)
    p, rho = _case(N, K)
    ctx = M.pm_create(p, 0)
    phi = grid(N)
    M.aqual_solve(ctx, dev(rho.ravel()), phi, want_info=False)
    ref, _ = orc.aqual_solve(oparams(p), rho.astype(np.float64))
    got = host(phi).reshape(ref.shape)
    assert rel_l2(got, ref) < TOL and rel_max(got, ref) < TOL
    ctx.close()


@pytest.mark.parametrize("N", [16, 64, 128])
@pytest.mark.parametrize("K", [2, 3])
def test_warm_start_from_the_kept_spectrum(M, N, K):
    """Three solves in a row; each oracle solve starts from the H of the one
    before.  The field entry point on the same context returns that F."""
    print("warm", N, K, flush=True)
    p, rho = _case(N, K, flags=M.PM_F_WARM_START)
    op = oparams(p)
    ctx = M.pm_create(p, 0)
    phi, F = grid(N), torch.zeros(3 * N ** 3, device="cuda")
    H = None
    for step in range(3):
        r = (rho * (1.0 + 0.1 * step)).astype(np.float32)
        if step == 1:
            M.aqual_solve_field(ctx, dev(r.ravel()), phi, F, want_info=False)
        else:
            M.aqual_solve(ctx, dev(r.ravel()), phi, want_info=False)
        if H is not None:
            _, gN = orc.newton_potential(op, r.astype(np.float64))
            H = H + gN_prev - gN                        # H0 = F_prev - g_N; the oracle projects it
        ref, info = orc.aqual_solve(op, r.astype(np.float64), H, keep_fields=True)
        got = host(phi).reshape(ref.shape)
        assert rel_l2(got, ref) < TOL and rel_max(got, ref) < TOL, step
        H, gN_prev = info.H, info.gN
        if step == 1:
            assert rel_l2(host(F).reshape(H.shape), H + gN_prev) < TOL
    ctx.close()


def test_start_in_component_form_then_potential_form(M):
    """A given H0 enters in component form; the later iterations take S from it."""
    N = 64
    p, rho = _case(N, 3)
    rng = np.random.default_rng(5)
    H0 = (rng.standard_normal((3, N, N, N)) * 1e-3).astype(np.float32)
    ctx = M.pm_create(p, 0)
    phi = grid(N)
    M.aqual_solve(ctx, dev(rho.ravel()), phi, H0=dev(H0.ravel()), want_info=False)
    ref, _ = orc.aqual_solve(oparams(p), rho.astype(np.float64), H0.astype(np.float64))
    got = host(phi).reshape(ref.shape)
    assert rel_l2(got, ref) < TOL and rel_max(got, ref) < TOL
    ctx.close()
