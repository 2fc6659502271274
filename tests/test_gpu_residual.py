"""GPU parity of the kernels that update the residual (k_forward, k_backward, k_train, k_jobs)
on shapes that they run, which are those outside the Gram form: every case says so first, so
that a change of that rule cannot leave them untested."""

import numpy as np
import pytest
import torch

import bench
import oracle
import synth
from gpu_util import (LLR_TOL_F32, Z_TOL_F32, dev, host, llr_rel_err, oracle_ref, say, z_rel_err)

pytestmark = pytest.mark.gpu

GRAD_TOL = 1e-3


@pytest.fixture(scope="module")
def ocd():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1611_08779_amd as m
    return m


def residual(B, U, W, S, K):
    assert not bench.gram_form(B, U, W, S, K), "a shape of the Gram form"


@pytest.mark.parametrize("mode", ["mmse", "hybrid"])
def test_adjoint_fits_the_lds_of_every_shape(ocd, mode):
    """The adjoint's plan leaves room for the kernel's own LDS: no shape whose tiles come
    close to the limit of a workgroup is refused at the launch."""
    W, Q, K = 2, 2, 1
    refused = []
    for B in (16, 24, 32, 40, 48, 64, 80, 96, 100, 128, 200, 256):
        for U in (2, 5, 8, 12, 16, 20, 24, 31, 32):
            for S in (1, 2, 3, 4, 7, 14):
                if U > B or bench.gram_form(B, U, W, S, K):
                    continue
                H = torch.randn(W, U, B, dtype=torch.complex64, device="cuda")
                y = torch.randn(W, S, B, dtype=torch.complex64, device="cuda")
                lam = torch.full((K,), 0.1, device="cuda")
                zh = torch.zeros(W, S, K, U, dtype=torch.complex64, device="cuda")
                dllr = torch.zeros(W, S, U, Q, device="cuda")
                try:
                    ocd.backward(H, y, zh, dllr, K, Q, mode, 0.1, 1.0, 0.9, lam=lam)
                except ocd.OCDError as e:
                    refused.append((B, U, S, e.status))
    torch.cuda.synchronize()
    assert not refused, refused


def test_adjoint_close_to_the_lds_limit(ocd):
    B, U, W, S, Q, K = 64, 24, 5, 2, 4, 1
    residual(B, U, W, S, K)
    wl = synth.make_workload(B, U, W, S, Q, 10.0, seed=[217, 0])
    N0, beta = float(np.float32(wl["N0"])), float(np.float32(0.9))
    lam = np.array([0.7 * N0], np.float32)
    H, y, lt = dev(wl["H"]), dev(wl["y"]), dev(lam)
    _, L, zh = ocd.detect(H, y, K, Q, "hybrid", N0, 1.0, beta, lam=lt, want_hist=True)
    dllr = torch.randn(W, S, U, Q, generator=torch.Generator().manual_seed(3)).cuda()
    dlam, _, dy = ocd.backward(H, y, zh, dllr, K, Q, "hybrid", N0, 1.0, beta, lam=lt)
    torch.cuda.synchronize()
    dlam_o, _, dy_o = oracle.grad(wl["H"], wl["y"], host(dllr), K, Q, "hybrid", N0=N0, lam=lam, beta=beta)
    for a, b in ((dlam, dlam_o), (dy, dy_o)):
        a, b = host(a).ravel(), np.asarray(b).ravel()
        assert np.linalg.norm(a - b) <= GRAD_TOL * np.linalg.norm(b)
