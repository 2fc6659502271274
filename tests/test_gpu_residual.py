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


def detect_and_compare(ocd, B, U, W, S, Q, K, mode, snr, seed, plan):
    residual(B, U, W, S, K)
    say("residual case", B, U, W, S, Q, K, mode, plan)
    wl = synth.make_workload(B, U, W, S, Q, snr, seed=seed)
    N0 = float(np.float32(wl["N0"]))
    pb = ocd.problem(B, U, W, S, Q, K, mode, "f32", N0)
    ocd.ocd_set_plan(pb, ocd.Plan(*(tuple(plan) + (0,) * (5 - len(plan)))))
    H, y = dev(wl["H"]), dev(wl["y"])
    z, L, _ = ocd.detect(H, y, K, Q, mode, N0)
    z2, L2, zh = ocd.detect(H, y, K, Q, mode, N0, want_hist=True)
    torch.cuda.synchronize()
    zo, Lo, zho = oracle_ref(wl["H"], wl["y"], K, Q, mode, N0, hist=True)
    assert z_rel_err(host(z), zo) <= Z_TOL_F32
    assert llr_rel_err(host(L), Lo) <= LLR_TOL_F32
    assert torch.equal(z, z2) and torch.equal(L, L2)
    for k in range(K):
        assert z_rel_err(host(zh)[:, :, k], zho[:, :, k]) <= Z_TOL_F32


@pytest.mark.parametrize("case", [
    (64, 24, 9, 3, 4, 2, "box", (8, 16, 0)), (60, 32, 5, 4, 6, 2, "mmse", (8, 8, 1)),
    (100, 24, 6, 2, 2, 1, "box", (16, 4, 0)), (120, 32, 3, 5, 4, 1, "box", (16, 5, 0, 0, 1)),
    (28, 16, 9, 3, 6, 4, "mmse", (4, 16, 0)), (63, 32, 5, 4, 4, 4, "box", (8, 8, 1)),
])
def test_chunked_user_loop(ocd, case):
    """Multiples of 8 users with at most 8 entries a lane: unrolled chunks of 8 users."""
    B, U, W, S, Q, K, mode, plan = case
    detect_and_compare(ocd, B, U, W, S, Q, K, mode, 15.0, [218, B, U], plan)


PLANS = [(4, 14, 0), (4, 16, 1), (8, 28, 0), (8, 64, 1), (16, 32, 0), (16, 14, 1), (16, 14, 0),
         (16, 28, 1), (16, 14, 1, 0, 4), (8, 28, 0, 0, 1), (16, 16, 1, 0, 2), (32, 16, 1)]


SHAPES_AND_PLANS = [(s, p) for s in ((8, 60, 14, 1), (7, 60, 14, 2)) for p in PLANS] + [
    ((8, 60, 2, 3), p) for p in ((4, 4, 0), (8, 6, 1), (16, 14, 1), (16, 5, 0, 0, 2), (32, 8, 1))]


@pytest.mark.parametrize("shape,plan", SHAPES_AND_PLANS)
def test_every_plan(ocd, shape, plan):
    """128 antennas under every lane split, tile size, tile order and staggering: 8 unrolled
    users and the run-time loop, subcarriers whole and split over workgroups."""
    U, W, S, K = shape
    detect_and_compare(ocd, 128, U, W, S, 6, K, "mmse", 20.0, [219, U, S], plan)


@pytest.mark.parametrize("plan", [(16, 14, 1, 0, 0), (16, 14, 1, 0, 2), (16, 16, 1, 0, 0), (16, 16, 1, 0, 2)])
def test_whole_slot(ocd, plan):
    """A slot of 1200 x 14 vectors, one sweep, on the tile shapes that fill the GPU."""
    detect_and_compare(ocd, 128, 8, 1200, 14, 6, 1, "mmse", 20.0, [220, 0], plan)


# B, U, W, K at 14 symbols: both many antennas, where the lane modes differ, and few
JOBS = [(64, 4, 21, 3), (128, 8, 30, 1), (256, 5, 5, 3), (128, 16, 11, 1), (120, 32, 4, 1),
        (256, 16, 7, 1), (33, 5, 6, 3), (96, 24, 4, 1), (200, 7, 9, 2), (256, 8, 6, 1), (15, 8, 5, 4)]


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("persistent", [False, True])
def test_jobs_every_lane_mode(ocd, mode, persistent):
    """The batched launch's residual tiles in every lane mode and both schedules, beside one
    job of the Gram form: against the oracle, and bit for bit against a launch of the job's
    own with the same lanes per vector."""
    say("residual jobs, lane mode %d persistent %s" % (mode, persistent))
    S, Q, probs, Hs, ys, wls = 14, 6, [], [], [], []
    for j, (B, U, W, K) in enumerate(JOBS + [(64, 8, 9, 3)]):
        if j < len(JOBS):
            residual(B, U, W, S, K)
        wl = synth.make_workload(B, U, W, S, Q, 20.0, seed=[221, j])
        probs.append(ocd.problem(B, U, W, S, Q, K, "mmse", "f32", float(np.float32(wl["N0"]))))
        Hs.append(dev(wl["H"]))
        ys.append(dev(wl["y"]))
        wls.append(wl)
    flags = ocd.OCD_JOBS_LANE_MODE(mode) | (ocd.OCD_JOBS_PERSISTENT if persistent else 0)
    z, L, _ = ocd.detect_jobs(probs, Hs, ys, flags=flags)
    torch.cuda.synchronize()
    for j, (pb, wl) in enumerate(zip(probs, wls)):
        zo, Lo, _ = oracle_ref(wl["H"], wl["y"], pb.K, pb.Q, "mmse", pb.N0)
        assert z_rel_err(host(z[j]), zo) <= Z_TOL_F32, j
        assert llr_rel_err(host(L[j]), Lo) <= LLR_TOL_F32, j
        if pb.B <= 16:
            continue   # zero-padded to 4 lanes of 8 entries, which no plan of one problem is
        npl = 16 if mode >= 1 and pb.B > 128 else 4 if mode == 2 and pb.B > 32 else 8
        lanes = 4
        while npl * lanes < pb.B:
            lanes *= 2
        if npl != 8 and lanes not in (16, 32):
            npl, lanes = 8, 4
            while 8 * lanes < pb.B:
                lanes *= 2
        ocd.ocd_set_plan(pb, ocd.Plan(lanes, 14, 0, 0))
        z1, L1, _ = ocd.detect(Hs[j], ys[j], pb.K, pb.Q, "mmse", pb.N0)
        torch.cuda.synchronize()
        assert torch.equal(z1, z[j]) and torch.equal(L1, L[j]), (j, lanes, npl)


@pytest.mark.parametrize("B,U,W,S,K,mode", [
    (128, 8, 12, 14, 1, "hybrid"), (64, 24, 5, 3, 2, "box"), (128, 7, 9, 14, 2, "mmse"),
    (60, 32, 4, 3, 2, "hybrid"), (28, 16, 6, 4, 4, "hybrid"), (128, 9, 9, 2, 2, "box")])
def test_gradients(ocd, B, U, W, S, K, mode):
    """Training step and adjoint: z, LLRs and dy bit for bit as in the two launches, the
    gradients against the oracle's reverse mode."""
    residual(B, U, W, S, K)
    gradients_against_oracle(ocd, B, U, W, S, 4, K, mode)


@pytest.mark.parametrize("B,U,W,S,K", [(32, 8, 600, 14, 2), (24, 12, 300, 17, 4), (34, 17, 520, 9, 8)])
def test_gradients_where_detection_alone_is_in_the_gram_form(ocd, B, U, W, S, K):
    """Past two tiles a compute unit these shapes detect in the Gram form, and in the residual
    form for the gradients: the detection that keeps the history has the gradients' bits."""
    assert bench.gram_form(B, U, W, S, K)
    gradients_against_oracle(ocd, B, U, W, S, 4, K, "hybrid")


def gradients_against_oracle(ocd, B, U, W, S, Q, K, mode):
    say("residual gradients", B, U, W, S, Q, K, mode)
    wl = synth.make_workload(B, U, W, S, Q, 10.0, seed=[222, B, U, S])
    N0 = float(np.float32(wl["N0"]))
    lam = (N0 * np.linspace(0.8, 1.3, K)).astype(np.float32) if mode == "hybrid" else None
    beta = 0.0 if mode == "mmse" else float(np.float32(0.8))
    H, y, bits = dev(wl["H"]), dev(wl["y"]), torch.from_numpy(wl["bits"]).cuda()
    kw = dict(lam=None if lam is None else dev(lam))
    z2, L2, zh = ocd.detect(H, y, K, Q, mode, N0, 1.0, beta, want_hist=True, **kw)
    dlam2, dbeta2, dy2 = ocd.backward(H, y, zh, None, K, Q, mode, N0, 1.0, beta, bits=bits, **kw)
    loss, dlam, dbeta, dy, z, L = ocd.train_step(H, y, bits, K, Q, mode, N0, 1.0, beta,
                                                 want_z=True, want_llr=True, **kw)
    z1, _, _ = ocd.detect(H, y, K, Q, mode, N0, 1.0, beta, **kw)
    torch.cuda.synchronize()
    assert torch.equal(z, z2) and torch.equal(L, L2) and torch.equal(dy, dy2)
    assert z_rel_err(host(z1), host(z).astype(np.complex128)) <= 2 * Z_TOL_F32
    zo, _, _ = oracle_ref(wl["H"], wl["y"], K, Q, mode, N0, 1.0, lam, beta)
    assert z_rel_err(host(z), zo) <= Z_TOL_F32
    Lh = host(L).astype(np.float64)
    dllr = (1.0 / (1.0 + np.exp(-Lh)) - wl["bits"]) / Lh.size
    dlam_o, dbeta_o, dy_o = oracle.grad(wl["H"], wl["y"], dllr, K, Q, mode, N0=N0, lam=lam, beta=beta)
    for name, a, b in (("dlam", dlam, dlam_o), ("dlam2", dlam2, dlam_o), ("dy", dy, dy_o)):
        a, b = host(a).ravel(), np.asarray(b).ravel()
        assert np.linalg.norm(a - b) <= GRAD_TOL * np.linalg.norm(b), name
    if mode != "mmse":
        for b in (dbeta, dbeta2):
            assert abs(float(host(b)[0]) - dbeta_o) <= GRAD_TOL * abs(dbeta_o)
    want = np.mean(np.logaddexp(0.0, np.where(wl["bits"] != 0, -Lh, Lh)))
    assert abs(float(host(loss)[0]) - want) <= 1e-5 * want
