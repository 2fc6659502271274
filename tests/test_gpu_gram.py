"""GPU parity of the Gram form of the detection (ocd_gram.h) at the sizes where its
tiles, antenna blocks and lane groups end: users around 8, 16 and 32, symbols around 8
and 16, antennas around whole blocks and around the changes of its summation length,
rows that are not 16-byte aligned, every option of the call, one and four waves per
subcarrier, and its gradients.  Against the FP64 oracle on the values the GPU received,
with the bars of the FP32 path."""

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import (LLR_TOL_F32, Z_TOL_F32, dev, from_f16_pairs, host, llr_rel_err, oracle_ref,
                      say, to_f16_pairs, z_rel_err)

pytestmark = pytest.mark.gpu

GRAD_TOL = 1e-3


@pytest.fixture(scope="module")
def ocd():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1611_08779_amd as m
    return m


CASES = [
    # B, U, W, S, Q, K, mode, storage: a tile's last user, symbol or antenna, and the next
    (16, 8, 5, 3, 4, 3, "mmse", "f32"), (18, 9, 4, 8, 6, 3, "box", "f32"),
    (32, 16, 3, 9, 2, 4, "mmse", "f16"), (34, 17, 3, 16, 4, 8, "box", "f32"),
    (64, 32, 2, 17, 6, 2, "mmse", "f32"), (62, 31, 2, 8, 4, 3, "hybrid", "f16"),
    (2, 1, 7, 3, 2, 16, "box", "f32"), (63, 4, 5, 14, 6, 4, "mmse", "f32"),
    (65, 12, 3, 33, 4, 2, "box", "f16"), (127, 8, 4, 14, 6, 3, "mmse", "f32"),
    (128, 8, 4, 14, 6, 3, "hybrid", "f16"), (130, 20, 3, 5, 4, 3, "box", "f32"),
    (136, 32, 2, 15, 2, 4, "hybrid", "f32"), (264, 3, 4, 1, 4, 6, "mmse", "f32"),
    (100, 12, 6, 1, 4, 3, "box", "f32"), (96, 24, 4, 2, 6, 3, "hybrid", "f32"),
    (1024, 8, 2, 4, 4, 2, "mmse", "f16"), (7, 3, 300, 6, 4, 256, "mmse", "f32"),
]


@pytest.mark.parametrize("case", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_gram_form_edges(ocd, case):
    B, U, W, S, Q, K, mode, storage = case
    say("gram case", case)
    wl = synth.make_workload(B, U, W, S, Q, 15.0, seed=[210, B, U, S])
    N0 = float(np.float32(wl["N0"]))
    lam, beta = None, 0.0
    if mode == "hybrid":
        lam = (N0 * np.linspace(0.5, 2.0, K)).astype(np.float32)
        beta = 0.9
    if storage == "f16":
        H, y = to_f16_pairs(wl["H"]), to_f16_pairs(wl["y"])
        Hr, yr = from_f16_pairs(H), from_f16_pairs(y)
    else:
        H, y = wl["H"], wl["y"]
        Hr, yr = H, y
    zo, Lo, _ = oracle_ref(Hr, yr, K, Q, mode, N0, 1.0, lam, float(np.float32(beta)))
    lam_t = None if lam is None else dev(lam)

    def shifted(a):   # the same array one entry past an aligned address
        flat = np.concatenate([a.reshape(-1)[:a[0, 0, 0].size], a.reshape(-1)])
        return dev(flat)[a[0, 0, 0].size:].reshape(a.shape)

    for name, Ht, yt in (("aligned", dev(H), dev(y)), ("shifted", shifted(H), shifted(y))):
        z, L, _ = ocd.detect(Ht, yt, K, Q, mode, N0, 1.0, beta, lam=lam_t, storage=storage)
        torch.cuda.synchronize()
        ez, el = z_rel_err(host(z), zo), llr_rel_err(host(L), Lo)
        say("  %s z err %.3g  llr err %.3g" % (name, ez, el))
        assert ez <= Z_TOL_F32 and el <= LLR_TOL_F32
        z1, _, _ = ocd.detect(Ht, yt, K, Q, mode, N0, 1.0, beta, lam=lam_t, storage=storage,
                              want_llr=False)
        _, L1, _ = ocd.detect(Ht, yt, K, Q, mode, N0, 1.0, beta, lam=lam_t, storage=storage,
                              want_z=False)
        pre = ocd.preprocess(Ht, K, Q, mode, N0, lam=lam_t, storage=storage)
        zp, Lp, _ = ocd.detect(Ht, yt, K, Q, mode, N0, 1.0, beta, lam=lam_t, storage=storage,
                               pre=pre)
        torch.cuda.synchronize()
        assert torch.equal(z1, z) and torch.equal(L1, L)
        assert torch.equal(zp, z) and torch.equal(Lp, L)


def test_one_vector_does_not_touch_another(ocd):
    """NaN in one receive vector stays in that vector; a zero column stays at zero."""
    B, U, W, S, Q, K = 64, 12, 3, 14, 4, 3
    wl = synth.make_workload(B, U, W, S, Q, 15.0, seed=[211, 0])
    N0 = float(np.float32(wl["N0"]))
    H, y = wl["H"].copy(), wl["y"].copy()
    H[1, 5] = 0
    z0, L0, _ = ocd.detect(dev(H), dev(y), K, Q, "mmse", N0)
    y[1, 3, 7] = np.nan
    z, L, _ = ocd.detect(dev(H), dev(y), K, Q, "mmse", N0)
    torch.cuda.synchronize()
    assert np.all(host(z0)[1, :, 5] == 0) and np.all(host(L0)[1, :, 5] == 0)
    keep = np.ones((W, S), bool)
    keep[1, 3] = False
    assert np.array_equal(host(z)[keep], host(z0)[keep])
    assert np.array_equal(host(L)[keep], host(L0)[keep])
    assert np.isnan(host(z)[1, 3]).any()


MANY = [
    # B, U, W, S, Q, K, mode, storage: one wave per subcarrier, around its
    # groups of four subcarriers, the users of a tile (8, 16) and its symbols (4, 8, 16)
    (32, 16, 2049, 3, 4, 3, "box", "f32"), (64, 9, 2051, 5, 4, 3, "mmse", "f16"),
    (17, 8, 2050, 8, 2, 2, "hybrid", "f32"), (40, 3, 1025, 17, 4, 6, "box", "f32"),
    (128, 16, 2048, 4, 4, 2, "hybrid", "f32"),
]


@pytest.mark.parametrize("case", MANY, ids=["-".join(map(str, c)) for c in MANY])
def test_many_subcarriers_equal_few(ocd, case):
    """One wave per subcarrier (many) against four (few): the same bits, forward and
    adjoint, so each subcarrier's results do not depend on how many others there are."""
    B, U, W, S, Q, K, mode, storage = case
    say("many", case)
    wl = synth.make_workload(B, U, W, S, Q, 15.0, seed=[212, B, U, S])
    N0 = float(np.float32(wl["N0"]))
    lam = dev((N0 * np.linspace(0.5, 2.0, K)).astype(np.float32)) if mode == "hybrid" else None
    beta = 0.0 if mode == "mmse" else 0.9
    f16 = storage == "f16"
    H, y = (dev(to_f16_pairs(wl[k]) if f16 else wl[k]) for k in ("H", "y"))
    g = torch.Generator().manual_seed(7)
    dllr = torch.randn(W, S, U, Q, generator=g).cuda()

    def run(a, b):
        kw = dict(lam=lam, storage=storage)
        z, L, zh = ocd.detect(H[a:b], y[a:b], K, Q, mode, N0, 1.0, beta, want_hist=True, **kw)
        _, _, dy = ocd.backward(H[a:b], y[a:b], zh, dllr[a:b].contiguous(), K, Q, mode, N0, 1.0,
                                beta, **kw)
        return z, L, zh, dy

    whole = run(0, W)
    torch.cuda.synchronize()
    for a, b in ((0, 129), (W - 130, W)):
        part = run(a, b)
        torch.cuda.synchronize()
        for name, p, q in zip(("z", "llr", "z_hist", "dy"), part, whole):
            assert torch.equal(p, q[a:b]), name


GRADS = [
    # B, U, W, S, Q, K, mode, storage
    (16, 8, 5, 3, 4, 3, "box", "f32"), (34, 9, 6, 8, 2, 3, "mmse", "f32"),
    (64, 16, 5, 9, 4, 3, "hybrid", "f16"), (35, 17, 3, 16, 4, 7, "hybrid", "f32"),
    (66, 32, 2, 17, 6, 3, "box", "f32"), (63, 5, 1025, 3, 4, 4, "hybrid", "f32"),
    (32, 12, 1027, 4, 4, 2, "box", "f32"), (272, 4, 3, 1, 4, 4, "mmse", "f16"),
    (64, 32, 3, 2, 4, 256, "mmse", "f32"),
]


@pytest.mark.parametrize("case", GRADS, ids=["-".join(map(str, c)) for c in GRADS])
def test_gram_gradients_edges(ocd, case):
    """The training step against the two launches (z, LLRs and dy bit for bit) and dy,
    dlambda and dbeta against the oracle's reverse mode, 1e-3 relative L2 as for the other
    shapes."""
    B, U, W, S, Q, K, mode, storage = case
    say("gram gradients", case)
    wl = synth.make_workload(B, U, W, S, Q, 10.0, seed=[213, B, U, S])
    N0 = float(np.float32(wl["N0"]))
    lam = (N0 * np.linspace(0.8, 1.3, K)).astype(np.float32) if mode == "hybrid" else None
    beta = 0.0 if mode == "mmse" else float(np.float32(0.8))
    if storage == "f16":
        H, y = to_f16_pairs(wl["H"]), to_f16_pairs(wl["y"])
        Hr, yr = from_f16_pairs(H), from_f16_pairs(y)
    else:
        H, y = wl["H"], wl["y"]
        Hr, yr = H, y
    H, y = dev(H), dev(y)
    bits = torch.from_numpy(wl["bits"]).cuda()
    kw = dict(lam=None if lam is None else dev(lam), storage=storage)
    z2, L2, zh = ocd.detect(H, y, K, Q, mode, N0, 1.0, beta, want_hist=True, **kw)
    dlam2, dbeta2, dy2 = ocd.backward(H, y, zh, None, K, Q, mode, N0, 1.0, beta, bits=bits, **kw)
    loss, dlam, dbeta, dy, z, L = ocd.train_step(H, y, bits, K, Q, mode, N0, 1.0, beta,
                                                 want_z=True, want_llr=True, **kw)
    torch.cuda.synchronize()
    assert torch.equal(z, z2) and torch.equal(L, L2) and torch.equal(dy, dy2)
    Lh = host(L).astype(np.float64)
    dllr = (1.0 / (1.0 + np.exp(-Lh)) - wl["bits"]) / Lh.size
    dlam_o, dbeta_o, dy_o = oracle.grad(Hr, yr, dllr, K, Q, mode, N0=N0, lam=lam, beta=beta)
    for name, a, b in (("dlam", dlam, dlam_o), ("dlam2", dlam2, dlam_o), ("dy", dy, dy_o)):
        a, b = host(a).ravel(), np.asarray(b).ravel()
        e = np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)
        say("  %s %.3g" % (name, e))
        assert e <= GRAD_TOL, name
    if mode != "mmse":
        for b in (dbeta, dbeta2):
            assert abs(float(host(b)[0]) - dbeta_o) <= GRAD_TOL * abs(dbeta_o)
    want = np.mean(np.logaddexp(0.0, np.where(wl["bits"] != 0, -Lh, Lh)))
    assert abs(float(host(loss)[0]) - want) <= 1e-5 * want


@pytest.mark.parametrize("B,U,W,S,mode", [(64, 8, 5, 3, "mmse"), (40, 12, 4, 4, "hybrid"),
                                          (64, 16, 3, 9, "mmse"), (64, 20, 3, 4, "hybrid"),
                                          (32, 8, 1026, 3, "hybrid")])
def test_sweep_with_infinite_regulariser(ocd, B, U, W, S, mode):
    """d^-1 = p = 0: an infinite lambda_k sends every z_u to 0 in sweep k and cuts the
    gradient there; a zero column with lambda_k = 0 stays at 0.  Detection and both
    gradients against the oracle."""
    say("infinite lambda", B, U, W, S, mode)
    Q, K = 4, 4
    wl = synth.make_workload(B, U, W, S, Q, 10.0, seed=[214, B, U, S])
    N0 = float(np.float32(wl["N0"]))
    lam = np.array([N0, np.inf, 0.0, N0], np.float32)
    H, beta = wl["H"].copy(), 0.0 if mode == "mmse" else float(np.float32(0.8))
    H[1, U - 1] = 0
    Ht, yt, lt = dev(H), dev(wl["y"]), dev(lam)
    bits = torch.from_numpy(wl["bits"]).cuda()
    z, L, zh = ocd.detect(Ht, yt, K, Q, mode, N0, 1.0, beta, lam=lt, want_hist=True)
    dlam, _, dy = ocd.backward(Ht, yt, zh, None, K, Q, mode, N0, 1.0, beta, bits=bits, lam=lt)
    _, dlam2, _, dy2, z2, L2 = ocd.train_step(Ht, yt, bits, K, Q, mode, N0, 1.0, beta, lam=lt,
                                              want_z=True, want_llr=True)
    torch.cuda.synchronize()
    zo, Lo, zho = oracle_ref(H, wl["y"], K, Q, mode, N0, 1.0, lam, beta, True)
    assert not host(zh)[:, :, 1].any()
    for k in range(K):
        assert z_rel_err(host(zh)[:, :, k], zho[:, :, k]) <= Z_TOL_F32
    assert llr_rel_err(host(L), Lo) <= LLR_TOL_F32
    assert torch.equal(z, z2) and torch.equal(L, L2) and torch.equal(dy, dy2)
    Lh = host(L).astype(np.float64)
    dllr = (1.0 / (1.0 + np.exp(-Lh)) - wl["bits"]) / Lh.size
    dlam_o, _, dy_o = oracle.grad(H, wl["y"], dllr, K, Q, mode, N0=N0, lam=lam, beta=beta)
    for a, b in ((dlam, dlam_o), (dlam2, dlam_o), (dy, dy_o)):
        a, b = host(a).ravel(), np.asarray(b).ravel()
        assert np.linalg.norm(a - b) <= GRAD_TOL * np.linalg.norm(b)


@pytest.mark.parametrize("B,U,W,S,per_sweep,box", [(64, 8, 5, 3, False, False), (40, 12, 4, 4, True, True),
                                                   (64, 20, 3, 4, True, False),
                                                   (32, 16, 2049, 3, False, True)])
def test_given_preprocessing_is_what_the_updates_take(ocd, B, U, W, S, per_sweep, box):
    """Updates take the given d^-1 and p also where they are not those of g and lambda:
    z = proj(d^-1 h^H r + p z) in FP64 with those very values (damped updates of some
    users, one never updated, one held by p = 1)."""
    say("given preprocessing", B, U, W, S, per_sweep, box)
    Q, K = 4, 4
    wl = synth.make_workload(B, U, W, S, Q, 15.0, seed=[215, B, U, S])
    N0, beta = float(np.float32(wl["N0"])), float(np.float32(0.8))
    mode = "hybrid" if box else "mmse"
    lam = dev((N0 * np.linspace(0.5, 2.0, K)).astype(np.float32)) if per_sweep else None
    H, y = dev(wl["H"]), dev(wl["y"])
    g, dinv, p = ocd.preprocess(H, K, Q, mode, N0, lam=lam)
    dinv[..., ::3] *= 0.75
    p[..., ::3] = 1.0 - 0.75 * (1.0 - p[..., ::3])
    dinv[..., 1] = 0.0
    p[..., 1] = 0.0
    p[..., U - 1] = 1.0
    z, _, _ = ocd.detect(H, y, K, Q, mode, N0, 1.0, beta, lam=lam, pre=(g, dinv, p))
    torch.cuda.synchronize()
    Hd, r = wl["H"].astype(np.complex128), wl["y"].astype(np.complex128)
    d64 = np.broadcast_to(host(dinv).astype(np.float64).reshape(W, -1, U), (W, K, U))
    p64 = np.broadcast_to(host(p).astype(np.float64).reshape(W, -1, U), (W, K, U))
    zr = np.zeros((W, S, U), np.complex128)
    for k in range(K):
        for u in range(U):
            h = Hd[:, None, u]
            c = (d64[:, k, u, None] * np.sum(h.conj() * r, -1) + p64[:, k, u, None] * zr[..., u])
            if box:
                c = np.clip(c.real, -beta, beta) + 1j * np.clip(c.imag, -beta, beta)
            r = r - h * (c - zr[..., u])[..., None]
            zr[..., u] = c
    assert z_rel_err(host(z), zr) <= Z_TOL_F32


def _correlated(kind, W, U, B, rng):
    """Channels that are not i.i.d.: users or antennas correlated, or unequal powers."""
    H = (rng.standard_normal((W, U, B)) + 1j * rng.standard_normal((W, U, B))) / np.sqrt(2 * B)
    what, x = kind
    if what == "users":
        return np.linalg.cholesky((1 - x) * np.eye(U) + x) @ H
    if what == "antennas":
        return H @ np.linalg.cholesky(x ** np.abs(np.subtract.outer(np.arange(B), np.arange(B)))).T
    return H * 10 ** (-x / 20 * rng.random((W, U, 1)))   # powers spread over x dB


@pytest.mark.parametrize("kind", [("users", 0.9), ("users", 0.99), ("antennas", 0.99), ("powers", 30.0)])
@pytest.mark.parametrize("B,U,K,storage", [(128, 8, 3, "f32"), (128, 8, 3, "f16"), (64, 8, 4, "f32"),
                                           (32, 8, 4, "f32"), (40, 7, 4, "f16"), (32, 16, 4, "f32"),
                                           (64, 32, 4, "f32"), (48, 24, 4, "f16"), (256, 32, 5, "f32"),
                                           (51, 12, 4, "f32")])
def test_error_on_ill_conditioned_channels(ocd, B, U, K, storage, kind):
    """The error of z where users or antennas are correlated or powers unequal: the inner
    products are FP64, so what is left are the roundings of g, den, d^-1 and z, 2^-24 each
    (root mean square over the vectors at most 4 x 2^-24), and no more than the residual
    form's, which up to 8 users a plan with the channel in registers runs."""
    say("ill-conditioned", B, U, K, storage, kind)
    W, S, Q = 32, 7, 4
    rng = np.random.default_rng([216, B, U, int(100 * kind[1])])
    H = _correlated(kind, W, U, B, rng)
    x = (rng.choice([-3, -1, 1, 3], (W, S, U)) + 1j * rng.choice([-3, -1, 1, 3], (W, S, U))) / np.sqrt(10)
    N0 = float(np.float32(0.01))
    y = x @ H + np.sqrt(N0 / 2) * (rng.standard_normal((W, S, B)) + 1j * rng.standard_normal((W, S, B)))
    if storage == "f16":
        Hx, yx = to_f16_pairs(H), to_f16_pairs(y)
        Hr, yr = from_f16_pairs(Hx), from_f16_pairs(yx)
    else:
        Hx, yx = Hr, yr = H.astype(np.complex64), y.astype(np.complex64)
    zo, _, _ = oracle_ref(Hr, yr, K, Q, "mmse", N0)
    Ht, yt = dev(Hx), dev(yx)

    def rms():
        z, _, _ = ocd.detect(Ht, yt, K, Q, "mmse", N0, storage=storage)
        torch.cuda.synchronize()
        e = np.linalg.norm(host(z) - zo, axis=-1) / np.linalg.norm(zo, axis=-1)
        return float(np.sqrt(np.mean(e ** 2)))

    e = rms()
    say("  rms error %.3g" % e)
    assert e <= 4 * 2.0 ** -24
    if U <= 8:
        pb = ocd.problem(B, U, W, S, Q, K, "mmse", storage, N0)
        plan = ocd.ocd_get_plan(pb)
        ocd.ocd_set_plan(pb, ocd.Plan(16, 8, 0, 1, 0))
        r = rms()
        ocd.ocd_set_plan(pb, plan)
        say("  residual form %.3g" % r)
        assert e <= r


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("B,U,W,S,K", [(228, 12, 601, 14, 3), (230, 12, 514, 9, 3)])
def test_one_wave_training_step_of_more_than_8_symbols(ocd, B, U, W, S, K, storage):
    """9 to 16 users, more than 8 symbols and more than 512 subcarriers: the training step on
    one wave a subcarrier, 16 symbols of z history for each of four, against the oracle."""
    test_gram_gradients_edges(ocd, (B, U, W, S, 4, K, "hybrid", storage))


LOOPS = [
    # B, U, W, S, K, subcarriers of a part: more tiles than workgroups (the partial sums of
    # 1 MiB), whose kernels take several tiles each
    (64, 8, 4100, 3, 256, 1000),     # adjoint one wave a subcarrier, training step four
    (64, 16, 4100, 1, 256, 1000),
    (34, 17, 1100, 1, 256, 500),
    (64, 8, 106000, 3, 9, 30000),    # training step on one wave a subcarrier
]


@pytest.mark.parametrize("case", LOOPS, ids=["-".join(map(str, c)) for c in LOOPS])
def test_gradients_of_more_tiles_than_workgroups(ocd, case):
    """The looping gradient kernels against parts of the subcarriers with a workgroup per
    tile: z, LLRs and the adjoint's dy bit for bit, the training step's dy (whose mean has
    another 1 / n) to 1e-6, dlambda, dbeta and the loss against the parts' sums (1e-4: FP32
    partial sums in another order); and one part against the oracle."""
    B, U, W, S, K, part = case
    Q, mode, beta = 4, "hybrid", float(np.float32(0.8))
    say("looping gradients", case)
    wl = synth.make_workload_device(B, U, W, S, Q, 10.0, seed=2160 + U, device="cuda")
    N0 = float(np.float32(wl["N0"]))
    lam = (N0 * np.linspace(0.8, 1.3, K)).astype(np.float32)
    H, y, bits, kw = wl["H"], wl["y"], wl["bits"], dict(lam=dev(lam))

    def train(a, b):
        loss, dlam, dbeta, dy, z, L = ocd.train_step(H[a:b], y[a:b], bits[a:b], K, Q, mode, N0, 1.0,
                                                     beta, want_z=True, want_llr=True, **kw)
        return z, L, dy, [t.double() for t in (loss, dlam, dbeta)]

    def adjoint(a, b, dllr):
        _, _, zh = ocd.detect(H[a:b], y[a:b], K, Q, mode, N0, 1.0, beta, want_hist=True, **kw)
        dlam, dbeta, dy = ocd.backward(H[a:b], y[a:b], zh, dllr, K, Q, mode, N0, 1.0, beta, **kw)
        return dy, [t.double() for t in (dlam, dbeta)]

    z, L, dy, means = train(0, W)
    dllr = torch.randn(W, S, U, Q, generator=torch.Generator(device="cuda").manual_seed(8), device="cuda")
    loops = K > 100   # the adjoint's workgroups loop at this K only
    dya, sums = adjoint(0, W, dllr) if loops else (None, [])
    want = [torch.zeros_like(t) for t in means + sums]
    for a in range(0, W, part):
        b = min(a + part, W)
        z1, L1, dy1, m = train(a, b)
        assert torch.equal(z1, z[a:b]) and torch.equal(L1, L[a:b]), a
        assert float((dy1 * ((b - a) / W) - dy[a:b]).norm()) <= 1e-6 * float(dy[a:b].norm()), a
        m = [t * ((b - a) / W) for t in m]
        if loops:
            dy1, s = adjoint(a, b, dllr[a:b])
            assert torch.equal(dy1, dya[a:b]), a
            m += s
        for t, x in zip(want, m):
            t += x
    for x, t in zip(means + sums, want):
        assert float((x - t).norm()) <= 1e-4 * float(t.norm())
    n = 40
    Hh, yh, bh = host(H[:n]), host(y[:n]), host(bits[:n])
    _, Lp, dyp, (loss, dlam, dbeta) = train(0, n)
    Lh = host(Lp).astype(np.float64)
    g = (1.0 / (1.0 + np.exp(-Lh)) - bh) / Lh.size
    dlam_o, dbeta_o, dy_o = oracle.grad(Hh, yh, g, K, Q, mode, N0=N0, lam=lam, beta=beta)
    for x, t in ((dlam, dlam_o), (dyp, dy_o), (dbeta, dbeta_o)):
        x, t = host(x).ravel(), np.asarray(t).ravel()
        assert np.linalg.norm(x - t) <= GRAD_TOL * np.linalg.norm(t)
    mean = np.mean(np.logaddexp(0.0, np.where(bh != 0, -Lh, Lh)))
    assert abs(float(loss) - mean) <= 1e-5 * mean


def test_gradients_whose_residual_plan_ends_at_the_lds_limit(ocd):
    """1024 x 19, K = 46: the residual form's smallest plan takes all but 104 bytes of the LDS
    of a workgroup, less than its kernels' own; the Gram form, which runs here, does not
    use it, so the call is accepted."""
    B, U, W, S, Q, K = 1024, 19, 2, 2, 4, 46
    say("residual plan at the limit")
    wl = synth.make_workload(B, U, W, S, Q, 10.0, seed=[223, 0])
    N0, beta = float(np.float32(wl["N0"])), float(np.float32(0.8))
    lam = (N0 * np.linspace(0.8, 1.3, K)).astype(np.float32)
    H, y, lt = dev(wl["H"]), dev(wl["y"]), dev(lam)
    _, L, zh = ocd.detect(H, y, K, Q, "hybrid", N0, 1.0, beta, lam=lt, want_hist=True)
    dllr = torch.randn(W, S, U, Q, generator=torch.Generator().manual_seed(4)).cuda()
    dlam, _, dy = ocd.backward(H, y, zh, dllr, K, Q, "hybrid", N0, 1.0, beta, lam=lt)
    torch.cuda.synchronize()
    dlam_o, _, dy_o = oracle.grad(wl["H"], wl["y"], host(dllr), K, Q, "hybrid", N0=N0, lam=lam, beta=beta)
    for a, b in ((dlam, dlam_o), (dy, dy_o)):
        a, b = host(a).ravel(), np.asarray(b).ravel()
        assert np.linalg.norm(a - b) <= GRAD_TOL * np.linalg.norm(b)
