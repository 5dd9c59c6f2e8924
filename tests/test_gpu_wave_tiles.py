"""Products on wave tiles (csrc/direct.hip) and on unaligned workgroup tiles,
against the dense FP64 oracle, at the sizes where their tiles and K steps end:
bonds one below, at and one above a K step (16 doubles, 32 floats) and a tile,
one K step or less, MPO bonds that do and do not divide a tile's rows, physical
dimensions with and without the fused W-map.

Tolerances: FP64 1e-12 and FP32 3e-5 of the largest entry, as in
test_gpu_parity (about sqrt(K) u for the longest sums here, K <= 8192)."""
import numpy as np
import pytest
import torch

from oracle import contract as C
from paper_1501_05504_amd import synth

pytestmark = pytest.mark.gpu

abi = pytest.importorskip("paper_1501_05504_amd.abi")

DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def ctx():
    c = abi.Context(0)
    yield c
    c.close()


def rel(got, ref):
    return float(np.abs(got - ref).max() / np.abs(ref).max())


def inputs(ml, d, mr, wl, wr, dt):
    g = [synth.gaussian(s, 900 + i) for i, s in enumerate([(ml, wl, ml), (wl, wr, d, d), (mr, wr, mr), (ml, d, mr)])]
    if dt == torch.float32:
        g = [x.astype(np.float32).astype(np.float64) for x in g]
    return g, [torch.tensor(x, dtype=dt, device=DEV) for x in g]


SHAPES = [(1, 2, 1, 1, 1), (15, 4, 16, 6, 6), (16, 4, 17, 6, 6), (17, 2, 15, 5, 5), (31, 4, 33, 6, 6),
          (33, 2, 31, 8, 8), (32, 4, 32, 1, 6), (40, 4, 64, 6, 1), (65, 2, 63, 40, 7), (9, 4, 70, 18, 18),
          (34, 3, 21, 5, 5), (50, 2, 47, 17, 3), (129, 4, 127, 6, 6), (257, 4, 255, 6, 6), (513, 2, 700, 5, 5)]


@pytest.mark.parametrize("dt", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("shape", SHAPES, ids=["-".join(map(str, s)) for s in SHAPES])
def test_heff_at_tile_edges(ctx, shape, dt):
    ml, d, mr, wl, wr = shape
    (L, W, R, psi), t = inputs(ml, d, mr, wl, wr, dt)
    out = torch.full((ml, d, mr), float("nan"), dtype=dt, device=DEV)
    ctx.apply_heff(*t, out)
    torch.cuda.synchronize()
    assert rel(out.cpu().double().numpy(), C.apply_heff(L, W, R, psi)) < (1e-12 if dt == torch.float64 else 3e-5)


@pytest.mark.parametrize("direction", ["l2r", "r2l"])
@pytest.mark.parametrize("shape", SHAPES[:13], ids=["-".join(map(str, s)) for s in SHAPES[:13]])
def test_expansion_and_environment_at_tile_edges(ctx, shape, direction):
    ml, d, mr, wl, wr = shape
    (L, W, R, psi), (tL, tW, tR, tpsi) = inputs(ml, d, mr, wl, wr, torch.float64)
    if direction == "l2r":
        T = np.einsum("awx,xty->awty", L, psi)
        T2 = np.einsum("wvst,awty->asvy", W, T)
        mt = np.concatenate([psi.reshape(ml * d, mr), 0.5 * T2.reshape(ml * d, wr * mr)], 1)
        env = np.einsum("asb,asvy->bvy", psi, T2)
        args = (abi.L2R, tL)
    else:
        Y = np.einsum("xty,bvy->xtbv", psi, R)
        Z = np.einsum("wvst,xtbv->wxsb", W, Y)
        mt = np.concatenate([psi.reshape(ml, d * mr), 0.5 * Z.reshape(wl * ml, d * mr)], 0)
        env = np.einsum("asb,wxsb->awx", psi, Z)
        args = (abi.R2L, tR)
    Mt = torch.full(mt.shape, float("nan"), dtype=torch.float64, device=DEV)
    ctx.expand_subspace(args[0], args[1], tW, tpsi, 0.5, Mt)
    out = torch.full(env.shape, float("nan"), dtype=torch.float64, device=DEV)
    ctx.update_env(args[0], args[1], tW, tpsi, out)
    torch.cuda.synchronize()
    assert rel(Mt.cpu().numpy(), mt) < 1e-12
    assert rel(out.cpu().numpy(), env) < 1e-12


@pytest.mark.parametrize("dt", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("mlp,mr,wr", [(33, 1, 6), (70, 1030, 8), (520, 65, 2), (1030, 1028, 2)])
def test_long_and_large_products(ctx, mlp, mr, wr, dt):
    """Two plain GEMMs (the centre-matrix application): sums long enough to be
    split over the grid, and sizes on both sides of the wave-tile rule."""
    g = [synth.gaussian(s, 950 + i) for i, s in enumerate([(mlp, wr, mlp), (mr, wr, mr), (mlp, mr)])]
    if dt == torch.float32:
        g = [x.astype(np.float32).astype(np.float64) for x in g]
    Lt, R, Cm = [torch.tensor(x, dtype=dt, device=DEV) for x in g]
    out = torch.full((mlp, mr), float("nan"), dtype=dt, device=DEV)
    ctx.apply_cwf(Lt, R, Cm, out)
    torch.cuda.synchronize()
    T = np.tensordot(g[0], g[2], axes=([2], [0]))
    ref = np.tensordot(T, g[1], axes=([1, 2], [1, 2]))
    assert rel(out.cpu().double().numpy(), ref) < (1e-12 if dt == torch.float64 else 3e-5)


def test_infinite_entry_stays_in_its_rows(ctx):
    """An Inf in one row of L reaches only that row's outputs, also where the
    last K step is not whole and tiles are padded."""
    ml, d, mr, w = 37, 4, 29, 6
    (L, W, R, psi), (tL, tW, tR, tpsi) = inputs(ml, d, mr, w, w, torch.float64)
    tL[5, 2, 36] = float("inf")
    out = torch.empty((ml, d, mr), dtype=torch.float64, device=DEV)
    ctx.apply_heff(tL, tW, tR, tpsi, out)
    torch.cuda.synchronize()
    o = out.cpu().numpy()
    ref = C.apply_heff(L, W, R, psi)
    keep = np.arange(ml) != 5
    assert not np.isfinite(o[5]).any()
    assert rel(o[keep], ref[keep]) < 1e-12


@pytest.mark.parametrize("ml, d, mr, wl, wr", [(1, 2, 3, 2, 3), (31, 2, 17, 3, 5), (32, 3, 20, 1, 1), (33, 4, 24, 6, 6),
                                               (64, 1, 16, 4, 4), (97, 2, 9, 5, 3)])
def test_mpo_adjoint(ctx, ml, d, mr, wl, wr):
    """Wbar summed over the left bond, at bonds and entry counts that do and do
    not divide its split."""
    from oracle.adjoint import heff_grad_W
    (L, W, R, psi), (Ld, Wd, Rd, pd) = inputs(ml, d, mr, wl, wr, torch.float64)
    ybar = synth.gaussian((ml, d, mr), 77)
    out = torch.empty(wl, wr, d, d, dtype=torch.float64, device=DEV)
    ctx.heff_grad_W(Ld, Rd, pd, torch.tensor(ybar, device=DEV), out)
    assert rel(out.cpu().numpy(), heff_grad_W(L, R, psi, ybar)) < 1e-12


@pytest.mark.parametrize("ml, d, mr", [(1, 2, 1), (3, 1, 1), (5, 2, 3), (31, 2, 16), (341, 1, 3), (32, 4, 8), (41, 5, 5), (63, 1, 65),
                                       (32, 2, 32), (683, 1, 3), (64, 1, 64), (17, 1, 241)])
@pytest.mark.parametrize("kmax", [8, 17, 60])
def test_lanczos_short_vectors(ctx, ml, d, mr, kmax):
    """Vectors from 2 to 4097 elements and 8 to 60 Krylov vectors, across the
    sizes at which the one-workgroup Gram-Schmidt changes its registers or ends:
    the Ritz pair satisfies the eigenvalue equation to the requested 1e-11 of
    the norm, ten times that for the restarts' accumulated rounding."""
    rng = np.random.default_rng(ml * mr)
    w = 3
    sym = lambda x: (x + x.transpose(2, 1, 0)) / 2
    L, R = sym(rng.standard_normal((ml, w, ml))), sym(rng.standard_normal((mr, w, mr)))
    W = rng.standard_normal((w, w, d, d))
    W = (W + W.transpose(0, 1, 3, 2)) / 2
    x = torch.tensor(rng.standard_normal((ml, d, mr)), device=DEV)
    th, nmv, ok = ctx.lanczos(*(torch.tensor(a, device=DEV) for a in (L, W, R)), x, tol=1e-11, kmax=kmax,
                              max_matvecs=4000)
    v = x.cpu().numpy()
    hv = C.apply_heff(L, W, R, v)
    norm = np.abs(th)
    assert ok and abs(np.linalg.norm(v) - 1) < 1e-12
    assert np.linalg.norm(hv - th * v) <= 1e-10 * max(1.0, norm)
    if v.size <= 512:
        H = C.heff_matrix(L, W, R)
        ref = np.linalg.eigvalsh((H + H.T) / 2)[0]
        assert abs(th - ref) <= 1e-10 * max(1.0, norm)


@pytest.mark.parametrize("ml, d, mr, wl, wr", [(7, 4, 9, 16, 4), (9, 2, 33, 17, 3), (11, 2, 17, 32, 2), (6, 2, 40, 33, 2),
                                               (96, 4, 96, 6, 6), (130, 2, 128, 8, 8), (129, 4, 121, 6, 5), (193, 4, 192, 6, 6)])
@pytest.mark.parametrize("dt, tol", [(torch.float64, 1e-12), (torch.float32, 3e-5)])
def test_fused_front_tile_heights(ctx, ml, d, mr, wl, wr, dt, tol):
    """MPO bonds that only some of the fused kernel's tile heights (16, 32, 48
    rows) can hold, and sizes on both sides of the rule that picks among them;
    both directions through the environment updates."""
    (L, W, R, psi), (Ld, Wd, Rd, pd) = inputs(ml, d, mr, wl, wr, dt)
    out = torch.empty(ml, d, mr, dtype=dt, device=DEV)
    ctx.apply_heff(Ld, Wd, Rd, pd, out)
    assert rel(out.cpu().numpy(), C.apply_heff(L, W, R, psi)) < tol
    if dt == torch.float64:
        env = torch.empty(ml, wl, ml, dtype=dt, device=DEV)
        ctx.update_env(abi.R2L, Rd, Wd, pd, env)
        assert rel(env.cpu().numpy(), C.update_right(R, W, psi)) < tol


@pytest.mark.parametrize("ml, d, mr, wl, wr", [(1, 2, 4, 3, 2), (2, 2, 2, 2, 2), (3, 2, 8, 4, 4), (33, 4, 64, 2, 3), (64, 3, 66, 5, 4),
                                               (65, 4, 68, 6, 6), (66, 4, 1028, 8, 3), (130, 1, 63, 3, 3), (31, 4, 124, 9, 2)])
def test_low_precision_vector_paths(ctx, ml, d, mr, wl, wr):
    """FP32 and BF16 products whose rows do and do not consist of whole vectors of
    four (the W-map) or pairs (the transposition of psi).  BF16: T1 is exact
    to FP32 rounding and T2 is rounded to eight bits, so the error is within
    2^-9 of the product of absolute values, doubled for the FP32 sums."""
    (L, W, R, psi), _ = inputs(ml, d, mr, wl, wr, torch.float32)
    for dt in (torch.float32, torch.bfloat16):
        Ld, Rd, pd = (torch.tensor(x, device=DEV).to(dt) for x in (L, R, psi))
        Wd = torch.tensor(W, dtype=torch.float32, device=DEV)
        out = torch.full((ml, d, mr), float("nan"), dtype=torch.float32, device=DEV)
        ctx.apply_heff(Ld, Wd, Rd, pd, out)
        Lh, Rh, ph = (x.double().cpu().numpy() for x in (Ld, Rd, pd))
        ref, got = C.apply_heff(Lh, W, Rh, ph), out.double().cpu().numpy()
        if dt == torch.float32:
            assert rel(got, ref) < 3e-5
        else:
            bound = 2.0 ** -8 * C.apply_heff(np.abs(Lh), np.abs(W), np.abs(Rh), np.abs(ph))
            assert np.all(np.abs(got - ref) <= bound)


@pytest.mark.parametrize("ml, d, mr, w", [(1, 1, 1, 1), (15, 1, 17, 2), (16, 1, 16, 3), (17, 3, 15, 2), (33, 3, 16, 5), (31, 1, 47, 7),
                                          (48, 3, 49, 5), (64, 3, 120, 9), (129, 3, 96, 6), (150, 3, 160, 6)])
@pytest.mark.parametrize("dt, tol", [(torch.float64, 1e-12), (torch.float32, 3e-5)])
def test_small_wave_tiles(ctx, ml, d, mr, w, dt, tol):
    """Products of few tiles, on both sides of a 16-row tile, of the wave count's
    rule (40 K steps) and of the tile count at which larger tiles take over; a
    physical dimension that the fused kernel does not take."""
    (L, W, R, psi), (Ld, Wd, Rd, pd) = inputs(ml, d, mr, w, w, dt)
    out = torch.empty(ml, d, mr, dtype=dt, device=DEV)
    ctx.apply_heff(Ld, Wd, Rd, pd, out)
    assert rel(out.cpu().numpy(), C.apply_heff(L, W, R, psi)) < tol


@pytest.mark.parametrize("d, w", [(2, 1), (2, 3), (2, 5), (2, 7), (2, 13), (4, 1), (4, 2), (4, 4), (4, 5), (4, 6), (4, 9)])
@pytest.mark.parametrize("dt", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_infinite_entry_gives_infinite_outputs(ctx, d, w, dt):
    """With positive operands an Inf in one row of L makes every output of that
    row +Inf, not NaN, whatever the sum over the MPO bond is padded to (both
    counts of its steps that stay in registers, and more); the other rows agree
    with the oracle.  FP64: the expansion term in both directions as well."""
    ml, mr, a = 21, 18, 5
    g = [np.abs(x) for x in inputs(ml, d, mr, w, w, dt)[0]]
    ref = C.apply_heff(*g)
    t = [torch.tensor(x, dtype=dt, device=DEV) for x in g]
    t[0][a, w - 1, 7] = float("inf")
    out = torch.empty((ml, d, mr), dtype=dt, device=DEV)
    ctx.apply_heff(*t, out)
    o = out.cpu().double().numpy()
    keep = np.arange(ml) != a
    assert np.all(o[a] == np.inf)
    assert rel(o[keep], ref[keep]) < (1e-12 if dt == torch.float64 else 3e-5)
    if dt == torch.float64:
        M = torch.empty((ml * d, (1 + w) * mr), dtype=dt, device=DEV)
        ctx.expand_subspace(abi.L2R, t[0], t[1], t[3], 0.5, M)
        o = M.cpu().numpy()[:, mr:].reshape(ml, d, w, mr)
        assert np.all(o[a] == np.inf) and np.isfinite(o[keep]).all()
        t[2][3, w - 1, 7] = float("inf")
        M = torch.empty(((1 + w) * ml, d * mr), dtype=dt, device=DEV)
        ctx.expand_subspace(abi.R2L, t[2], t[1], t[3], 0.5, M)
        o = M.cpu().numpy()[ml:].reshape(w, ml, d, mr)
        keep = np.arange(mr) != 3
        assert np.all(o[..., 3] == np.inf) and np.isfinite(o[..., keep]).all()


def step_times(ctx, shape, dt, calls=4):
    """Summed milliseconds of GEMM-1, W-map and GEMM-2 over `calls` products."""
    ml, d, mr, wl, wr = shape
    wide = torch.float32 if dt == torch.bfloat16 else dt
    t = [torch.randn(s, device=DEV).to(e) for s, e in [((ml, wl, ml), dt), ((wl, wr, d, d), wide), ((mr, wr, mr), dt), ((ml, d, mr), dt)]]
    out = torch.empty((ml, d, mr), dtype=wide, device=DEV)
    ctx.apply_heff(*t, out)
    ctx.profile_begin(calls)
    for _ in range(calls):
        ctx.apply_heff(*t, out)
    ms, n = ctx.profile_end()
    assert n == calls
    return ms


@pytest.mark.parametrize("dt", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_profile_of_fused_steps(ctx, dt):
    """The profile has no time at all for a W-map that was part of GEMM-1's
    launch, and a time for one that ran by itself."""
    small = (37, 4, 29, 6, 6)
    ms = step_times(ctx, small, dt)
    assert ms[0] > 0 and ms[1] == 0 and ms[2] > 0
    ctx.set_tile_config(1)
    try:
        ms = step_times(ctx, small, dt)
    finally:
        ctx.set_tile_config(-1)
    assert min(ms) > 0
    assert step_times(ctx, small, dt)[1] == 0


@pytest.mark.parametrize("dt", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("shape, fused", [((37, 4, 29, 6, 6), True), ((256, 4, 250, 6, 6), True), ((500, 2, 500, 8, 8), True),
                                          ((1024, 4, 1024, 6, 6), False), ((1400, 4, 1400, 6, 6), False),
                                          ((2000, 2, 2000, 8, 8), False)], ids=lambda x: str(x).replace(" ", ""))
def test_fused_steps_where_they_are_faster(ctx, shape, fused, dt):
    """GEMM-1 and the W-map are one launch at the sizes where that is measured
    to be 13 to 50 % faster, and two where it is 5 to 17 % slower."""
    assert (step_times(ctx, shape, dt)[1] == 0) == fused


@pytest.mark.parametrize("dt", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("ml, mr", [(250, 1939), (500, 1939)])
def test_long_sums_of_many_tiles(ctx, ml, mr, dt):
    """The last GEMM of H_eff at 1952 and 3843 tiles of 32x32 with a sum over
    11634 elements takes no longer by the rule than on 256x128 workgroup tiles
    (FP64: it was 3 and 31 % more), ten per cent allowed for two timings; split
    sums agree with the oracle."""
    shape = (ml, 4, mr, 6, 6)
    best = lambda: min(step_times(ctx, shape, dt)[2] for _ in range(4))
    ctx.set_tile_config(2)
    try:
        fixed = best()
    finally:
        ctx.set_tile_config(-1)
    assert best() <= 1.1 * fixed
    g = [synth.gaussian(s, 970 + i) for i, s in enumerate([(ml, 6, ml), (6, 6, 4, 4), (mr, 6, mr), (ml, 4, mr)])]
    t = [torch.tensor(x, dtype=dt, device=DEV) for x in g]
    out = torch.full((ml, 4, mr), float("nan"), dtype=dt, device=DEV)
    ctx.apply_heff(*t, out)
    L, W, R, psi = [x.double().cpu().numpy() for x in t]
    ref = C.apply_heff(L, W, R, psi)
    assert rel(out.cpu().double().numpy(), ref) < (1e-12 if dt == torch.float64 else 3e-5)


@pytest.mark.parametrize("m, w", [(32, 8), (64, 8), (128, 8), (128, 6)])
def test_small_map_of_whole_vectors(ctx, m, w):
    """BF16: at small bonds the W-map takes no longer for rows of whole vectors
    than for the next shorter, ragged ones (it was 1.6 to 1.8 times as long);
    a quarter more allowed for two timings."""
    best = lambda mr: min(step_times(ctx, (m, 4, mr, w, w), torch.bfloat16, 20)[1] for _ in range(5))
    ragged = best(m - 1)
    assert best(m) <= 1.25 * ragged


@pytest.mark.parametrize("ml, mr", [(1876, 192), (1876, 188), (580, 600), (510, 600), (280, 1248), (280, 1252), (240, 1548),
                                    (240, 1552), (340, 1496), (401, 1500), (200, 1696), (200, 1700), (180, 1996), (180, 2000)])
@pytest.mark.parametrize("w", [6, 8])
def test_map_rule_edges(ctx, ml, mr, w):
    """FP32 and BF16 products on both sides of the sizes at which the W-map
    changes between one and four columns a thread; bounds as in
    test_low_precision_vector_paths."""
    d, rng = 4, np.random.default_rng(ml + mr)
    L, W, R, psi = [torch.tensor(rng.standard_normal(s), device=DEV) for s in [(ml, w, ml), (w, w, d, d), (mr, w, mr), (ml, d, mr)]]
    for dt in (torch.float32, torch.bfloat16):
        a = [L.to(dt), W.float(), R.to(dt), psi.to(dt)]
        out = torch.full((ml, d, mr), float("nan"), dtype=torch.float32, device=DEV)
        ctx.set_tile_config(1)             # the W-map by itself in FP32 too
        try:
            ctx.apply_heff(*a, out)
        finally:
            ctx.set_tile_config(-1)

        def ref(f):                        # the oracle's contraction order, on the device
            l, x, r, p = (f(v.double()) for v in a)
            T = torch.matmul(l.reshape(ml * w, ml), p.reshape(ml, d * mr)).reshape(ml, w, d, mr)
            T = torch.tensordot(T, x, dims=([1, 2], [0, 3])).permute(0, 3, 2, 1).reshape(ml * d, w * mr).contiguous()
            return torch.matmul(T, r.reshape(mr, w * mr).t().contiguous()).reshape(ml, d, mr)
        err = (out.double() - ref(lambda v: v)).abs()
        if dt == torch.float32:
            assert float(err.max() / ref(lambda v: v).abs().max()) < 3e-5
        else:
            assert bool((err <= 2.0 ** -8 * ref(torch.abs)).all())


@pytest.mark.parametrize("dt, mlp, mr, wr", [(torch.float64, 33, 1040, 8), (torch.float64, 70, 1030, 8), (torch.float32, 30, 2060, 8),
                                             (torch.float64, 1000, 1939, 6), (torch.float64, 2960, 1480, 5),
                                             (torch.float32, 2960, 1480, 5)])
def test_split_sums_equal_unsplit(ctx, dt, mlp, mr, wr):
    """Sums that the rules split over the grid (few wave tiles of a very long sum;
    workgroup tiles of a large product) against the same product unsplit: that
    the split ran shows in the rounding, its result agrees with the unsplit one
    and with the contraction in FP64, and a second run is bitwise the same."""
    gen = torch.Generator(device=DEV).manual_seed(mlp)
    Lt, R, Cm = [torch.randn(s, generator=gen, device=DEV, dtype=dt) for s in [(mlp, wr, mlp), (mr, wr, mr), (mlp, mr)]]
    outs = []
    try:
        for on in (True, False, True):
            ctx.set_splitk(on)
            out = torch.full((mlp, mr), float("nan"), dtype=dt, device=DEV)
            ctx.apply_cwf(Lt, R, Cm, out)
            outs.append(out)
    finally:
        ctx.set_splitk(True)
    T = torch.matmul(Lt.double().reshape(mlp * wr, mlp), Cm.double()).reshape(mlp, wr * mr)
    ref = torch.matmul(T, R.double().reshape(mr, wr * mr).t().contiguous())
    scale = float(ref.abs().max())
    tol = 1e-12 if dt == torch.float64 else 3e-5
    assert all(float((o.double() - ref).abs().max()) < tol * scale for o in outs)
    assert torch.equal(outs[0], outs[2]) and not torch.equal(outs[0], outs[1])
