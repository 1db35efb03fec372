"""GPU parity of the dense (matrix-core) SB path and of its reduced-precision
forms against the CPU oracle, through the C ABI."""
import ctypes as C

import numpy as np
import pytest

import oracle
import workloads as wl
from gpu_helpers import rel_inf_error, unpack_spins

pytestmark = pytest.mark.gpu

# the two dense tile kernels: 64 x 128 register tiles, and 128 x 128 tiles staged through LDS
DENSE_PATHS = ["dense", "dense_staged"]


@pytest.fixture(scope="module")
def q():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_26477_amd as q
    return q


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _small_int_instance(n, m, seed, lim=15, kind="complete"):
    """Weights in [-lim, lim] * 2^16: exactly representable in bf16 and e4m3 after
    the per-objective power-of-two scaling, so every MFMA product is exact."""
    base = wl.random_instance(n, m, kind, seed=seed)
    rng = np.random.default_rng(seed)
    w = rng.integers(-lim, lim + 1, size=base.weights.shape).astype(np.int64) << 16
    return wl.Instance(n, m, base.edge_u, base.edge_v, w.astype(np.int32))


def _field(q, prob, prec, phi):
    import torch
    count = phi.shape[0]
    b = C.c_size_t()
    L = q._lib
    L.qaia_dense_field_workspace_bytes.argtypes = [C.c_void_p, C.c_int32, C.c_int64, C.POINTER(C.c_size_t)]
    L.qaia_dense_field.argtypes = [C.c_void_p, C.c_int32, C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p,
                                   C.c_size_t, C.c_void_p]
    q._check(L.qaia_dense_field_workspace_bytes(prob.handle, prec, count, C.byref(b)))
    ws = torch.empty(b.value, dtype=torch.uint8, device="cuda")
    ph = _dev(phi.astype(np.float32))
    out = torch.empty((count, prob.m, prob.n), dtype=torch.float32, device="cuda")
    q._check(L.qaia_dense_field(prob.handle, prec, C.c_void_p(ph.data_ptr()), count,
                                C.c_void_p(out.data_ptr()), C.c_void_p(ws.data_ptr()), b.value,
                                C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


# ---------------------------------------------------------------- trajectories

@pytest.mark.parametrize("path", DENSE_PATHS)
def test_dense_fp32_trace_parity_bsb(q, path):
    inst = wl.random_instance(12, 3, "deg3", seed=41, num_edges=16)
    c = wl.dirichlet_weights(6, 3, 42)
    prob = q.problem_from_instance(inst)
    s = q.make_schedule("bsb", steps=1000, dt=0.5, seed=43, path=path)
    _, _, _, tr = q.qaia_sample_trace(prob, _dev(c), 8, s, 100)
    _, ref = oracle.sb_sample(inst, c, 8, 1000, "bsb", dt=0.5, seed=43, trace_steps=100)
    err = rel_inf_error(tr.cpu().numpy(), ref)
    print(f"dense fp32 bsb: max rel err {err.max():.3e}")
    assert err.max() <= 1e-5


@pytest.mark.parametrize("path", DENSE_PATHS)
def test_dense_fp32_trace_parity_complete_graph(q, path):
    """A complete 70-node graph (two 64-spin tiles, ragged; one ragged 128-spin tile) for 100 steps."""
    inst = wl.random_instance(70, 2, "complete", seed=44)
    c = wl.dirichlet_weights(3, 2, 45)
    prob = q.problem_from_instance(inst)
    s = q.make_schedule("bsb", steps=1000, dt=0.5, seed=46, path=path)
    _, _, _, tr = q.qaia_sample_trace(prob, _dev(c), 5, s, 100)
    _, ref = oracle.sb_sample(inst, c, 5, 1000, "bsb", dt=0.5, seed=46, trace_steps=100)
    err = rel_inf_error(tr.cpu().numpy(), ref)
    print(f"dense fp32 complete-70: max rel err {err.max():.3e}")
    assert err.max() <= 1e-5


@pytest.mark.parametrize("path", DENSE_PATHS)
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp8"])
def test_dense_dsb_trace_parity(q, prec, path):
    """Discrete SB with exactly representable weights: every precision follows the
    FP64 oracle within 1e-5 for 100 steps (seed pre-screened away from x = 0)."""
    inst = _small_int_instance(40, 3, seed=47)
    c = wl.dirichlet_weights(2, 3, 48)
    seed = None
    for sd in range(200, 260):
        _, ref = oracle.sb_sample(inst, c, 2, 1000, "dsb", dt=0.5, seed=sd, trace_steps=100)
        if np.abs(ref).min() >= 1e-4:
            seed = sd
            break
    if seed is None:
        pytest.skip("no seed without near-zero crossings")
    prob = q.problem_from_instance(inst)
    s = q.make_schedule("dsb", precision=prec, steps=1000, dt=0.5, seed=seed, path=path)
    _, _, _, tr = q.qaia_sample_trace(prob, _dev(c), 2, s, 100)
    err = rel_inf_error(tr.cpu().numpy(), ref)
    print(f"dense dsb {prec}: max rel err {err.max():.3e}")
    assert err.max() <= 1e-5


@pytest.mark.parametrize("path", DENSE_PATHS)
def test_low_precision_reproduces_fp32_bitwise_when_exact(q, path):
    """With weights exact in bf16 and e4m3 every product and partial sum is an
    exact integer in fp32, so the BF16 and FP8 forms of discrete SB must produce
    exactly the FP32 dense trajectory and spins."""
    inst = _small_int_instance(96, 3, seed=49)
    c = wl.dirichlet_weights(8, 3, 50)
    prob = q.problem_from_instance(inst)
    outs = {}
    for prec in ("fp32", "bf16", "fp8"):
        s = q.make_schedule("dsb", precision=prec, steps=400, dt=0.5, seed=51, path=path)
        sp, ob, _, tr = q.qaia_sample_trace(prob, _dev(c), 16, s, 50)
        outs[prec] = (sp.cpu().numpy(), ob.cpu().numpy(), tr.cpu().numpy())
    for prec in ("bf16", "fp8"):
        assert np.array_equal(outs[prec][2], outs["fp32"][2]), prec
        assert np.array_equal(outs[prec][0], outs["fp32"][0]), prec
        assert np.array_equal(outs[prec][1], outs["fp32"][1]), prec


def test_staged_tile_order_at_scale_matches_register_tiles(q):
    """At 1024 spins x 2048 columns (8 x 16 tiles) the staged kernel deals its
    tiles to the XCDs in row-first patches (each XCD a quarter of the row
    tiles times half of the column tiles); with exact weights both dense
    kernels compute exact fields, so their spins and cuts agree bit for bit
    in every precision: a tile computed twice or not at all would not."""
    import torch
    inst = _small_int_instance(1024, 3, seed=61)
    c = wl.dirichlet_weights(256, 3, 62)
    prob = q.problem_from_instance(inst)
    for prec in ("fp32", "bf16", "fp8"):
        got = {}
        for path in DENSE_PATHS:
            s = q.make_schedule("dsb", precision=prec, steps=150, dt=0.5, seed=63, path=path)
            sp, ob, _ = q.qaia_sample(prob, _dev(c), 8, s)
            torch.cuda.synchronize()
            got[path] = (sp.cpu().numpy(), ob.cpu().numpy())
        a, b = (got[p_] for p_ in DENSE_PATHS)
        assert np.array_equal(a[0], b[0]), prec
        assert np.array_equal(a[1], b[1]), prec


# ---------------------------------------------------------------- exact cuts

@pytest.mark.parametrize("path", DENSE_PATHS)
@pytest.mark.parametrize("variant,prec", [("bsb", "fp32"), ("dsb", "fp32"), ("dsb", "bf16"), ("dsb", "fp8")])
def test_dense_cut_values_bit_exact(q, variant, prec, path):
    inst = wl.random_instance(150, 3, "complete", seed=52)
    c = wl.dirichlet_weights(16, 3, 53)
    prob = q.problem_from_instance(inst)
    s = q.make_schedule(variant, precision=prec, steps=300, dt=0.5, seed=54, path=path)
    import torch
    spins, obj, ws = q.qaia_sample(prob, _dev(c), 8, s)
    torch.cuda.synchronize()
    spins, obj = spins.cpu().numpy(), obj.cpu().numpy()
    assert np.array_equal(obj, oracle.cut_values(inst, unpack_spins(spins, inst.n)))
    # well above a random cut in the scalarised objective
    cr = np.repeat(c, 8, axis=0).astype(np.float64)
    assert np.mean((obj * cr).sum(1) > (inst.weights.sum(1) / 2.0 * cr).sum(1)) > 0.95
    assert q.qaia_workspace_status(ws) is None


@pytest.mark.parametrize("path", DENSE_PATHS)
def test_dense_invalid_rows_and_determinism(q, path):
    import torch
    inst = wl.random_instance(90, 2, "p0.3", seed=55)
    c = wl.dirichlet_weights(5, 2, 56)
    c[2] = [np.nan, 1.0]
    prob = q.problem_from_instance(inst)
    s = q.make_schedule("dsb", precision="bf16", steps=200, seed=57, path=path)
    a, oa, ws = q.qaia_sample(prob, _dev(c), 4, s)
    b, ob, _ = q.qaia_sample(prob, _dev(c), 4, s)
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(oa, ob)
    assert q.qaia_workspace_status(ws) == 2
    assert not a[8:12].any() and not oa[8:12].any()


@pytest.mark.parametrize("m", [1, 2, 3, 4])
@pytest.mark.parametrize("variant,prec", [("bsb", "fp32"), ("dsb", "bf16"), ("dsb", "fp8")])
def test_staged_tiles_match_register_tiles_when_exact(q, variant, prec, m):
    """Exact weights make every partial sum an exact integer, so the two tile
    kernels must agree bit for bit whatever their k order: 300 spins (three
    128-spin tiles, ragged) and 20 x 16 replicas (three 128-column tiles,
    ragged).  The staged variants this covers: 128-byte chunks in three
    stages (m <= 2) or two (m = 3), 64-byte chunks for m = 4 (where an FP8
    chunk holds one k-group and the units split the accumulators); four
    waves (FP32) or eight (BF16, FP8); x and y prefetched during the k loop
    (m = 1, and m = 2 in FP32) or loaded after it."""
    inst = _small_int_instance(300, m, seed=60, kind="p0.6")
    c = wl.dirichlet_weights(20, m, 61)
    prob = q.problem_from_instance(inst)
    outs = []
    for path in DENSE_PATHS:
        s = q.make_schedule(variant, precision=prec, steps=300, dt=0.5, seed=62, path=path)
        sp, ob, _, tr = q.qaia_sample_trace(prob, _dev(c), 16, s, 40)
        outs.append((sp.cpu().numpy(), ob.cpu().numpy(), tr.cpu().numpy()))
    for a, b in zip(outs[0], outs[1]):
        assert np.array_equal(a, b)
    assert np.array_equal(outs[0][1], oracle.cut_values(inst, unpack_spins(outs[0][0], inst.n)))


@pytest.mark.parametrize("prec,m", [("bf16", 2), ("bf16", 3), ("fp8", 2), ("fp8", 3)])
def test_wide_tiles_match_register_tiles_when_exact(q, prec, m):
    """Launches whose columns fill 256-column tiles, with at least one such
    tile per CU, run the 128 x 256 wide tile (eight waves on 32 x 128 wave
    tiles, one fragment set, 64-byte chunks) in BF16 with m = 2 or 3 and in
    FP8 with m = 3 (each chunk one k-group, so a unit is half of the wave's
    four column blocks); FP8 with m = 2 runs the 128 x 128 tile.  At 2000
    spins (16 row tiles, the last ragged) and 500 x 8 = 4000 replicas (the
    last column tile ragged) every case agrees bit for bit with the register
    tiles under exact weights."""
    import torch
    inst = _small_int_instance(2000, m, seed=70 + m)
    c = wl.dirichlet_weights(500, m, 71)
    prob = q.problem_from_instance(inst)
    got = []
    for path in DENSE_PATHS:
        s = q.make_schedule("dsb", precision=prec, steps=60, dt=0.5, seed=72, path=path)
        sp, ob, _ = q.qaia_sample(prob, _dev(c), 8, s)
        torch.cuda.synchronize()
        got.append((sp.cpu().numpy(), ob.cpu().numpy()))
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])


# ---------------------------------------------------------------- field error (precision form)

def test_field_exact_for_small_integers(q):
    inst = _small_int_instance(130, 4, seed=58, kind="p0.7")
    prob = q.problem_from_instance(inst)
    rng = np.random.default_rng(1)
    phi = (1 - 2 * rng.integers(0, 2, size=(37, inst.n))).astype(np.float64)
    ref = oracle.objective_fields(inst, phi)
    for prec in (0, 1, 2):
        assert np.array_equal(_field(q, prob, prec, phi), ref), prec


def test_field_error_against_fp64(q):
    """Gaussian fixed-point weights on a complete 512-node graph, random +-1 spins:
    relative RMS field error vs the FP64 oracle (stated, and bounded by the
    formats' unit roundoff: fp32 2^-24, bf16 2^-9, e4m3 2^-4)."""
    inst = wl.random_instance(512, 3, "complete", seed=59)
    prob = q.problem_from_instance(inst)
    rng = np.random.default_rng(2)
    phi = (1 - 2 * rng.integers(0, 2, size=(64, inst.n))).astype(np.float64)
    ref = oracle.objective_fields(inst, phi)
    rms_ref = np.sqrt((ref ** 2).mean())
    errs = {}
    for prec, name in ((0, "fp32"), (1, "bf16"), (2, "fp8")):
        f = _field(q, prob, prec, phi)
        errs[name] = (np.sqrt(((f - ref) ** 2).mean()) / rms_ref, np.abs(f - ref).max() / np.abs(ref).max())
        print(f"field error {name}: rel RMS {errs[name][0]:.3e}, rel inf {errs[name][1]:.3e}")
    assert errs["fp32"][0] < 1e-6
    assert errs["bf16"][0] < 4e-3
    assert errs["fp8"][0] < 6e-2
    assert errs["fp32"][0] < errs["bf16"][0] < errs["fp8"][0]


def _both_tiles(q, n, m, W, R, T, variant, prec, alpha, trace_steps=3, kind="complete", bad=()):
    """Spins, cuts and the traced x of the staged path and of the register
    tiles (64 x 128, one launch per step), which do the same arithmetic."""
    import torch
    inst = wl.random_instance(n, m, kind, seed=2100 + n)
    p = q.problem_from_instance(inst)
    c = wl.dirichlet_weights(W, m, 2200 + n)
    for row in bad:
        c[row] = -1.0
    c = torch.from_numpy(c).cuda()
    out = []
    for path in ("dense_staged", "dense"):
        s = q.make_schedule(variant, precision=prec, steps=T, dt=0.5, noise_alpha=alpha, seed=23, replica_offset=5,
                            path=path)
        spins, obj, ws, tr = q.qaia_sample_trace(p, c, R, s, trace_steps)
        torch.cuda.synchronize()
        assert q.qaia_workspace_status(ws) == (min(bad) if bad else None)
        out.append([t.cpu().numpy() for t in (spins, obj, tr)])
    return inst, out


@pytest.mark.parametrize("n,m,W,R,T", [
    (2, 1, 1, 1, 5), (31, 2, 3, 11, 40), (32, 3, 1, 32, 40), (33, 4, 11, 3, 40), (64, 1, 33, 1, 40), (65, 3, 5, 13, 40),
    (97, 4, 3, 43, 40), (128, 2, 1, 127, 40), (255, 3, 4, 8, 25), (256, 4, 1, 33, 25), (257, 3, 2, 16, 25),
    (509, 4, 3, 11, 15), (512, 3, 1, 64, 15)])
@pytest.mark.parametrize("variant,prec,alpha", [("bsb", "fp32", 0.0), ("dsb", "fp32", 0.1), ("bsb", "fp32", 0.2),
                                                ("dsb", "bf16", 0.0), ("dsb", "fp8", 0.1)])
def test_resident_run_equals_register_tiles_bitwise(q, n, m, W, R, T, variant, prec, alpha):
    """Up to 512 spins the staged path keeps a block's columns on chip for all
    steps: edges of its 32-spin tiles, k-groups (8, 16, 64 spins), column tiles
    (1, 2 or 4 per block, ragged) and wave counts (1 to 16), with an invalid
    weight row where there is more than one."""
    bad = (W - 1,) if W > 1 else ()
    inst, (a, b) = _both_tiles(q, n, m, W, R, T, variant, prec, alpha, bad=bad)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    rows = W * R - len(bad) * R
    assert np.array_equal(a[1][:rows], oracle.cut_values(inst, unpack_spins(a[0][:rows], n)))


@pytest.mark.parametrize("n,m,W,R", [(513, 1, 3, 50), (520, 2, 2, 64), (600, 3, 1, 129), (640, 4, 5, 27)])
@pytest.mark.parametrize("variant,prec,alpha", [("bsb", "fp32", 0.0), ("dsb", "fp32", 0.1), ("dsb", "bf16", 0.0),
                                                ("dsb", "fp8", 0.0)])
def test_staged_tiles_equal_register_tiles_bitwise(q, n, m, W, R, variant, prec, alpha):
    """Past 512 spins the staged path launches its LDS tiles step by step."""
    _, (a, b) = _both_tiles(q, n, m, W, R, 10, variant, prec, alpha)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("n,W,R", [(5, 3, 50), (40, 5, 13), (70, 2, 64), (100, 3, 43), (130, 2, 33), (190, 1, 32),
                                   (200, 3, 11), (250, 2, 40), (300, 1, 65), (321, 2, 16)])
@pytest.mark.parametrize("largest,alpha", [(127, 0.1), (128, 0.0), (32639, 0.0), (32640, 0.1), ("edge", 0.1), ("over", 0.1),
                                           (8355711, 0.0), (8355712, 0.0)])
def test_exact_digits_equal_register_tiles_bitwise(q, n, W, R, largest, alpha):
    """Discrete SB in single precision multiplies base-256 digits where rounding
    cannot differ: one, two and three digits at their largest weights, every
    number of 32-spin groups, a row whose weights add up to 2^24 - 1 (exact) and
    to 2^24 (the FP32 product), against the register tiles' FP32 product."""
    import torch
    m = 1 + n % 4
    u, v = np.triu_indices(n, 1)
    rng = np.random.default_rng(n)
    if isinstance(largest, str):
        top = ((1 << 24) - 1) // (n - 1)
        w = rng.choice([-1, 1], size=(m, u.size)) * rng.integers(top // 2, top + 1, size=(m, u.size))
        first = u == 0
        total = np.abs(w[0][first]).sum()
        w[0, 0] += np.sign(w[0, 0]) * ((1 << 24) - (largest == "edge") - total)
        assert np.abs(w[0][first]).sum() == (1 << 24) - (largest == "edge")
    else:
        # few large weights per row, so that the rows' sums stay below 2^24 where that is possible
        w = rng.integers(-3, 4, size=(m, u.size))
        w[:, 0] = -largest
        w[:, -1] = largest
    inst = wl.Instance(n, m, u.astype(np.int32), v.astype(np.int32), w.astype(np.int32))
    p = q.problem_from_instance(inst)
    c = torch.from_numpy(wl.dirichlet_weights(W, m, 17)).cuda()
    out = []
    for path in ("dense_staged", "dense"):
        s = q.make_schedule("dsb", steps=25, dt=0.5, noise_alpha=alpha, seed=29, path=path)
        spins, obj, ws, tr = q.qaia_sample_trace(p, c, R, s, 25)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (spins, obj, tr)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    assert np.array_equal(out[0][1], oracle.cut_values(inst, unpack_spins(out[0][0], n)))


@pytest.mark.parametrize("largest,frac", [(1, 0), (255, 0), (448, 0), (449, 4), (262143, 16), (2**31 - 1, 16)])
def test_image_rounding(q, largest, frac):
    """The reduced images' values, read off as the field of disjoint edges: ties,
    subnormals, every binade and both signs, against the host's conversions of
    the scaled weights."""
    import torch
    rng = np.random.default_rng(largest % 997)
    mags = [largest] + [largest >> s for s in range(1, 31)] + [(3 * largest) >> (s + 1) for s in range(1, 30)]
    mags += [(17 << s) >> 1 for s in range(0, 27)] + [(257 << s) >> 1 for s in range(0, 22)]
    mags += rng.integers(0, largest + 1, 150).tolist()
    w = np.array([x for x in mags if 0 <= x <= largest], np.int64)
    w[1::2] *= -1
    n = 2 * w.size
    inst = wl.Instance(n, 1, np.arange(0, n, 2, dtype=np.int32), np.arange(1, n, 2, dtype=np.int32),
                       w.astype(np.int32)[None], frac)
    p = q.problem_from_instance(inst)
    phi = torch.ones((1, n), device="cuda")
    e16 = int(np.floor(np.log2(largest))) - 7
    e8 = int(np.ceil(np.log2(largest / 448.0)))
    e8 += int(largest * 2.0**-e8 > 448)
    v16 = torch.from_numpy(w * 2.0**-e16).float().to(torch.bfloat16).double() * 2.0**e16
    v8 = torch.from_numpy(w * 2.0**-e8).float().to(torch.float8_e4m3fn).double() * 2.0**e8
    for prec, want in (("bf16", v16), ("fp8", v8), ("fp32", torch.from_numpy(w).float().double())):
        got = q.qaia_dense_field(p, prec, phi).cpu().double()[0, 0]
        assert torch.equal(got[0::2], want) and torch.equal(got[1::2], want), prec


@pytest.mark.parametrize("n,m,W,R", [(257, 1, 3, 50), (300, 2, 1, 2049), (384, 3, 5, 27), (512, 4, 2, 1024), (512, 1, 1, 2049),
                                     (640, 2, 13, 99), (700, 4, 1, 1), (1030, 3, 7, 9)])
@pytest.mark.parametrize("variant,alpha", [("bsb", 0.0), ("dsb", 0.0), ("bsb", 0.2), ("dsb", 0.1)])
def test_thin_tiles_equal_register_tiles_bitwise(q, n, m, W, R, variant, alpha):
    """FP32 with few columns: steps of 64 x 64 tiles, on both sides of one and
    two tiles per CU, ragged columns and padded rows."""
    _, (a, b) = _both_tiles(q, n, m, W, R, 9, variant, "fp32", alpha)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
