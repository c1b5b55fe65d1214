"""The set-up and post-processing kernels at the edges of their tiles and
dispatch rules (needs an MI355X and the built libjarq.so): sizes just below, at
and above a tile, remainders, unaligned pointers, and inputs that fp32
arithmetic turns into infinities or NaN.  References are the float64 oracle or
plain torch in float64."""

import numpy as np
import pytest
import torch

import paper_2609_38599_amd as jq
from oracle import hosts, jarq, post
from oracle.qep import corrected_weights
from paper_2609_38599_amd import binding as jb
from tests._gpu_common import (GpuLayer, check_scales, random_layer, to_dev)

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


# Scales of well-conditioned systems from fp32 Gram entries and W H: four times
# the largest error over these layers (9.9e-7 of a scale, at G = 128)
WELL_RTOL = 4e-6


def _spd(d, seed):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((2 * d, d)) * (1.0 + 4.0 * (rng.random(d) < 0.05))
    H = X.T @ X / (2 * d)
    H += 0.01 * np.mean(np.diag(H)) * np.eye(d)
    return np.ascontiguousarray(H.astype(np.float32))


# G = cols / g systems: one panel of 16, its edges, one and two rows a lane
@pytest.mark.parametrize("G", [1, 15, 16, 17, 32, 33, 48, 63, 64, 65, 80, 81, 96, 97, 112, 113, 128])
def test_scale_solve_sizes(G):
    g = 32
    W, H, q, s, z = random_layer(21, G * g, g, 3, seed=G)
    gk = GpuLayer(W, H, q, s, z, g, 3)
    # a byte pattern that reads as NaN: what no kernel wrote must not matter
    gk.ws.fill_(0xff)
    jq.prepare(gk.p, gk.W, gk.H, gk.ws)
    gk.scale_step()
    _, sg = gk.state()
    ref, ridge = jarq.scale_step(W, H, q, z, g)
    assert not ridge.any()
    check_scales(sg, ref, f" G={G}", WELL_RTOL)
    g2 = GpuLayer(W, H, q, s, z, g, 3, sweeps=1)
    g2.ws.fill_(0xff)
    jq.prepare(g2.p, g2.W, g2.H, g2.ws)
    st = jq.sweeps(g2.p, g2.W, g2.H, g2.codes, g2.scales, g2.zeros, g2.ws)
    assert st["ridge_rows"][0] == 0
    check_scales(g2.state()[1], ref, f" sweep G={G}", WELL_RTOL)


# panels of 512 columns, their remainders, one and two row blocks a work-group
@pytest.mark.parametrize("rows,cols,g", [(17, 512, 32), (33, 544, 32), (70, 640, 128), (5, 1088, 64),
                                         (4100, 640, 64)])
def test_gptq_panels(rows, cols, g):
    rng = np.random.default_rng(cols + rows)
    W = (0.02 * rng.standard_normal((rows, cols))).astype(np.float32)
    H = _spd(cols, cols)
    p = jq.make_params(rows, cols, g, 3)
    q, s, z = jb.gptq(p, to_dev(W), to_dev(H))
    some = np.unique(np.linspace(0, rows - 1, 24).astype(int))
    qo, so, zo = hosts.gptq_host(W[some], H, g, 3)
    assert np.array_equal(q.cpu().numpy()[some], qo)
    assert np.array_equal(s.cpu().numpy()[some], so)
    assert np.array_equal(z.cpu().numpy()[some], zo)


# diagonal inverses doubled up to 512 columns: every kind of remainder
@pytest.mark.parametrize("cols", [32, 64, 96, 160, 224, 352, 512, 544, 608, 736, 992, 1120])
def test_corrected_target_remainders(cols):
    rows = 19
    rng = np.random.default_rng(cols)
    W = (0.02 * rng.standard_normal((rows, cols))).astype(np.float32)
    H = _spd(cols, cols)
    D = 0.05 * rng.standard_normal((cols, cols))
    p = jq.make_params(rows, cols, 32, 3)
    got = jb.qep_correct(p, to_dev(W), to_dev(H), to_dev(D), 0.25).cpu().numpy().astype(np.float64)
    ref = corrected_weights(W, H, D, 0.25)   # the oracle's W + 0.75 (W D^T) H^-1
    # the bound of the full-size test: half an fp32 ulp and 1e-9 of the correction
    bound = 0.5 * np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64) * 1.0001 + \
        1e-9 * np.abs(ref - W).max()
    assert np.all(np.abs(got - ref) <= bound)


def _hess64(X):
    X = X.double()
    return X.t() @ X


# tiles of 128 and 64 channels, chunks of 32 to 256 tokens, and their remainders
@pytest.mark.parametrize("m,d", [(1, 8), (31, 64), (33, 72), (255, 128), (257, 136), (300, 200),
                                 (129, 320), (513, 1024), (40, 4104)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_hessian_tiles(m, d, dtype):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m * 10007 + d)
    X = torch.randn(m, d, generator=gen, device="cuda").to(dtype)
    H0 = torch.randn(d, d, generator=gen, device="cuda", dtype=torch.float64)
    H0 = H0 + H0.t()
    H = H0.clone()
    jb.hessian_accumulate(X, H, 0.5)
    assert torch.equal(H, H.t())
    # fp32 sums of at most 256 products: (256 + 1) u |X|^T |X| covers them
    bound = 0.5 * 257 * 2.0 ** -24 * _hess64(X.abs()) + 1e-12 * H0.abs()
    assert bool(((H - H0 - 0.5 * _hess64(X)).abs() <= bound).all())


@pytest.mark.parametrize("m,d", [(33, 72), (300, 200), (64, 1152)])
def test_cross_tiles(m, d):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + d)
    X = torch.randn(m, d, generator=gen, device="cuda")
    Xq = X + 0.1 * torch.randn(m, d, generator=gen, device="cuda")
    D = torch.zeros(d, d, device="cuda", dtype=torch.float64)
    jb.cross_accumulate(Xq, X, D, 2.0)
    diff = (X - Xq).double()
    bound = 2.0 * 257 * 2.0 ** -24 * (Xq.double().abs().t() @ diff.abs()) + 1e-300
    assert bool(((D - 2.0 * (Xq.double().t() @ diff)).abs() <= bound).all())


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38, 1e30, 1e-40])
def test_hessian_of_extreme_inputs_is_fp32_arithmetic(value):
    """Infinities, NaN, values that round to infinity in bf16, overflow and
    denormals: what fp32 products and sums of them give."""
    m, d = 70, 136
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    X = torch.randint(-3, 4, (m, d), generator=gen, device="cuda").float()
    X[5, 3] = value
    X[9, 130] = value
    X[20:30, 7] = 0.0
    H = torch.zeros(d, d, device="cuda", dtype=torch.float64)
    jb.hessian_accumulate(X, H, 1.0)
    Xc = X.cpu()
    ref = torch.zeros(d, d)
    for t in range(m):
        ref = ref + Xc[t][:, None] * Xc[t][None, :]
    got = H.cpu()
    fin = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(got) & (got.abs() <= 3.5e38), fin)
    # (two products of finite values that overflow with opposite signs: NaN where
    # each is rounded, an infinity where they are fused into the sum)
    if not np.isfinite(value):
        assert torch.equal(torch.isnan(got), torch.isnan(ref))
    tol = 257 * 2.0 ** -24 * (Xc.double().nan_to_num(0, 0, 0).abs().t()
                              @ Xc.double().nan_to_num(0, 0, 0).abs()) + 1e-44
    assert bool(((got - ref.double()).abs() <= tol)[fin].all())


@pytest.mark.parametrize("rows,cols,g", [(3, 32, 32), (64, 64, 64), (65, 192, 64), (130, 2176, 128),
                                         (2050, 2176, 128)])
def test_objective_tiles(rows, cols, g):
    W, H, q, s, z = random_layer(rows, cols, g, 4, seed=rows)
    gk = GpuLayer(W, H, q, s, z, g, 4, prepare=False)
    F = jarq.objective_rows(W, H, q, s, z, g)
    assert np.all(np.abs(gk.objective() - F) <= 1e-5 * F)


def test_objective_of_an_infinite_weight():
    W, H, q, s, z = random_layer(70, 128, 64, 4, seed=3)
    W[5, 9] = np.inf
    W[69, 100] = np.nan
    F = GpuLayer(W, H, q, s, z, 64, 4, prepare=False).objective()
    ref = jarq.objective_rows(np.delete(W, [5, 69], 0), H, np.delete(q, [5, 69], 0),
                              np.delete(s, [5, 69], 0), np.delete(z, [5, 69], 0), 64)
    assert not np.isfinite(F[5]) and not np.isfinite(F[69])
    assert np.all(np.abs(np.delete(F, [5, 69]) - ref) <= 1e-5 * ref)


@pytest.mark.parametrize("g", [32, 64, 128])
def test_rtn_ties_and_non_finite_weights(g):
    """Weights on the grid's halves (exact ties), and groups with an infinity
    or NaN, round as a correctly rounded division does."""
    rows, cols, bits = 9, 4 * g, 3
    rng = np.random.default_rng(g)
    W = rng.integers(-14, 15, (rows, cols)).astype(np.float32) * np.float32(0.5)
    W[:, 0], W[:, 1] = -3.5, 3.5
    W[2, g + 3] = np.inf
    W[3, g + 3] = -np.inf
    W[4, g + 3] = np.nan
    W[5, :g] = 0.0
    W[6] *= np.float32(1e-42)
    p = jq.make_params(rows, cols, g, bits)
    q, s, z = (t.cpu().numpy() for t in jb.rtn(p, to_dev(W)))
    with np.errstate(all="ignore"):
        qo, so, zo = hosts.rtn_host(W, g, bits)
    ok = np.isfinite(W).reshape(rows, -1, g).all(2)
    assert np.array_equal(s[ok], so[ok]) and np.array_equal(z[ok], zo[ok])
    wide = np.repeat(ok, g, axis=1)
    assert np.array_equal(q[wide], qo[wide])
    assert q.max() <= 7


def _refined(rows, cols, g, bits, seed):
    rng = np.random.default_rng(seed)
    q = rng.integers(0, 1 << bits, (rows, cols)).astype(np.uint8)
    s = (0.01 * rng.standard_normal((rows, cols // g))).astype(np.float32)
    z = rng.integers(0, 1 << bits, (rows, cols // g)).astype(np.int32)
    return q, s, z


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("perm", [False, True])
def test_dequantize_any_alignment(dtype, shift, perm):
    """Codes and outputs that are not 16-byte aligned, and a permutation with
    entries outside the columns (skipped, the columns they miss left alone)."""
    rows, cols, g = 13, 416, 32
    q, s, z = _refined(rows, cols, g, 4, 1)
    p = jq.make_params(rows, cols, g, 4)
    buf = torch.empty(rows * cols + 16, dtype=torch.uint8, device="cuda")
    codes = buf[shift:shift + rows * cols].view(rows, cols)
    codes.copy_(to_dev(q))
    out = torch.full((rows * cols + 16,), 7.0, dtype=dtype, device="cuda")
    o = out[shift:shift + rows * cols].view(rows, cols)
    pm = None
    order = np.arange(cols)
    if perm:
        order = np.random.default_rng(2).permutation(cols)
        order[5], order[40] = -1, cols
        pm = to_dev(order.astype(np.int32))
    jb.dequantize(p, codes, to_dev(s), to_dev(z), dtype=dtype, perm=pm, out=o)
    w = s.repeat(g, axis=1) * (q.astype(np.float32) - z.repeat(g, axis=1).astype(np.float32))
    ref = torch.full((rows, cols), 7.0, dtype=dtype)
    live = (order >= 0) & (order < cols)
    ref[:, order[live]] = torch.from_numpy(w[:, live]).to(dtype)
    assert torch.equal(o.cpu(), ref)
    assert bool((out[rows * cols + shift:] == 7.0).all()) and bool((out[:shift] == 7.0).all())


@pytest.mark.parametrize("bits", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("shift", [0, 3])
def test_pack_any_alignment(bits, shift):
    rows, cols, g = 11, 352, 32
    q, _, _ = _refined(rows, cols, g, bits, bits)
    p = jq.make_params(rows, cols, g, bits)
    buf = torch.empty(rows * cols + 16, dtype=torch.uint8, device="cuda")
    codes = buf[shift:shift + rows * cols].view(rows, cols)
    codes.copy_(to_dev(q))
    packed = jb.pack_codes(p, codes)
    assert np.array_equal(packed.cpu().numpy().view(np.uint32), post.pack(q, bits))
    back = torch.zeros(rows * cols + 16, dtype=torch.uint8, device="cuda")
    b = back[shift:shift + rows * cols].view(rows, cols)
    jb.unpack_codes(p, packed, out=b)
    assert np.array_equal(b.cpu().numpy(), q)
    assert int(back[rows * cols + shift:].sum()) == 0


@pytest.mark.parametrize("d", [1, 15, 16, 17, 4095, 4096, 4097])
def test_act_order_sizes(d):
    rng = np.random.default_rng(d)
    diag = rng.integers(0, max(2, d // 3), d).astype(np.float32)   # many ties
    H = torch.zeros(d, d, device="cuda")
    H.diagonal().copy_(to_dev(diag))
    perm = jb.act_order(H).cpu().numpy()
    assert np.array_equal(perm, np.argsort(-diag, kind="stable"))


# both tile sizes of the residual product and of W M^T, at and beside the lines
# between them, the same rows in a layer of either kind: the same bits
@pytest.mark.parametrize("few,many,cols,g", [(63, 4100, 1024, 64), (65, 4097, 1056, 32),
                                             (300, 8200, 640, 128), (1000, 3841, 1536, 128)])
def test_small_and_large_tiles_agree(few, many, cols, g):
    W, H, q, s, z = random_layer(many, cols, g, 3, seed=few)
    states = []
    for n in (few, many):
        gk = GpuLayer(W[:n], H, q[:n], s[:n], z[:n], g, 3)
        gk.scale_step()
        gk.code_step(trace=False)
        states.append(gk.state())
    (qa, sa), (qb, sb) = states
    assert np.array_equal(sa, sb[:few]) and np.array_equal(qa, qb[:few])
    s_ref, _ = jarq.scale_step(W[:few], H, q[:few], z[:few], g)
    check_scales(sa, s_ref, f" few {few}", WELL_RTOL)


# the walk of a pair of groups in one part and in many, odd and even numbers of
# groups, and the span of M's formation: the same bits as in a layer of many rows
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 16, 31, 33, 64, 67])
def test_gram_walk_parts_agree(G):
    g = 32
    many = 128 * (512 // ((G + 1) // 2)) + 1 if G > 8 else 4500
    W, H, q, s, z = random_layer(many, G * g, g, 3, seed=G)
    out = []
    for n in (130, many):
        gk = GpuLayer(W[:n], H, q[:n], s[:n], z[:n], g, 3)
        gk.ws.fill_(0xff)
        jq.prepare(gk.p, gk.W, gk.H, gk.ws)
        gk.scale_step()
        out.append(gk.state()[1])
    assert np.array_equal(out[0], out[1][:130])
    check_scales(out[0], jarq.scale_step(W[:130], H, q[:130], z[:130], g)[0], f" G={G}",
                 WELL_RTOL)


def _scales_of(W, H, codes, zeros, g, bits=8):
    gk = GpuLayer(W, H, codes, np.ones((W.shape[0], W.shape[1] // g), np.float32), zeros, g, bits)
    gk.scale_step()
    return gk.state()[1].astype(np.float64)


# W H in small tiles, and in large ones (160 of them and more)
@pytest.mark.parametrize("rows,cols", [(70, 96), (300, 1024), (5200, 1024)])
def test_scales_of_an_integer_layer_are_exact(rows, cols):
    """Integer W, H and codes whose Gram entries and W H fit fp32: everything
    ahead of the fp64 solve is exact, so a scale is its 64-bit value rounded."""
    g = 32
    G = cols // g
    rng = np.random.default_rng(rows + cols)
    X = rng.integers(-1, 2, (cols + 64, cols))
    X[:, 1:] += X[:, :-1]                       # correlated channels
    H = (X.T @ X + 8 * np.eye(cols, dtype=np.int64)).astype(np.float64)
    W = rng.integers(-9, 10, (rows, cols)).astype(np.float64)
    codes = rng.integers(0, 3, (rows, cols)).astype(np.uint8)
    zeros = np.ones((rows, G), np.int32)
    C = codes.astype(np.float64) - 1.0
    # no sum of magnitudes, in any order, passes 2^24
    assert (np.abs(W) @ np.abs(H)).max() < 2 ** 24
    assert (np.abs(C) @ np.abs(H)).max() * g < 2 ** 24
    got = _scales_of(W.astype(np.float32), H.astype(np.float32), codes, zeros, g)
    WH = W @ H
    A = np.empty((rows, G, G))
    for a in range(G):
        T = C[:, a * g:(a + 1) * g] @ H[a * g:(a + 1) * g]
        A[:, a] = (T * C).reshape(rows, G, g).sum(2)
    ref = np.linalg.solve(A, (WH * C).reshape(rows, G, g).sum(2)[:, :, None])[:, :, 0]
    # half an fp32 ulp, and the fp64 solves (condition numbers below 1e4)
    bound = 0.5 * np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64) + \
        1e-11 * np.abs(ref).max(axis=1, keepdims=True)
    assert np.all(np.abs(got - ref) <= bound)


def _one_code_layer(rows, g, seed, value=None):
    """Two groups without correlation between them, one code of 1 in each: a
    scale is (W H)_n / H_nn of that code's column.  Channel scales are powers of
    two over 28 octaves, which scale W, H and W H without rounding."""
    cols = 2 * g
    rng = np.random.default_rng(seed)
    D = np.ldexp(1.0, -rng.integers(0, 29, cols))
    D[0], D[g - 1], D[g], D[2 * g - 1] = 1.0, 2.0 ** -28, 1.0, 2.0 ** -28
    X = rng.standard_normal((4 * g, cols))
    H0 = X.T @ X / (4 * g)
    H0[:g, g:] = H0[g:, :g] = 0.0
    np.fill_diagonal(H0, 1.0)
    H0 = H0.astype(np.float32).astype(np.float64)
    H0 = np.triu(H0) + np.triu(H0, 1).T + np.eye(cols)     # diagonal 2
    W0 = rng.standard_normal((rows, cols)).astype(np.float32).astype(np.float64)
    H, W = H0 * D * D[:, None], W0 / D
    if value is not None:
        W[5, 0] = value
    codes = np.zeros((rows, cols), np.uint8)
    codes[:, 0] = codes[:, g] = 1               # the channels of scale 1
    return W.astype(np.float32), H.astype(np.float32), codes, np.zeros((rows, 2), np.int32)


@pytest.mark.parametrize("rows", [70, 41000])
def test_scales_where_weights_span_many_octaves(rows):
    """W H to fp32 rounding whatever the range of a row of W: sums of 64 terms,
    (64 + 2) u of the sum of magnitudes, and the scale's own rounding."""
    g = 64
    W, H, codes, zeros = _one_code_layer(rows, g, 11)
    got = _scales_of(W, H, codes, zeros, g)
    W, H = W.astype(np.float64), H.astype(np.float64)
    n = [0, g]
    ref, size = (W @ H)[:, n] / 2.0, (np.abs(W) @ np.abs(H))[:, n] / 2.0
    assert np.all(np.abs(got - ref) <= 66 * 2.0 ** -24 * size + 2.0 ** -24 * np.abs(ref))


@pytest.mark.parametrize("rows", [70, 41000])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3.4e38])
def test_scales_of_extreme_weights(rows, value):
    """An infinity, a NaN, or a weight that rounds to infinity in bf16 stays in
    its row and group, and is what fp32 arithmetic makes of it."""
    g = 64
    W, H, codes, zeros = _one_code_layer(rows, g, 12)
    H *= np.float32(0.25)                       # 3.4e38 H_nn is finite
    base = _scales_of(W, H, codes, zeros, g)
    W[5, 0] = value
    got = _scales_of(W, H, codes, zeros, g)
    others = np.delete(np.arange(rows), 5)
    assert np.array_equal(got[others], base[others])
    if np.isfinite(value):
        assert abs(got[5, 0] - value) <= 66 * 2.0 ** -24 * value
    else:
        assert not np.isfinite(got[5, 0])


# the permuted write-back scatters up to 64 rows and gathers from there on
@pytest.mark.parametrize("rows,cols", [(1, 416), (64, 416), (65, 416), (1030, 288), (64, 16384),
                                       (70, 16384)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_dequantize_permuted_rows(rows, cols, dtype):
    g = 32 if cols < 4096 else 128
    q, s, z = _refined(rows, cols, g, 4, rows)
    order = np.random.default_rng(rows).permutation(cols)
    order[7], order[cols - 1] = cols + 3, -2
    out = torch.full((rows, cols), 7.0, dtype=dtype, device="cuda")
    jb.dequantize(jq.make_params(rows, cols, g, 4), to_dev(q), to_dev(s), to_dev(z), dtype=dtype,
                  perm=to_dev(order.astype(np.int32)), out=out)
    w = s.repeat(g, axis=1) * (q.astype(np.float32) - z.repeat(g, axis=1).astype(np.float32))
    ref = torch.full((rows, cols), 7.0, dtype=dtype)
    live = (order >= 0) & (order < cols)
    ref[:, order[live]] = torch.from_numpy(w[:, live]).to(dtype)
    assert torch.equal(out.cpu(), ref)


# the last round of 128-wide tiles whole, in halves and in quarters; bf16: 64-wide
# tiles alone, and whole ones with a last round cut and not
@pytest.mark.parametrize("d,dtype", [(1440, torch.float32), (1928, torch.float32),
                                     (2824, torch.float32), (2816, torch.bfloat16),
                                     (3080, torch.bfloat16), (4168, torch.bfloat16)])
def test_hessian_splits(d, dtype):
    m = 300
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    X = torch.randn(m, d, generator=gen, device="cuda").to(dtype)
    H = torch.zeros(d, d, device="cuda", dtype=torch.float64)
    jb.hessian_accumulate(X, H, 1.0)
    assert torch.equal(H, H.t())
    bound = 257 * 2.0 ** -24 * _hess64(X.abs()) + 1e-300
    assert bool(((H - _hess64(X)).abs() <= bound).all())


@pytest.mark.parametrize("d", [1000, 1096, 1416, 1480, 2312])
def test_cross_splits(d):
    m = 300
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d)
    X = torch.randn(m, d, generator=gen, device="cuda")
    Xq = X + 0.1 * torch.randn(m, d, generator=gen, device="cuda")
    D = torch.zeros(d, d, device="cuda", dtype=torch.float64)
    jb.cross_accumulate(Xq, X, D, 1.0)
    diff = (X - Xq).double()
    bound = 257 * 2.0 ** -24 * (Xq.double().abs().t().contiguous() @ diff.abs()) + 1e-300
    assert bool(((D - Xq.double().t().contiguous() @ diff).abs() <= bound).all())
    # an infinity: that channel's rows alone
    Xq[3, 5] = float("inf")
    E = torch.zeros(d, d, device="cuda", dtype=torch.float64)
    jb.cross_accumulate(Xq, X, E, 1.0)
    keep = torch.arange(d, device="cuda") != 5
    assert not bool(torch.isfinite(E[5]).any()) and not bool(torch.isfinite(E[:, 5]).any())
    some = keep[:, None] & keep[None, :]
    assert bool(((E - D).abs() <= 2 * bound)[some].all())
