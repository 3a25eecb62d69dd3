"""Operator-level parity of the HIP kernels against the CPU oracle, through the
C ABI.  Tolerances: max|gpu-ref| / max|ref| <= 1e-4 in fp32 and <= 2e-2 in bf16
(the bounds the stage step has to meet); most operators are far inside them and
are held to tighter figures derived from one rounding of the output."""
import numpy as np
import pytest
import torch

import synthetic as syn
from oracle import stage as O
from paper_2505_05856_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {torch.float32: 2e-5, torch.bfloat16: 8e-3}   # one output rounding: 2^-8 relative in bf16


def dev(a, dt):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(DEV).to(dt).contiguous()


def host(t):
    return t.float().cpu().numpy().astype(np.float64)


def rnd(shape, seed, dt, scale=1.0):
    a = scale * syn.normal(seed, 0, int(np.prod(shape))).reshape(shape)
    a = a.astype(np.float32)
    return syn.round_to_bf16(a) if dt == torch.bfloat16 else a


def ws_for(rows, cols):
    return torch.empty(B.op_workspace_bytes(rows, cols), dtype=torch.uint8, device=DEV)


@pytest.mark.parametrize("kind", ["layer", "rms"])
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols", [(1, 8), (7, 16), (130, 128), (37, 1600), (9, 4096), (5, 8192), (2, 2056),
                                       (1301, 4096), (270, 5000), (515, 8192)])
def test_layernorm(dt, rows, cols, kind):
    fwd, bwd = O.NORMS[kind]
    op_fwd, op_bwd = (B.op_layernorm_fwd, B.op_layernorm_bwd) if kind == "layer" else (B.op_rmsnorm_fwd, B.op_rmsnorm_bwd)
    x = rnd((rows, cols), 11, dt, 2.0) + 0.5
    x = syn.round_to_bf16(x) if dt == torch.bfloat16 else x
    g = rnd((cols,), 12, dt) * 0.1 + 1
    g = syn.round_to_bf16(g) if dt == torch.bfloat16 else g
    b = rnd((cols,), 13, dt, 0.1)
    dy = rnd((rows, cols), 14, dt)
    dres = rnd((rows, cols), 15, dt)
    y_ref, mu, r = fwd(x.astype(np.float64), g.astype(np.float64), b.astype(np.float64), 1e-5)
    dx_ref, dg_ref, db_ref = bwd(dy.astype(np.float64), x.astype(np.float64), mu, r, g.astype(np.float64))
    tx, tg, tb, tdy, tres = (dev(a, dt) for a in (x, g, b, dy, dres))
    y = torch.empty_like(tx); stats = torch.empty(rows, 2, dtype=torch.float32, device=DEV)
    op_fwd(tx, tg, tb, 1e-5, y, stats)
    assert O.max_rel_err(host(y), y_ref) < TOL[dt]
    assert np.allclose(host(stats)[:, 0], mu, atol=1e-5) and np.allclose(host(stats)[:, 1], r, rtol=1e-5)
    # stats only / y only
    stats2 = torch.zeros_like(stats)
    op_fwd(tx, tg, tb, 1e-5, None, stats2)
    assert torch.equal(stats, stats2)
    dx = torch.empty_like(tx); dg = torch.empty_like(tg); db = torch.empty_like(tb)
    ws = ws_for(rows, cols)
    op_bwd(tdy, tx, stats, tg, None, dx, dg, db, ws)
    assert O.max_rel_err(host(dx), dx_ref) < TOL[dt]
    assert O.max_rel_err(host(dg), dg_ref) < TOL[dt] and O.max_rel_err(host(db), db_ref) < TOL[dt]
    # with the residual gradient added, written in place over dy
    dy2 = tdy.clone()
    dsum = torch.empty_like(tg)
    op_bwd(dy2, tx, stats, tg, tres, dy2, dg, db, ws, dx_colsum=dsum)
    assert O.max_rel_err(host(dy2), dx_ref + dres) < TOL[dt]
    assert O.max_rel_err(host(dg), dg_ref) < TOL[dt] and O.max_rel_err(host(db), db_ref) < TOL[dt]
    # column sums of dx as stored (a bias gradient): exact sum of the kernel's own output up to fp32 ordering
    assert O.max_rel_err(host(dsum), host(dy2).sum(axis=0)) < TOL[dt]


# 16 rows a block and more (7681), a block a row: rows cut short (in columns; the last block's, which come in fours), whole ones;
# the forward's lanes past the row
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols", [(7681, 1032), (8192, 2048), (41, 2568), (1303, 4088), (6, 520), (33, 5000)])
def test_layernorm_a_block_a_row(dt, rows, cols):
    test_layernorm(dt, rows, cols, "layer")


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("kind", [0, 1, 2])
@pytest.mark.parametrize("rows,cols", [(1237, 8), (77, 1032), (300, 4104)])
def test_gelu(dt, kind, rows, cols):
    """Forward, and the backward kernel the stage runs: dx = dy * gelu'(x) and the column sums of dx as stored."""
    x = rnd((rows, cols), 21, dt, 2.5)
    dy = rnd((rows, cols), 22, dt)
    name = ("erf", "tanh", "relu")[kind]
    tx, tdy = dev(x, dt), dev(dy, dt)
    y = torch.empty_like(tx); dx = torch.empty_like(tx)
    db = torch.empty(cols, dtype=dt, device=DEV)
    ws = ws_for(rows, cols)
    B.op_gelu_fwd(tx, y, kind)
    B.op_gelu_bwd(tdy, tx, dx, db, ws, kind)
    dx_ref = dy * O.gelu_grad(x.astype(np.float64), name)
    assert O.max_rel_err(host(y), O.gelu_fwd(x.astype(np.float64), name)) < TOL[dt]
    assert O.max_rel_err(host(dx), dx_ref) < TOL[dt]
    assert O.max_rel_err(host(db), dx_ref.sum(axis=0)) < TOL[dt]
    db2 = torch.empty_like(db)
    B.op_gelu_bwd(tdy, tx, tdy, db2, ws, kind)     # in place
    assert torch.equal(tdy, dx) and torch.equal(db2, db)


def test_gelu_tanh_bf16_far_out():
    """The logistic form of the tanh approximation where its exponential is 0 or overflows."""
    x = torch.tensor([float("inf"), float("nan"), 1e15, -1e15, 3e38, -3e38, 0.0, -0.0, 20.0, -20.0, -100.0, -6.0, 6.0, 1e-30, -1e13, 2e13],
                     dtype=torch.bfloat16, device=DEV).view(2, 8)
    y, dx, db = torch.empty_like(x), torch.empty_like(x), torch.empty(8, dtype=torch.bfloat16, device=DEV)
    B.op_gelu_fwd(x, y, 1)
    B.op_gelu_bwd(torch.ones_like(x), x, dx, db, ws_for(2, 8), 1)
    x64 = x.double()
    s = torch.sigmoid(1.5957691216057308 * (x64 + 0.044715 * x64 ** 3))
    assert torch.allclose(y.double(), x64 * s, rtol=2.0 ** -8, atol=1e-12, equal_nan=True)      # one rounding to bf16
    want = s + x64 * s * (1 - s) * 1.5957691216057308 * (1 + 0.134145 * x64 ** 2)
    far = x.abs() > 1e19    # the square overflows in 32 bits
    assert torch.allclose(dx.double()[~far], want[~far], rtol=2.0 ** -7, atol=1e-9, equal_nan=True)


def test_gelu_tanh_bf16_rounds_to_the_nearest():
    """Value and derivative of every bf16 number between -8 and 8, and -inf."""
    x = torch.arange(-32768, 32768, dtype=torch.int32, device=DEV).to(torch.int16).view(torch.bfloat16)
    x = x[x.float().abs() <= 8].view(-1, 2).repeat(1, 4).contiguous()
    y, dx, db = torch.empty_like(x), torch.empty_like(x), torch.empty(8, dtype=torch.bfloat16, device=DEV)
    B.op_gelu_fwd(x, y, 1)
    B.op_gelu_bwd(torch.ones_like(x), x, dx, db, ws_for(*x.shape), 1)
    x64 = x.double()
    s = torch.sigmoid(1.5957691216057308 * (x64 + 0.044715 * x64 ** 3))
    for got, want in ((y, x64 * s), (dx, s + x64 * s * (1 - s) * 1.5957691216057308 * (1 + 0.134145 * x64 ** 2))):
        seen = want.abs() > 1e-30   # (smaller ones may be flushed)
        assert torch.equal(got[seen], want.bfloat16()[seen])
    low = torch.full((1, 8), -float("inf"), dtype=torch.bfloat16, device=DEV)
    out = torch.empty_like(low)
    B.op_gelu_fwd(low, out, 1)
    assert torch.isnan(out).all()   # -inf * 0, as 0.5 x (1 + tanh u) gives


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols", [(1, 8), (33, 24), (1000, 1600), (4096, 520)])
def test_colsum(dt, rows, cols):
    x = rnd((rows, cols), 31, dt)
    tx = dev(x, dt)
    out = torch.empty(cols, dtype=dt, device=DEV)
    B.op_colsum(tx, out, ws_for(rows, cols))
    assert O.max_rel_err(host(out), x.astype(np.float64).sum(axis=0)) < TOL[dt]


GEMM_SHAPES = [(1, 8, 8), (5, 16, 24), (64, 64, 64), (100, 72, 40), (128, 384, 128), (257, 136, 520),
               (300, 1600, 96), (512, 256, 1024), (1000, 520, 1032), (264, 136, 4104), (2048, 1024, 512),
               (4096, 4096, 192),   # the 256x256 tile in both forms
               (3900, 4200, 128),
               # ragged edges, both forms (rows of 8 elements for TN); every tile of the LDS-direct kernel: GEMM_TILES
               (200, 328, 192), (1096, 1304, 256), (3904, 4200, 128), (3900, 4200, 448)]


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm(dt, mode, M, N, K):
    a = rnd((M, K), 41, dt); b = rnd((K, N), 42, dt)
    bias = rnd((N,), 43, dt); res = rnd((M, N), 44, dt)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    if mode == 0:     # A [M,K], B given as [N,K]
        ta, tb = dev(a, dt), dev(b.T, dt)
    else:             # A given as [K,M], B [K,N]
        ta, tb = dev(a.T, dt), dev(b, dt)
    c = torch.empty(M, N, dtype=dt, device=DEV)
    B.op_gemm(mode, M, N, K, ta, tb, None, None, c)
    assert O.max_rel_err(host(c), ref) < TOL[dt]
    B.op_gemm(mode, M, N, K, ta, tb, dev(bias, dt), dev(res, dt), c)
    assert O.max_rel_err(host(c), ref + bias + res) < TOL[dt]
    # res may be C itself (C += A B): every element is read and written by one lane, once
    c = dev(res, dt)
    B.op_gemm(mode, M, N, K, ta, tb, None, c, c)
    assert O.max_rel_err(host(c), ref + res) < TOL[dt]


def test_calls_go_to_the_current_stream():
    side = torch.cuda.Stream()
    for s in (torch.cuda.current_stream(), side, torch.cuda.current_stream()):
        with torch.cuda.stream(s):
            assert (B._stream_ptr(None) or 0) == torch.cuda.current_stream().cuda_stream == (B._stream_ptr(s) or 0)


# one launch for few rows: waves and passes of rows cut short, slabs of 16 and 32 columns cut short; outputs that lie in the inputs
# (in place, the sums over gamma) take the two launches
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols", [(1, 8), (15, 24), (17, 136), (128, 128), (257, 40), (1000, 776), (1024, 2048), (1025, 48),
                                       (2048, 520), (2049, 72), (33, 2056)])
def test_column_sums_of_few_rows(dt, rows, cols):
    x, dy, dres = rnd((rows, cols), 11, dt, 2.0), rnd((rows, cols), 14, dt), rnd((rows, cols), 15, dt)
    g = rnd((cols,), 12, dt) * 0.1 + 1
    g = syn.round_to_bf16(g) if dt == torch.bfloat16 else g
    tx, tg, tdy, tres = (dev(a, dt) for a in (x, g, dy, dres))
    ws = ws_for(rows, cols)
    new = lambda *shape: torch.full(shape, float("nan"), dtype=dt, device=DEV)
    y, stats = new(rows, cols), torch.empty(rows, 2, dtype=torch.float32, device=DEV)
    B.op_layernorm_fwd(tx, tg, dev(g, dt), 1e-5, y, stats)
    _, mu, r = O.layernorm_fwd(x.astype(np.float64), g.astype(np.float64), g.astype(np.float64), 1e-5)
    dx_ref, dg_ref, db_ref = O.layernorm_bwd(dy.astype(np.float64), x.astype(np.float64), mu, r, g.astype(np.float64))
    for in_place in (False, True):
        src = tdy.clone()
        dx, dg, db = (src, tg.clone(), new(cols)) if in_place else (new(rows, cols), new(cols), new(cols))
        B.op_layernorm_bwd(src, tx, stats, dg if in_place else tg, tres, dx, dg, db, ws)
        assert O.max_rel_err(host(dx), dx_ref + dres) < TOL[dt]
        assert O.max_rel_err(host(dg), dg_ref) < TOL[dt] and O.max_rel_err(host(db), db_ref) < TOL[dt]
    out = new(cols)
    B.op_colsum(tdy, out, ws)
    assert O.max_rel_err(host(out), dy.astype(np.float64).sum(axis=0)) < TOL[dt]
    ref = dy * O.gelu_grad(x.astype(np.float64), "erf")
    dx, src = new(rows, cols), tdy.clone()
    B.op_gelu_bwd(tdy, tx, dx, out, ws, 0)
    assert O.max_rel_err(host(dx), ref) < TOL[dt]
    assert O.max_rel_err(host(out), host(dx).sum(axis=0)) < TOL[dt]   # of dx as stored
    B.op_gelu_bwd(src, tx, src, out, ws, 0)                           # in place
    assert torch.equal(src, dx)


# the last row count, column count and byte count on either side of each rule (GELU 256 and 512 rows, norms 512 and 1000, column sums
# 1800, all but norms 8 MiB)
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols", [(256, 1024), (256, 1032), (257, 1032), (512, 1024), (512, 1032), (513, 72), (1000, 264), (1001, 264),
                                       (1800, 2328), (1800, 2336), (1801, 72), (1800, 1160), (1800, 1168), (512, 8192), (512, 8200),
                                       (256, 8200)])
def test_column_sums_on_either_side_of_each_rule(dt, rows, cols):
    if cols <= 8192:
        test_column_sums_of_few_rows(dt, rows, cols)
        return
    x, dy = dev(rnd((rows, cols), 11, dt), dt), dev(rnd((rows, cols), 14, dt), dt)   # (wider than a norm takes)
    dx, db = torch.empty_like(x), torch.empty(cols, dtype=dt, device=DEV)
    B.op_gelu_bwd(dy, x, dx, db, ws_for(rows, cols), 0)
    assert O.max_rel_err(host(dx), host(dy) * O.gelu_grad(host(x), "erf")) < TOL[dt]
    assert O.max_rel_err(host(db), host(dx).sum(axis=0)) < TOL[dt]


def test_sums_that_lie_in_an_input_take_two_launches():
    """One output in one input a call: the sums then have the bits of the two-pass order, and an input is whole until it is read."""
    dt, rows, cols = torch.float32, 200, 136
    x, dy, dres, g = (dev(rnd(s, seed, dt), dt) for seed, s in ((11, (rows, cols)), (14, (rows, cols)), (15, (rows, cols)), (12, (cols,))))
    stats, ws = torch.empty(rows, 2, dtype=torch.float32, device=DEV), ws_for(rows, cols)
    B.op_layernorm_fwd(x, g, g, 1e-5, torch.empty_like(x), stats)
    st = stats.cpu().numpy()
    sums = {"dg": ordered_sums(dy.cpu().numpy(), 8, (x.cpu().numpy() - st[:, :1]) * st[:, 1:]), "db": ordered_sums(dy.cpu().numpy(), 8)}
    dx, out = torch.empty_like(x), {"dg": torch.empty_like(g), "db": torch.empty_like(g)}
    B.op_layernorm_bwd(dy, x, stats, g, dres, dx, out["dg"], out["db"], ws)
    assert not all(np.array_equal(out[k].cpu().numpy(), sums[k]) for k in sums)   # (one launch adds in another order)
    for which in ("dg", "db"):
        for place in ("x", "dy", "dres", "g", "stats"):
            t = {"x": x.clone(), "dy": dy.clone(), "dres": dres.clone(), "g": g.clone(), "stats": stats.clone()}
            into = dict(out, **{which: t[place].view(-1)[:cols]})
            got = torch.empty_like(x)
            B.op_layernorm_bwd(t["dy"], t["x"], t["stats"], t["g"], t["dres"], got, into["dg"], into["db"], ws)
            assert np.array_equal(into[which].cpu().numpy(), sums[which]), (which, place)
            assert torch.equal(got, dx), (which, place)
    for place in ("x", "dy"):
        t = {"x": x.clone(), "dy": dy.clone()}
        B.op_layernorm_bwd(t["dy"], t["x"], stats, g, dres, t[place], out["dg"], out["db"], ws)
        assert torch.equal(t[place], dx) and all(np.array_equal(out[k].cpu().numpy(), sums[k]) for k in sums)
    want = ordered_sums(dy.cpu().numpy(), 16)
    src = dy.clone()
    B.op_colsum(src, src[7], ws)
    assert np.array_equal(src[7].cpu().numpy(), want)
    want = ordered_sums((dy * (x > 0)).cpu().numpy(), 16)   # ReLU: whole products
    for place in ("x", "dy"):
        t = {"x": x.clone(), "dy": dy.clone()}
        B.op_gelu_bwd(t["dy"], t["x"], torch.empty_like(x), t[place][rows - 1], ws, 2)
        assert np.array_equal(t[place][rows - 1].cpu().numpy(), want), place


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cols", [24, 776, 1600, 2048])
def test_norm_backward_of_few_rows_has_the_dx_of_two_launches(dt, cols):
    rows = 200
    tx, tdy, tres = (dev(rnd((rows, cols), seed, dt), dt) for seed in (11, 14, 15))
    tg, stats = dev(rnd((cols,), 12, dt) * 0.1 + 1, dt), torch.empty(rows, 2, dtype=torch.float32, device=DEV)
    B.op_layernorm_fwd(tx, tg, tg, 1e-5, torch.empty_like(tx), stats)
    for res in (None, tres):
        one, two, (dg, db, ds) = torch.empty_like(tx), torch.empty_like(tx), (torch.empty_like(tg) for _ in range(3))
        B.op_layernorm_bwd(tdy, tx, stats, tg, res, one, dg, db, ws_for(rows, cols))
        B.op_layernorm_bwd(tdy, tx, stats, tg, res, two, dg, db, ws_for(rows, cols), dx_colsum=ds)
        assert torch.equal(one, two)


# the norm backward with the column sums of dx: 8 waves a block up to 2048 rows, and for rows of at most 2 KB up to 4096 (with a residual
# gradient 3072); 4 from there on
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols", [(9, 1608), (1000, 776), (2048, 2048), (2049, 520), (4090, 1024), (2300, 1032), (4097, 72)])
def test_norm_backward_waves(dt, rows, cols):
    x, dy, dres = rnd((rows, cols), 11, dt, 2.0), rnd((rows, cols), 14, dt), rnd((rows, cols), 15, dt)
    g = rnd((cols,), 12, dt) * 0.1 + 1
    g = syn.round_to_bf16(g) if dt == torch.bfloat16 else g
    tx, tg, tdy, tres = (dev(a, dt) for a in (x, g, dy, dres))
    y, stats = torch.empty_like(tx), torch.empty(rows, 2, dtype=torch.float32, device=DEV)
    B.op_layernorm_fwd(tx, tg, tg, 1e-5, y, stats)
    _, mu, r = O.layernorm_fwd(x.astype(np.float64), g.astype(np.float64), g.astype(np.float64), 1e-5)
    dx_ref, dg_ref, db_ref = O.layernorm_bwd(dy.astype(np.float64), x.astype(np.float64), mu, r, g.astype(np.float64))
    for res in (tres, None):
        dx, (dg, db, ds) = torch.full_like(tx, float("nan")), (torch.full_like(tg, float("nan")) for _ in range(3))
        B.op_layernorm_bwd(tdy, tx, stats, tg, res, dx, dg, db, ws_for(rows, cols), dx_colsum=ds)
        assert O.max_rel_err(host(dx), dx_ref + (dres if res is not None else 0)) < TOL[dt]
        assert O.max_rel_err(host(dg), dg_ref) < TOL[dt] and O.max_rel_err(host(db), db_ref) < TOL[dt]
        if res is not None:   # (without it the columns of dx nearly cancel)
            assert O.max_rel_err(host(ds), host(dx).sum(axis=0)) < TOL[dt]


def ordered_sums(a, min_rows, factor=None, waves=4):
    """Column sums of fp32 rows in the two-pass order: blocks of at least `min_rows` rows, wave w of `waves` adds rows w, w + waves, ...
    (with a factor: products, unrounded), the waves in turn, then block g, g + 16, ... in 16 groups, the groups in turn."""
    rows, cols = a.shape
    nb = min(512, -(-rows // min_rows))
    rpb = -(-rows // nb)
    nb = -(-rows // rpb)
    acc = np.zeros((nb, waves, cols), np.float32)
    for at in range(0, rpb, waves):
        r = np.arange(nb)[:, None] * rpb + at + np.arange(waves)
        ok = ((r < rows) & (at + np.arange(waves) < rpb))[..., None]
        r = np.minimum(r, rows - 1)
        v = a[r] if factor is None else a[r].astype(np.longdouble) * factor[r]
        acc = np.where(ok, (acc + v).astype(np.float32), acc)
    part = acc[:, 0]
    for w in range(1, waves):
        part = part + acc[:, w]
    out = np.zeros(cols, np.float32)
    for g in range(16):
        s = np.zeros(cols, np.float32)
        for b in range(g, nb, 16):
            s += part[b]
        out += s
    return out


# however many waves take a block's rows, the sums keep the order of four: the same bits at every row count (row counts on either
# side of each rule; blocks cut short)
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,cols", [(3, 24), (9, 1608), (1000, 776), (2048, 2048), (2049, 520), (2049, 1032), (3072, 512), (3073, 512),
                                       (4096, 1024), (4097, 72)])
def test_norm_backward_sums_keep_their_order(dt, rows, cols):
    tx, tdy, tres = (dev(rnd((rows, cols), seed, dt), dt) for seed in (11, 14, 15))
    tg = dev(rnd((cols,), 12, dt) * 0.1 + 1, dt)
    y, stats = torch.empty_like(tx), torch.empty(rows, 2, dtype=torch.float32, device=DEV)
    B.op_layernorm_fwd(tx, tg, tg, 1e-5, y, stats)
    st, f32 = stats.cpu().numpy(), lambda t: t.float().cpu().numpy()
    xhat = (f32(tx) - st[:, :1]) * st[:, 1:]
    want_dg, want_db = ordered_sums(f32(tdy), 8, xhat), ordered_sums(f32(tdy), 8)
    for res in (None, tres):
        dx, (dg, db, ds) = torch.empty_like(tx), (torch.empty_like(tg) for _ in range(3))
        B.op_layernorm_bwd(tdy, tx, stats, tg, res, dx, dg, db, ws_for(rows, cols), dx_colsum=ds)
        assert torch.equal(dg.cpu(), torch.from_numpy(want_dg).to(dt)) and torch.equal(db.cpu(), torch.from_numpy(want_db).to(dt))
        if dt == torch.bfloat16:   # (in fp32 the sum may take the value before its rounding)
            assert torch.equal(ds.cpu(), torch.from_numpy(ordered_sums(f32(dx), 8)).to(dt))


# sixteen waves a block up to 1024 blocks of at most 16 rows (8192 rows), four from there on: the same order (in fp32 the last kind
# alone: the other sums may take the value before its rounding)
@pytest.mark.parametrize("dt,kind", [(torch.bfloat16, 0), (torch.bfloat16, 1), (torch.float32, 2)])
@pytest.mark.parametrize("rows,cols", [(520, 520), (1000, 3072), (8192, 1024), (8193, 1024), (9001, 264), (2049, 4104)])
def test_gelu_backward_sums_keep_their_order(dt, kind, rows, cols):
    x, dy = dev(rnd((rows, cols), 11, dt), dt), dev(rnd((rows, cols), 14, dt), dt)
    dx, db = torch.empty_like(x), torch.empty(cols, dtype=dt, device=DEV)
    B.op_gelu_bwd(dy, x, dx, db, ws_for(rows, cols), kind)
    assert torch.equal(db.cpu(), torch.from_numpy(ordered_sums(dx.float().cpu().numpy(), 16)).to(dt))


# a row's dx does not depend on how many rows a call has (8 rows a block and 16 or more, several to a wave)
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("cols", [1032, 1600, 2048])
def test_norm_backward_rows_alone_and_among_others(dt, cols):
    rows, few = 8192, 3000
    tx, tdy = dev(rnd((rows, cols), 11, dt), dt), dev(rnd((rows, cols), 14, dt), dt)
    tg, stats = dev(rnd((cols,), 12, dt) * 0.1 + 1, dt), torch.empty(rows, 2, dtype=torch.float32, device=DEV)
    B.op_layernorm_fwd(tx, tg, tg, 1e-5, torch.empty_like(tx), stats)
    out = []
    for n in (rows, few):
        dx, (dg, db, ds) = torch.empty_like(tx[:n]), (torch.empty_like(tg) for _ in range(3))
        B.op_layernorm_bwd(tdy[:n], tx[:n], stats[:n], tg, None, dx, dg, db, ws_for(n, cols), dx_colsum=ds)
        out.append(dx[:few])
    assert torch.equal(*out)


# rows of more than 2048 columns with a guarded end: the residual gradient is added to dx as rounded without it, and the column
# sums are those of dx as stored
@pytest.mark.parametrize("sums", [False, True])
@pytest.mark.parametrize("rows,cols", [(9, 2568), (1303, 4088), (33, 4096), (130, 5000)])
def test_norm_backward_wide_adds_the_residual_to_the_rounded_gradient(rows, cols, sums):
    dt = torch.float32
    tx, tdy, tres = (dev(rnd((rows, cols), seed, dt), dt) for seed in (11, 14, 15))
    tg, stats = dev(rnd((cols,), 12, dt) * 0.1 + 1, dt), torch.empty(rows, 2, dtype=torch.float32, device=DEV)
    B.op_layernorm_fwd(tx, tg, tg, 1e-5, torch.empty_like(tx), stats)
    dx, dxr, (dg, db, ds) = torch.empty_like(tx), torch.empty_like(tx), (torch.empty_like(tg) for _ in range(3))
    for res, out in ((None, dx), (tres, dxr)):
        B.op_layernorm_bwd(tdy, tx, stats, tg, res, out, dg, db, ws_for(rows, cols), dx_colsum=ds if sums else None)
        if sums:
            assert np.array_equal(ds.cpu().numpy(), ordered_sums(out.cpu().numpy(), 8, waves=1))
    assert torch.equal(dxr, dx + tres)


# K that no k-step divides (whole 8-element rows for NT; any K for TN), one k-step and a little more, two, four and more,
# and C, bias and residual rows of 8-byte alignment only (N a multiple of 4)
GEMM_RAGGED_K = [(0, 256, 264, 72), (0, 1096, 1304, 248), (0, 3904, 4200, 200), (0, 3904, 4200, 456), (0, 200, 132, 136),
                 (0, 3904, 4204, 200), (1, 256, 264, 65), (1, 264, 328, 127), (1, 1096, 1304, 250), (1, 3904, 4200, 193),
                 (1, 3904, 4200, 451), (1, 768, 3072, 1000)]


@pytest.mark.parametrize("mode,M,N,K", GEMM_RAGGED_K)
def test_gemm_ragged_k(mode, M, N, K):
    dt = torch.bfloat16
    a = rnd((M, K), 45, dt); b = rnd((K, N), 46, dt)
    bias = rnd((N,), 47, dt); res = rnd((M, N), 48, dt)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    ta, tb = (dev(a, dt), dev(b.T, dt)) if mode == 0 else (dev(a.T, dt), dev(b, dt))
    c = torch.full((M, N), float("nan"), dtype=dt, device=DEV)
    B.op_gemm(mode, M, N, K, ta, tb, None, None, c)
    assert O.max_rel_err(host(c), ref) < TOL[dt]
    B.op_gemm(mode, M, N, K, ta, tb, dev(bias, dt), dev(res, dt), c)
    assert O.max_rel_err(host(c), ref + bias + res) < TOL[dt]
    # 8-byte aligned C and residual
    pad = torch.zeros(M * N + 4, dtype=dt, device=DEV)
    pad[4:].copy_(dev(res, dt).view(-1))
    c8 = pad[4:].view(M, N)
    B.op_gemm(mode, M, N, K, ta, tb, None, c8, c8)
    assert O.max_rel_err(host(c8), ref + res) < TOL[dt]


# Every tile of the LDS-direct kernel in both forms: ragged against it in rows, columns and K (no k-step divides it), rows of
# 8-byte alignment (NT) or of 8 elements (TN); the fewest k-steps the tile's ring of stages takes, one more, several rounds
GEMM_TILES = [((256, 256), 0, 2310, 3332, (136, 200, 456)), ((256, 256), 1, 3336, 2312, (131, 193, 451)),
              ((256, 128), 0, 1667, 2308, (72, 136, 456)), ((256, 128), 1, 1672, 2336, (65, 131, 451)),
              ((128, 256), 0, 2316, 1668, (72, 136, 456)), ((128, 256), 1, 2312, 1672, (65, 131, 451)),
              ((128, 128), 0, 451, 4100, (72, 136, 456)), ((128, 128), 1, 4112, 456, (65, 131, 451)),
              ((128, 64), 0, 193, 4148, (72, 136, 456)), ((128, 64), 1, 200, 4136, (65, 131, 451)),
              ((64, 128), 0, 4143, 196, (72, 136, 456)), ((64, 128), 1, 4136, 200, (65, 131, 451)),
              ((64, 64), 0, 146, 132, (72, 136, 456)), ((64, 64), 1, 136, 168, (65, 131, 451))]


@pytest.mark.parametrize("tile,mode,M,N,K", [(t, mode, M, N, K) for t, mode, M, N, ks in GEMM_TILES for K in ks])
def test_gemm_every_tile_ragged(tile, mode, M, N, K):
    assert B.op_gemm_tile(mode, M, N, K) == tile     # (a change of the rule has to bring other sizes here)
    test_gemm_ragged_k(mode, M, N, K)


# The tiles of 192 rows or columns, which take nine k-steps or more: as above, from the fewest on
GEMM_TILES_192 = [((256, 192), 0, 3670, 2316, (520, 584, 1096)), ((256, 192), 1, 3664, 2312, (515, 577, 1091)),
                  ((192, 256), 0, 2312, 3656, (520, 584, 1096)), ((192, 256), 1, 2320, 3664, (515, 577, 1091)),
                  ((192, 192), 0, 2316, 3336, (520, 584, 1096)), ((192, 192), 1, 3336, 2320, (515, 577, 1091)),
                  ((192, 128), 0, 3212, 1160, (520, 584, 1096)), ((192, 128), 1, 3592, 1032, (515, 577, 1091)),
                  ((128, 192), 0, 1153, 3236, (520, 584, 1096)), ((128, 192), 1, 1032, 3592, (515, 577, 1091))]


@pytest.mark.parametrize("tile,mode,M,N,K", [(t, mode, M, N, K) for t, mode, M, N, ks in GEMM_TILES_192 for K in ks])
def test_gemm_every_192_tile_ragged(tile, mode, M, N, K):
    assert B.op_gemm_tile(mode, M, N, K) == tile
    test_gemm_ragged_k(mode, M, N, K)


# Both products of a linear layer's backward in one launch: every tile on either side, ragged against it in rows, columns and
# contraction, from the fewest k-steps its ring of stages takes
LINEAR_BWD = [(150, 152, 136, (64, 64), (64, 64)), (216, 136, 136, (64, 128), (64, 64)), (394, 136, 152, (128, 64), (64, 64)),
              (1006, 216, 176, (128, 128), (64, 64)), (1857, 136, 136, (256, 128), (64, 64)), (1044, 3024, 136, (128, 256), (64, 64)),
              (2885, 264, 144, (256, 192), (64, 64)), (2070, 2696, 136, (192, 256), (64, 64)), (2814, 2704, 160, (256, 256), (64, 64)),
              (136, 136, 712, (64, 64), (64, 128)), (160, 216, 1064, (64, 64), (128, 64)), (136, 224, 1816, (64, 64), (128, 128)),
              (129, 272, 2160, (64, 64), (256, 128)), (130, 136, 2344, (64, 64), (128, 256)), (131, 2120, 3080, (64, 64), (256, 192)),
              (129, 2208, 2208, (64, 64), (192, 256)), (130, 2728, 2888, (128, 64), (256, 256))]


@pytest.mark.parametrize("T,n_in,n_out,nt,tn", LINEAR_BWD)
def test_linear_backward_in_one_launch_has_the_bits_of_two(T, n_in, n_out, nt, tn, dt=torch.bfloat16):
    if dt == torch.bfloat16:
        assert B.op_linear_bwd_tiles(T, n_in, n_out) == (nt, tn)     # (a change of the rule has to bring other sizes here)
    dy, w, x = (dev(rnd(s, seed, dt), dt) for s, seed in (((T, n_out), 51), ((n_in, n_out), 52), ((T, n_in), 53)))
    res, dw0 = dev(rnd((T, n_in), 54, dt), dt), dev(rnd((n_in, n_out), 55, dt), dt)
    want_dx, want_dw = torch.empty_like(x), torch.empty_like(w)
    for r, acc in ((None, False), (res, True)):
        dx, dw = torch.full_like(x, float("nan")), dw0.clone() if acc else torch.full_like(w, float("nan"))
        B.op_gemm(0, T, n_in, n_out, dy, w, None, r, want_dx)
        B.op_gemm(1, n_in, n_out, T, x, dy, None, dw0 if acc else None, want_dw)
        B.op_linear_bwd(dy, w, x, r, dx, dw, acc)
        assert torch.equal(dx, want_dx) and torch.equal(dw, want_dw)
    dx = res.clone()                                                 # res may be dx
    B.op_linear_bwd(dy, w, x, dx, dx, dw)
    assert torch.equal(dx, want_dx)


# fp32: 16x16 and 32x32 tiles on either side; tiles of 64 (two launches)
@pytest.mark.parametrize("T,n_in,n_out", [(4, 4, 4), (37, 52, 20), (300, 260, 36), (33, 516, 300), (700, 260, 260), (1100, 700, 260)])
def test_linear_backward_f32_has_the_bits_of_two(T, n_in, n_out):
    test_linear_backward_in_one_launch_has_the_bits_of_two(T, n_in, n_out, None, None, torch.float32)


# fp32 on the matrix cores: ragged against the 32- and 64-row parts and the 16-deep chunks, both waves' arrangements
# (64x64 and 32x32 tiles with a divided contraction; 128x128 tiles, TN and short NT ones), fewer chunks than waves, rows of 4
GEMM_F32 = [(0, 4, 4, 4), (0, 33, 36, 20), (0, 65, 132, 68), (0, 1000, 516, 332), (0, 700, 1100, 1028), (1, 4, 4, 4),
            (0, 1413, 1524, 4), (0, 1601, 1604, 20), (0, 1500, 1412, 64), (0, 1500, 1412, 68),
            (1, 36, 20, 5), (1, 68, 132, 67), (1, 516, 1000, 333), (1, 1412, 1524, 129), (1, 1600, 1604, 31)]
# 16x16 tiles up to 256 of them, 32x32 from there on: cut short on either side of that line, short contractions and long ones
GEMM_F32_LINE = [(0, 253, 252, 4), (0, 256, 256, 1028), (0, 257, 252, 132), (0, 255, 260, 516), (1, 252, 256, 3), (1, 256, 252, 515),
                 (1, 260, 252, 67), (1, 20, 2052, 130)]


@pytest.mark.parametrize("mode,M,N,K", GEMM_F32)
def test_gemm_f32(mode, M, N, K):
    dt = torch.float32
    a = rnd((M, K), 45, dt); b = rnd((K, N), 46, dt)
    bias = rnd((N,), 47, dt); res = rnd((M, N), 48, dt)
    ref = a.astype(np.float64) @ b.astype(np.float64)
    ta, tb = (dev(a, dt), dev(b.T, dt)) if mode == 0 else (dev(a.T, dt), dev(b, dt))
    c = torch.full((M, N), float("nan"), dtype=dt, device=DEV)
    tol = 2 * (K + 2) ** 0.5 * 2.0 ** -24     # K roundings of random sign, relative to the largest result
    B.op_gemm(mode, M, N, K, ta, tb, None, None, c)
    assert O.max_rel_err(host(c), ref) < tol
    B.op_gemm(mode, M, N, K, ta, tb, dev(bias, dt), dev(res, dt), c)
    assert O.max_rel_err(host(c), ref + bias + res) < tol
    c = dev(res, dt)
    B.op_gemm(mode, M, N, K, ta, tb, None, c, c)
    assert O.max_rel_err(host(c), ref + res) < tol


@pytest.mark.parametrize("mode,M,N,K", GEMM_F32_LINE)
def test_gemm_f32_small_tiles(mode, M, N, K):
    test_gemm_f32(mode, M, N, K)


# a short contraction over a large output takes a form of its own, which adds chunk sums as the waves of the other form do:
# the first rows alone (too few tiles for it) have the same bits
@pytest.mark.parametrize("K", [4, 20, 40, 64])
def test_gemm_f32_short_contraction_keeps_its_sums(K):
    M, N = 1501, 1412
    a, b = dev(rnd((M, K), 45, torch.float32), torch.float32), dev(rnd((N, K), 46, torch.float32), torch.float32)
    c, part = torch.full((M, N), float("nan"), device=DEV), torch.full((64, N), float("nan"), device=DEV)
    B.op_gemm(0, M, N, K, a, b, None, None, c)
    B.op_gemm(0, 64, N, K, a[:64].contiguous(), b, None, None, part)
    torch.cuda.synchronize()
    assert torch.equal(c[:64], part)


ATTN_SHAPES = [(1, 8, 1, 8), (2, 5, 2, 16), (2, 64, 2, 64), (1, 200, 3, 64), (2, 96, 2, 128), (1, 384, 2, 64),
               (1, 1024, 3, 64), (1, 2048, 2, 128)]     # the last two: sequence and head width of C3/C4 and of C5


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Bn,S,nh,dh", ATTN_SHAPES)
@pytest.mark.parametrize("sharp", [False, True])
def test_attention(dt, causal, Bn, S, nh, dh, sharp):
    H = nh * dh
    qkv = rnd((Bn * S, 3 * H), 51, dt)
    if sharp:     # logits with a standard deviation of a few units
        qkv[:, :2 * H] *= 2.0
        qkv = syn.round_to_bf16(qkv) if dt == torch.bfloat16 else qkv
    d_o = rnd((Bn * S, H), 52, dt)
    q64 = qkv.astype(np.float64)
    o_ref, lse_ref = O.attention_fwd(q64, Bn, S, nh, causal)
    dq_ref = O.attention_bwd(d_o.astype(np.float64), q64, Bn, S, nh, causal)
    tq, tdo = dev(qkv, dt), dev(d_o, dt)
    o = torch.empty(Bn * S, H, dtype=dt, device=DEV)
    lse = torch.empty(Bn, nh, S, dtype=torch.float32, device=DEV)
    B.op_attention_fwd(tq, Bn, S, nh, dh, causal, o, lse)
    tol = TOL[dt] * (2 if dt == torch.bfloat16 else 1)     # P is rounded to bf16 as well
    assert O.max_rel_err(host(o), o_ref) < tol
    assert np.allclose(host(lse), lse_ref, atol=2e-5 if dt == torch.float32 else 2e-3)
    # single outputs
    lse2 = torch.zeros_like(lse)
    B.op_attention_fwd(tq, Bn, S, nh, dh, causal, None, lse2)
    assert torch.equal(lse, lse2)
    dqkv = torch.empty_like(tq)
    ws = ws_for(Bn * S, nh)
    # the backward is fed the oracle-consistent O the kernel itself produced
    B.op_attention_bwd(tq, o, lse, tdo, Bn, S, nh, dh, causal, dqkv, ws)
    got = host(dqkv)
    for blk in range(3):
        assert O.max_rel_err(got[:, blk * H:(blk + 1) * H], dq_ref[:, blk * H:(blk + 1) * H]) < 2 * tol, blk


# a wave a row on the vector ALUs: pieces of 32 columns cut short and whole, the widest head they take and the first they do not,
# batches of eight rows cut short, blocks of four waves (from 2048 rows) with waves left over
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Bn,S,nh,dh", [(1, 1, 1, 32), (2, 7, 3, 24), (1, 33, 2, 40), (3, 65, 2, 72), (1, 47, 2, 128), (1, 31, 2, 136),
                                        (1, 685, 3, 40), (2, 256, 4, 64)])
def test_attention_rows(Bn, S, nh, dh, causal):
    test_attention(torch.float32, causal, Bn, S, nh, dh, False)


# three pieces and four, twice the batches from 64 keys on, in bf16 too; wider heads than the rows kernels take, more than one batch
@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Bn,S,nh,dh", [(2, 63, 2, 24), (2, 64, 2, 40), (1, 129, 2, 72), (1, 70, 1, 96), (1, 67, 2, 104), (1, 685, 3, 40),
                                        (2, 33, 2, 136), (2, 130, 1, 160)])
def test_attention_other_head_dimensions(dt, Bn, S, nh, dh, causal):
    test_attention(dt, causal, Bn, S, nh, dh, False)


# the forward's tile loop: one tile, two, odd and even counts, tiles that end on and just past a boundary, with none, some and
# all of them masked; the last shape has more than two workgroups a CU
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("Bn,S,nh,dh", [(1, s, 2, dh) for dh in (64, 128) for s in (1, 63, 64, 65, 128, 129, 192, 193, 256, 257, 321)]
                         + [(9, 257, 30, 64)])
def test_attention_fwd_tiles(Bn, S, nh, dh, causal):
    dt = torch.bfloat16
    H = nh * dh
    qkv = rnd((Bn * S, 3 * H), 53, dt)
    qkv[:, :H] *= 3.0     # a maximum that moves between tiles
    qkv = syn.round_to_bf16(qkv)
    o_ref, lse_ref = O.attention_fwd(qkv.astype(np.float64), Bn, S, nh, causal)
    o = torch.full((Bn * S, H), float("nan"), dtype=dt, device=DEV)
    lse = torch.full((Bn, nh, S), float("nan"), dtype=torch.float32, device=DEV)
    B.op_attention_fwd(dev(qkv, dt), Bn, S, nh, dh, causal, o, lse)
    assert O.max_rel_err(host(o), o_ref) < 2 * TOL[dt]     # (P is rounded to bf16 as well)
    assert np.allclose(host(lse), lse_ref, atol=2e-3)



# Causal grids of more blocks than CUs take their row tiles by weight (heads that 8 divides and not, one group of heads and more, a
# tile a head and many): every row has the bits it has in a call of its own sample.
@pytest.mark.parametrize("Bn,S,nh,dh", [(9, 257, 30, 64), (5, 700, 13, 64), (8, 1000, 5, 128), (2, 2048, 21, 128), (30, 100, 9, 64), (1, 1500, 32, 64)])
@pytest.mark.parametrize("drop", [None, (0.2, 5, 7, 1)])
def test_causal_attention_by_weight_has_the_bits_of_single_samples(Bn, S, nh, dh, drop):
    dt, H = torch.bfloat16, nh * dh
    qkv, d_o = dev(rnd((Bn * S, 3 * H), 61, dt), dt), dev(rnd((Bn * S, H), 62, dt), dt)

    def run(q, g, n, heads):
        o, lse = torch.full_like(g, float("nan")), torch.full((n, heads, S), float("nan"), device=DEV)
        dqkv, ws = torch.full_like(q, float("nan")), torch.empty(n * S * heads, device=DEV)
        extra = (B.Dropout(*drop),) if drop else ()
        (B.op_attention_dropout_fwd if drop else B.op_attention_fwd)(q, n, S, heads, dh, True, o, lse, *extra)
        (B.op_attention_dropout_bwd if drop else B.op_attention_bwd)(q, o, lse, g, n, S, heads, dh, True, dqkv, ws, *extra)
        return o, lse, dqkv

    o, lse, dqkv = run(qkv, d_o, Bn, nh)
    assert all(torch.isfinite(t).all() for t in (o, lse, dqkv))
    # (dropout masks count heads over the whole batch: the first sample's alone are the same in a call of its own)
    for b in range(1 if drop else Bn):
        rows = slice(b * S, (b + 1) * S)
        heads = nh if nh * ((S + 127) // 128) <= 256 else 256 // ((S + 127) // 128)
        q = torch.cat([t[rows, :heads * dh] for t in qkv.split(H, 1)], 1).contiguous()
        o1, lse1, dq1 = run(q, d_o[rows, :heads * dh].contiguous(), 1, heads)
        assert torch.equal(o1, o[rows, :heads * dh]) and torch.equal(lse1[0], lse[b, :heads])
        assert torch.equal(dq1, torch.cat([t[rows, :heads * dh] for t in dqkv.split(H, 1)], 1))


@pytest.mark.parametrize("dt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("dh", [64, 128])
def test_attention_with_a_maximum_that_creeps_and_then_jumps(dt, dh):
    """Logits that grow by about two units per 64-key tile, with a jump of thirty for every other query late in
    the row: the forward kernel's reference point for the exponents follows the maximum with a lag, and O and
    the log-sum-exp must not depend on where it stood (the softmax is invariant under the shift)."""
    Bn, S, nh = 1, 1024, 2
    H = nh * dh
    rng = np.random.default_rng(77)
    u = rng.standard_normal(dh); u /= np.linalg.norm(u)
    q = np.tile(u * np.sqrt(dh), (S, 1)) + 0.05 * rng.standard_normal((S, dh))    # q.k / sqrt(dh) = the key's ramp
    ramp = 2.0 * np.arange(S) / 64.0
    k = ramp[:, None] * u[None, :] + 0.05 * rng.standard_normal((S, dh))
    k[700] += 30.0 * u                      # one key far above the ramp ...
    q[0::2] *= 1.0; q[1::2] *= 0.25         # ... by thirty units for even queries, by a quarter of that for odd ones
    v = rng.standard_normal((S, dh))
    qkv = np.zeros((Bn * S, 3 * H))
    for h in range(nh):
        qkv[:, h * dh:(h + 1) * dh] = q
        qkv[:, H + h * dh:H + (h + 1) * dh] = k
        qkv[:, 2 * H + h * dh:2 * H + (h + 1) * dh] = v * (h + 1)
    qkv = syn.round_to_bf16(qkv.astype(np.float32)) if dt == torch.bfloat16 else qkv.astype(np.float32)
    d_o = rnd((Bn * S, H), 78, dt)
    q64 = qkv.astype(np.float64)
    for causal in (False, True):
        o_ref, lse_ref = O.attention_fwd(q64, Bn, S, nh, causal)
        dq_ref = O.attention_bwd(d_o.astype(np.float64), q64, Bn, S, nh, causal)
        tq, tdo = dev(qkv, dt), dev(d_o, dt)
        o = torch.empty(Bn * S, H, dtype=dt, device=DEV)
        lse = torch.empty(Bn, nh, S, dtype=torch.float32, device=DEV)
        B.op_attention_fwd(tq, Bn, S, nh, dh, causal, o, lse)
        tol = TOL[dt] * (2 if dt == torch.bfloat16 else 1)
        assert O.max_rel_err(host(o), o_ref) < tol
        assert np.allclose(host(lse), lse_ref, atol=2e-5 * 40 if dt == torch.float32 else 2e-3 * 40)   # lse reaches ~60
        dqkv = torch.empty_like(tq)
        B.op_attention_bwd(tq, o, lse, tdo, Bn, S, nh, dh, causal, dqkv, ws_for(Bn * S, nh))
        got = host(dqkv)
        for blk in range(3):
            assert O.max_rel_err(got[:, blk * H:(blk + 1) * H], dq_ref[:, blk * H:(blk + 1) * H]) < 2 * tol, (causal, blk)


def test_mfma_issue_probe_reports_a_plausible_rate():
    """The diagnostic behind the roofline discussion: rate = CUs * 4096 flop/clk * clock, so the two numbers it
    returns must agree with each other, and zeros must not run slower than random mantissas."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    zeros = torch.zeros(1 << 16, dtype=torch.bfloat16, device=DEV)
    noise = torch.randint(-2 ** 15, 2 ** 15, (1 << 16,), dtype=torch.int16, device=DEV).view(torch.bfloat16)
    tz, fz = B.probe_mfma(zeros, 20000)
    tn, fn = B.probe_mfma(noise, 20000)
    for t, f in ((tz, fz), (tn, fn)):
        assert 500 < f < 3000
        assert abs(t * 1e12 - cus * 4096 * f * 1e6) <= 0.25 * t * 1e12     # one CU's clock; launch and drain included
    assert tz >= 0.98 * tn
    with pytest.raises(B.DpError):
        B.probe_mfma(zeros[:4], 10)


@pytest.mark.parametrize("mode,M,N,K", [(0, 4096, 4096, 4096), (0, 4096, 4096, 11008), (0, 3072, 1600, 6400),
                                        (1, 4096, 4096, 16384), (1, 1600, 6400, 32768), (1, 4096, 11008, 8192)])
def test_gemm_long_contractions_of_the_wide_configurations(mode, M, N, K):
    """The contraction lengths of C4/C5 (hidden 4096, ffn 11008; weight gradients over 16384 and 32768 tokens) at
    output sizes that take the 256x256 tiles and their five-tile ring, against a float32 reference product (its
    own rounding, ~K * 6e-8 relative, is far below one bf16 rounding of the output)."""
    dt = torch.bfloat16
    a = rnd((M, K), 91, dt, 0.5); b = rnd((K, N), 92, dt, 0.5)
    ref = a @ b                                  # float32 in, float32 out
    ta, tb = (dev(a, dt), dev(np.ascontiguousarray(b.T), dt)) if mode == 0 else (dev(np.ascontiguousarray(a.T), dt), dev(b, dt))
    c = torch.empty(M, N, dtype=dt, device=DEV)
    B.op_gemm(mode, M, N, K, ta, tb, None, None, c)
    got = c.float().cpu().numpy()
    scale = np.abs(ref).max()
    assert np.abs(got - ref).max() <= TOL[dt] * scale
    # every 4096th element exactly as one rounding of the float64 product of that row and column
    rows = np.arange(0, M, 509)[:6]; cols = np.arange(0, N, 613)[:6]
    exact = a[rows].astype(np.float64) @ b[:, cols].astype(np.float64)
    assert np.abs(got[np.ix_(rows, cols)] - exact).max() <= 2.0 ** -8 * np.abs(exact).max() + 1e-6


# The column reductions at the token counts of the wide configurations (C5: 16384 tokens, C4: 32768): above 4096
# (LayerNorm backward) or 8192 rows (the other two) a row block of the two-pass reductions covers more than its
# minimum number of rows, a regime the smaller shapes above never enter.
@pytest.mark.parametrize("rows", [16384, 32768])
@pytest.mark.parametrize("cols", [1600, 4096])
def test_layernorm_backward_over_many_rows(rows, cols):
    dt = torch.bfloat16
    fwd, bwd = O.NORMS["layer"]
    x = syn.round_to_bf16(rnd((rows, cols), 11, dt, 2.0) + 0.5)
    g = syn.round_to_bf16(rnd((cols,), 12, dt) * 0.1 + 1)
    b = rnd((cols,), 13, dt, 0.1)
    dy = rnd((rows, cols), 14, dt)
    dres = rnd((rows, cols), 15, dt)
    x64, g64 = x.astype(np.float64), g.astype(np.float64)
    _, mu, r = fwd(x64, g64, b.astype(np.float64), 1e-5)
    dx_ref, dg_ref, db_ref = bwd(dy.astype(np.float64), x64, mu, r, g64)
    tx, tg, tdy, tres = (dev(a, dt) for a in (x, g, dy, dres))
    stats = torch.from_numpy(np.stack([mu, r], axis=1).astype(np.float32)).to(DEV)
    dx = torch.empty_like(tx); dgo = torch.empty_like(tg); dbo = torch.empty_like(tg); dsum = torch.empty_like(tg)
    B.op_layernorm_bwd(tdy, tx, stats, tg, tres, dx, dgo, dbo, ws_for(rows, cols), dx_colsum=dsum)
    assert O.max_rel_err(host(dx), dx_ref + dres) < TOL[dt]
    assert O.max_rel_err(host(dgo), dg_ref) < TOL[dt] and O.max_rel_err(host(dbo), db_ref) < TOL[dt]
    assert O.max_rel_err(host(dsum), host(dx).sum(axis=0)) < TOL[dt]


@pytest.mark.parametrize("rows", [16384, 32768])
@pytest.mark.parametrize("cols", [1600, 6400])
def test_gelu_backward_and_column_sums_over_many_rows(rows, cols):
    dt = torch.bfloat16
    x = rnd((rows, cols), 21, dt, 2.5)
    dy = rnd((rows, cols), 22, dt)
    tx, tdy = dev(x, dt), dev(dy, dt)
    dx = torch.empty_like(tx)
    db = torch.empty(cols, dtype=dt, device=DEV)
    ws = ws_for(rows, cols)
    B.op_gelu_bwd(tdy, tx, dx, db, ws, 0)
    dx_ref = dy * O.gelu_grad(x.astype(np.float64), "erf")
    assert O.max_rel_err(host(dx), dx_ref) < TOL[dt]
    assert O.max_rel_err(host(db), dx_ref.sum(axis=0)) < TOL[dt]
    out = torch.empty(cols, dtype=dt, device=DEV)
    B.op_colsum(tx, out, ws)
    assert O.max_rel_err(host(out), x.astype(np.float64).sum(axis=0)) < TOL[dt]
