"""GPU parity at the shapes where the kernels' vector maps change: widths around whole 16-byte
vectors, buffers at element alignment, guard elements around every output."""
import numpy as np
import pytest

import oracle
from paper_2103_00959_amd import synth

from gpu_util import (TOL_ALPHA, TOL_F32, alpha_bound_scale, alpha_close, dev, features, graph_to_dev, say, scaled_error,
                      to_f64, tol_for)
from test_gpu_ops import _bwd_inputs, _check_bwd

pytestmark = pytest.mark.gpu

GUARD = 24


@pytest.fixture(scope="module")
def cg():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2103_00959_amd as m
    m.lib()
    return m


def _graph(seed=0, n=700, m=450):
    """Empty rows, rows of one to a few edges, and rows of several hundred (split at group size 40)."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 14, n)
    deg[rng.choice(n, 8, replace=False)] = rng.integers(41, 420, 8)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.concatenate([np.sort(rng.choice(m, d, replace=False)) for d in deg]).astype(np.int32)
    col[:3] = m - 1                      # the last row of X, whose last vector ends the buffer
    val = rng.standard_normal(col.size).astype(np.float32)
    return synth.Graph(rowptr, col, val, n, m)


def _shifted(x, by):
    """A contiguous copy of x whose first element sits `by` elements past an aligned address."""
    import torch
    buf = torch.empty(x.numel() + by, dtype=x.dtype, device=x.device)
    out = buf[by:].view(x.shape)
    out.copy_(x)
    return out


def _guarded(shape, dtype, by):
    """(output view, its whole buffer): GUARD + by elements before it and GUARD after, all 7."""
    import torch
    n = int(np.prod(shape))
    buf = torch.full((n + 2 * GUARD + by,), 7, dtype=dtype, device="cuda")
    return buf[GUARD + by:GUARD + by + n].view(shape), buf


def _untouched(buf, n, by):
    import torch
    assert torch.all(buf[:GUARD + by] == 7) and torch.all(buf[GUARD + by + n:] == 7), "wrote past the output"


def _plans(cg, rp, cl, g, width, heads=0):
    yield None
    for kw in ({"mode": "neighbor_group", "group_size": 40}, {"mode": "neighbor_group", "group_size": 64},
               {"mode": "neighbor_group", "group_size": 40, "col": cl, "n_cols": g.n_cols, "slice_min": 30}):
        p = cg.Plan(rp, g.nnz, max_feat=width, max_heads=heads, **kw)
        try:
            yield p
        finally:
            p.close()


@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 24, 31, 32, 33, 41, 63, 65, 129, 257, 300, 515, 2051])
@pytest.mark.parametrize("xk,yk", [("f32", "f32"), ("bf16", "bf16"), ("f16", "f32")])
def test_spmm_odd_widths_and_alignment(cg, F, xk, yk):
    import torch
    g = _graph(F)
    say(f"spmm F={F} {xk}->{yk}")
    rp, cl, vl = graph_to_dev(g)
    xh, xc, xd = features((g.n_cols, F), 31 + F, xk)
    bias = np.random.default_rng(F).standard_normal(F).astype(np.float32)
    bd = torch.from_numpy(bias).cuda()
    ydt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[yk]
    Yr, Ar = oracle.spmm(g.rowptr, g.col, g.val, xh, x_dtype=xc)
    Mr, _, Er = oracle.gspmm(g.rowptr, g.col, g.val, xh, "max", x_dtype=xc)
    code = {"f32": oracle.F32, "bf16": oracle.BF16, "f16": oracle.F16}[yk]
    Mr = oracle.decode(oracle.round_to(Mr, code), code).reshape(Mr.shape)
    tol = tol_for(xk, yk)
    for by in (0, 1, 3):
        xs = _shifted(xd, by)
        for plan in _plans(cg, rp, cl, g, F):
            out, buf = _guarded((g.n_rows, F), ydt, by)
            cg.spmm(rp, cl, vl, xs, plan=plan, out=out)
            assert scaled_error(out, Yr, Ar) <= tol, (F, xk, by, "sum")
            _untouched(buf, g.n_rows * F, by)
            out, buf = _guarded((g.n_rows, F), ydt, by)
            cg.gspmm(rp, cl, vl, xs, "mean", plan=plan, bias=bd, out=out)
            deg = np.maximum(np.diff(g.rowptr), 1)[:, None]
            assert scaled_error(out, Yr / deg + bias, Ar / deg + np.abs(bias)) <= tol, (F, xk, by, "mean + bias")
            _untouched(buf, g.n_rows * F, by)
            if yk == xk or yk == "f32":
                out, buf = _guarded((g.n_rows, F), ydt, by)
                arg, abuf = _guarded((g.n_rows, F), torch.int32, by)
                cg.gspmm(rp, cl, vl, xs, "max", plan=plan, out=out, arg=arg)
                assert np.array_equal(to_f64(out), Mr), (F, xk, by, "max")
                assert np.array_equal(arg.cpu().numpy(), Er), (F, xk, by, "arg")
                _untouched(buf, g.n_rows * F, by)
                _untouched(abuf, g.n_rows * F, by)


@pytest.mark.parametrize("F", [3, 8, 16, 24, 33, 41, 65, 128])
@pytest.mark.parametrize("xk", ["f32", "bf16"])
@pytest.mark.parametrize("n", [9000, 60000])
def test_spmm_past_the_unit_limits(cg, F, xk, n):
    """The same sums with more units than run a wavefront each (8192 for narrow rows, 55000
    with a plan, 16384 without)."""
    g = _graph(F, n=n, m=3000)
    say(f"spmm n={n} F={F} {xk}")
    rp, cl, vl = graph_to_dev(g)
    xh, xc, xd = features((g.n_cols, F), 11 + F, xk)
    Yr, Ar = oracle.spmm(g.rowptr, g.col, g.val, xh, x_dtype=xc)
    deg = np.maximum(np.diff(g.rowptr), 1)[:, None]
    for plan in _plans(cg, rp, cl, g, F):
        out, buf = _guarded((g.n_rows, F), xd.dtype, 0)
        cg.spmm(rp, cl, vl, xd, plan=plan, out=out)
        assert scaled_error(out, Yr, Ar) <= tol_for(xk, xk), (F, xk, n)
        _untouched(buf, g.n_rows * F, 0)
        out = cg.gspmm(rp, cl, vl, xd, "mean", plan=plan)
        assert scaled_error(out, Yr / deg, Ar / deg) <= tol_for(xk, xk), (F, xk, n, "mean")


# one head of an odd width; heads below a vector; groups of 1, 2, 4 and 8 owner lanes; heads past one
# wavefront (slabs, the last one part full); more heads than lanes a head; a head too wide for the map
HEADS = [(1, 41, "bf16"), (1, 8, "bf16"), (2, 9, "f16"), (3, 17, "bf16"), (1, 5, "bf16"), (2, 3, "f32"), (4, 32, "bf16"),
         (8, 16, "f32"), (8, 51, "bf16"), (6, 128, "bf16"), (5, 200, "f32"), (64, 2, "f32"), (11, 24, "f16"),
         (1, 300, "f32"), (1, 513, "bf16")]


@pytest.mark.parametrize("H,D,xk", HEADS)
def test_head_maps_backward(cg, H, D, xk):
    """sddmm_dot, and the backward on given weights, at the edges of the head-to-lane map."""
    import torch
    g = _graph(H * D)
    W = H * D
    say(f"backward H={H} D={D} {xk}")
    rp, cl, _ = graph_to_dev(g)
    sd, ss, alpha, (xh, xc, xd), (gh, gc, gd) = _bwd_inputs(g, H, D, xk, 300 + W)
    colptr, row_t, _, perm = oracle.csr_to_csc(g.rowptr, g.col, None, g.n_cols)
    cp_d, rt_d, pm_d, sd_d, ss_d, al_d = (dev(a) for a in (colptr, row_t, perm, sd, ss, alpha))
    dot, dab = oracle.sddmm_dot(g.rowptr, g.col, gh.reshape(g.n_rows, W), xh.reshape(g.n_cols, W), H, D, p_dtype=gc,
                                q_dtype=xc)
    ref = oracle.gat_backward(g.rowptr, g.col, sd, ss, alpha, xh.reshape(g.n_cols, W), gh.reshape(g.n_rows, W), H, D,
                              slope=0.2, x_dtype=xc, dy_dtype=gc)
    gt = synth.Graph(colptr, row_t, None, g.n_cols, g.n_rows)
    for by in (0, 1):
        xs, gs = _shifted(xd, by), _shifted(gd, by)
        for plan, plan_t in zip(_plans(cg, rp, cl, g, W, H), _plans(cg, cp_d, rt_d, gt, W, H)):
            out, buf = _guarded((g.nnz, H), torch.float32, by)
            cg.sddmm_dot(rp, cl, gs, xs, plan=plan, out=out)
            assert scaled_error(out, dot, dab) <= TOL_F32, (H, D, by, "dot")
            _untouched(buf, g.nnz * H, by)
            dX, xbuf = _guarded((g.n_cols, H, D), torch.float32, by)
            o = cg.gat_backward(rp, cl, cp_d, rt_d, pm_d, sd_d, ss_d, al_d, xs, gs, 0.2, plan=plan, plan_t=plan_t,
                                out={"dX": dX})
            _check_bwd(o, ref, (H, D, by), alpha)
            _untouched(xbuf, g.n_cols * W, by)


@pytest.mark.parametrize("xk", ["f32", "bf16"])
def test_head_tail_keeps_infinities_apart(cg, xk):
    """A ragged head's masked features: an infinity in one feature of a head gives that head's
    dot products their infinity and leaves its neighbours' finite."""
    import torch
    H, D = 3, 11
    rp, cl = dev(np.array([0, 2], np.int32)), dev(np.array([0, 1], np.int32))
    dt = torch.float32 if xk == "f32" else torch.bfloat16
    P = torch.ones((1, H, D), dtype=dt, device="cuda")
    for d in range(D):
        Q = torch.ones((2, H, D), dtype=dt, device="cuda")
        Q[0, 1, d] = float("inf")
        want = torch.tensor([[D, float("inf"), D], [D, D, D]], dtype=torch.float32, device="cuda")
        assert torch.equal(cg.sddmm_dot(rp, cl, P, Q), want), d


def _alpha_ok(alpha, g, sd, ss):
    ref = oracle.edge_softmax(g.rowptr, g.col, sd, ss, slope=0.2)
    scale = np.asarray(alpha_bound_scale(g.rowptr, g.col, sd, ss)).reshape(ref.shape)
    return alpha_close(alpha, ref, scale) <= TOL_ALPHA


@pytest.mark.parametrize("H,D,xk", HEADS)
def test_head_maps_forward(cg, H, D, xk):
    """The aggregation with and without alpha out, on given weights, with bias and ELU, and
    through row states with the backward that rebuilds the weights, at the same head shapes."""
    import torch
    g = _graph(H * D + 1)
    W = H * D
    say(f"forward H={H} D={D} {xk}")
    rp, cl, _ = graph_to_dev(g)
    sd, ss, alpha, (xh, xc, xd), (gh, gc, gd) = _bwd_inputs(g, H, D, xk, 700 + W)
    sd_d, ss_d, al_d = dev(sd), dev(ss), dev(alpha)
    colptr, row_t, _, perm = oracle.csr_to_csc(g.rowptr, g.col, None, g.n_cols)
    cp_d, rt_d, pm_d = dev(colptr), dev(row_t), dev(perm)
    gt = synth.Graph(colptr, row_t, None, g.n_cols, g.n_rows)
    Yr, Ar = oracle.gat(g.rowptr, g.col, sd, ss, xh.reshape(g.n_cols, W), H, D, slope=0.2, x_dtype=xc)
    bias = np.random.default_rng(W).standard_normal(W).astype(np.float32)
    Yb = Yr + bias
    Yb = np.where(Yb > 0, Yb, np.expm1(np.minimum(Yb, 0.0)))
    tol = tol_for("f32")
    for by in (0, 1):
        xs, gs = _shifted(xd, by), _shifted(gd, by)
        for plan, plan_t in zip(_plans(cg, rp, cl, g, W, H), _plans(cg, cp_d, rt_d, gt, W, H)):
            Y, buf = _guarded((g.n_rows, H, D), torch.float32, by)
            Y2, buf2 = _guarded((g.n_rows, H, D), torch.float32, by)
            al, abuf = _guarded((g.nnz, H), torch.float32, 0)
            cg.gat_aggregate(rp, cl, sd_d, ss_d, xs, 0.2, plan=plan, out=Y)
            cg.gat_aggregate(rp, cl, sd_d, ss_d, xs, 0.2, plan=plan, out=Y2, alpha_out=al)
            assert scaled_error(Y.reshape(Yr.shape), Yr, Ar) <= tol, (H, D, by)
            assert torch.equal(Y, Y2) and _alpha_ok(al, g, sd, ss), (H, D, by)
            for b in (buf, buf2):
                _untouched(b, g.n_rows * W, by)
            _untouched(abuf, g.nnz * H, 0)
            Yg = cg.gat_aggregate(rp, cl, None, None, xs, 0.2, alpha_in=al_d, plan=plan, out_dtype=torch.float32)
            assert scaled_error(Yg.reshape(Yr.shape), Yr, Ar) <= tol, (H, D, by, "given weights")
            Ye = cg.gat_aggregate(rp, cl, sd_d, ss_d, xs, 0.2, plan=plan, out_dtype=torch.float32, bias=dev(bias),
                                  act="elu")
            assert scaled_error(Ye.reshape(Yr.shape), Yb, Ar + np.abs(bias)) <= tol, (H, D, by, "elu")
            Ys, st = cg.gat_aggregate_stats(rp, cl, sd_d, xs, s_src=ss_d, negative_slope=0.2, plan=plan,
                                            out_dtype=torch.float32)
            assert torch.equal(Y, Ys), (H, D, by, "stats")
            args = (rp, cl, cp_d, rt_d, pm_d, sd_d, ss_d)
            a = cg.gat_backward(*args, al, xs, gs, 0.2, plan=plan, plan_t=plan_t, dx_dtype=torch.float32)
            b = cg.gat_backward(*args, None, xs, gs, 0.2, plan=plan, plan_t=plan_t, dx_dtype=torch.float32,
                                row_stats=st)
            for k in a:
                assert torch.equal(a[k], b[k]), (H, D, by, k)


@pytest.mark.parametrize("H,D,xk", [(4, 32, "bf16"), (8, 16, "f32"), (1, 8, "f16"), (3, 16, "bf16"), (2, 128, "bf16"),
                                    (5, 4, "f32"), (1, 512, "bf16"), (8, 64, "f16"), (2, 8, "f32")])
def test_head_maps_projected(cg, H, D, xk):
    """Projected source scores over every number of lanes that share a batch's scores, against
    the aggregation on the scores in fp64 (bound: the aggregation's, plus each score's rounding
    2 (D 2^-24 max sum|x a| + 2^-24 max|s|))."""
    import torch
    g = _graph(H * D + 2)
    W = H * D
    say(f"projected H={H} D={D} {xk}")
    rp, cl, _ = graph_to_dev(g)
    xh, xc, xd = features((g.n_cols, H, D), 900 + W, xk)
    rng = np.random.default_rng(W)
    a = (rng.standard_normal((H, D)) / np.sqrt(D)).astype(np.float32)
    sd = rng.standard_normal((g.n_rows, H)).astype(np.float32)
    x64 = oracle.decode(xh, xc).reshape(g.n_cols, H, D)
    s64 = (x64 * a.astype(np.float64)).sum(-1)
    ss = s64.astype(np.float32)
    Yr, Ar = oracle.gat(g.rowptr, g.col, sd, ss, xh.reshape(g.n_cols, W), H, D, slope=0.2, x_dtype=xc)
    extra = 2 * (D * 2.0 ** -24 * (np.abs(x64) * np.abs(a)).sum(-1).max() + 2.0 ** -24 * np.abs(s64).max())
    for plan in _plans(cg, rp, cl, g, W, H):
        Y, buf = _guarded((g.n_rows, H, D), torch.float32, 0)
        cg.gat_aggregate_proj(rp, cl, dev(sd), dev(a), xd, 0.2, plan=plan, out=Y)
        assert scaled_error(Y.reshape(Yr.shape), Yr, Ar) <= TOL_F32 + extra, (H, D)
        _untouched(buf, g.n_rows * W, 0)


@pytest.mark.parametrize("F,G", [(64, 64), (100, 64), (1, 64), (63, 128), (65, 64), (129, 128), (256, 256), (300, 256),
                                 (512, 512), (515, 512), (192, 192), (320, 64), (1030, 512), (1024, 1024), (700, 1024)])
@pytest.mark.parametrize("xk", ["f32", "bf16", "f16"])
def test_codec_widths_and_alignment(cg, F, G, xk):
    """Every code width on whole, ragged, unaligned and odd-sized groups: codes, minima, steps and
    decoded values bit for bit, nothing written past them."""
    import torch
    n = 37
    say(f"codec F={F} G={G} {xk}")
    xh, xc, xd = features((n, F), 50 + F, xk)
    for by in (0, 1):
        xs = _shifted(xd, by)
        for bits in range(1, 9):
            seed = 0x123456789ABC + bits + F
            words, nst = cg.act_codec_size(n, F, bits, G)
            codes, cbuf = _guarded((words,), torch.int64, 0)
            stats, sbuf = _guarded((nst,), torch.float32, 0)
            cg.act_compress(xs, bits, G, seed, codes=codes, stats=stats)
            c_ref, s_ref = oracle.act_compress(xh, bits, G, seed, a_dtype=xc)
            assert np.array_equal(codes.cpu().numpy().view(np.uint64), c_ref), (F, G, bits, by)
            assert np.array_equal(stats.cpu().numpy().view(np.uint32), s_ref.view(np.uint32)), (F, G, bits, by)
            out, obuf = _guarded((n, F), torch.float32, by)
            cg.act_decompress(codes, stats, n, F, bits, G, out=out)
            y_ref = oracle.act_decompress(c_ref, s_ref, n, F, bits, G)
            assert np.array_equal(out.cpu().numpy().view(np.uint32), y_ref.view(np.uint32)), (F, G, bits, by)
            o16, o16buf = _guarded((n, F), torch.bfloat16, by)
            cg.act_decompress(codes, stats, n, F, bits, G, out=o16)
            assert np.array_equal(o16.cpu().view(torch.int16).numpy().view(np.uint16),
                                  oracle.round_to(y_ref.astype(np.float64), oracle.BF16)), (F, G, bits, by)
            for b, m, k in ((cbuf, words, 0), (sbuf, nst, 0), (obuf, n * F, by), (o16buf, n * F, by)):
                _untouched(b, m, k)


@pytest.mark.parametrize("k,m", [(8, 1), (9, 7), (15, 41), (16, 32), (17, 33), (47, 129), (48, 129), (63, 64), (64, 65), (65, 128),
                                 (129, 300), (602, 128), (623, 127), (624, 97), (640, 97), (1160, 32), (1433, 16)])
@pytest.mark.parametrize("n", [2047, 2048, 2081])
@pytest.mark.parametrize("xk,yk", [("bf16", "f32"), ("f16", "f16")])
def test_linear_streamed_shapes(cg, k, m, n, xk, yk):
    """The dense layer around the streaming kernel's limits: slots and chunks of k, column tiles,
    ragged row tiles, unaligned operands and outputs."""
    import torch
    say(f"linear n={n} k={k} m={m} {xk}->{yk}")
    xh, xc, xd = features((n, k), 7 + k, xk)
    wh, wc, wd = features((m, k), 8 + m, xk)
    bias = np.random.default_rng(m).standard_normal(m).astype(np.float32)
    ydt = torch.float32 if yk == "f32" else torch.float16
    x64, w64 = oracle.decode(xh, xc).reshape(n, k), oracle.decode(wh, wc).reshape(m, k)
    Yr = np.maximum(x64 @ w64.T + bias, 0.0)
    Ar = np.abs(x64) @ np.abs(w64).T + np.abs(bias)
    for by in (0, 1):
        out, buf = _guarded((n, m), ydt, by)
        cg.linear(_shifted(xd, by), _shifted(wd, by), dev(bias), act="relu", out=out)
        # fp32 accumulation of exact products: k 2^-24 of the terms' sum at most; fp16 also rounds the result
        assert scaled_error(out, Yr, Ar) <= k * 2.0 ** -24 + (0 if yk == "f32" else 1e-6), (k, m, n, by)
        _untouched(buf, n * m, by)


@pytest.mark.parametrize("n,k,m", [(2048, 48, 32768), (2048, 48, 32769), (2081, 620, 33000), (4096, 512, 40000),
                                   (30001, 48, 300), (30001, 602, 300), (70001, 64, 129),
                                   (30001, 24, 300), (2081, 9, 401), (2048, 47, 1025), (2048, 8, 129)])
def test_linear_grids(cg, n, k, m):
    """The streaming kernel's grid: column blocks as many as the resident workgroups and more, three
    and two of them over more row tiles than one round takes."""
    import torch
    say(f"linear n={n} k={k} m={m}")
    g = torch.Generator(device="cuda")
    g.manual_seed(k + m)
    x = torch.randn((n, k), device="cuda", generator=g).to(torch.bfloat16)
    w = torch.randn((m, k), device="cuda", generator=g).to(torch.bfloat16)
    y = cg.linear(x, w, out_dtype=torch.float32)
    for r0 in range(0, n, 4096):
        rows = x[r0:r0 + 4096].double()
        bound = rows.abs() @ w.double().abs().T * (k * 2.0 ** -24)   # fp32 sums of exact products
        assert torch.all((y[r0:r0 + 4096].double() - rows @ w.double().T).abs() <= bound), (n, k, m, r0)


@pytest.mark.parametrize("n", [39000, 42000])
@pytest.mark.parametrize("mode", ["auto", "neighbor_group", "row_split"])
@pytest.mark.parametrize("F,xk", [(41, "bf16"), (64, "bf16"), (33, "f32")])
def test_spmm_small_groups(cg, n, mode, F, xk):
    """Plans cut into groups of 32 edges around the size (2^18 edges) from where those that chose
    their mode stop running a wavefront a unit; those that asked for it never do."""
    import torch
    g = _graph(F, n=n, m=3000)
    assert (g.nnz > 1 << 18) == (n == 42000)
    say(f"spmm groups of 32 n={n} {mode} F={F} {xk}")
    rp, cl, vl = graph_to_dev(g)
    xh, xc, xd = features((g.n_cols, F), 17 + F, xk)
    Yr, Ar = oracle.spmm(g.rowptr, g.col, g.val, xh, x_dtype=xc)
    plan = cg.Plan(rp, g.nnz, max_feat=F, mode=mode, group_size=32)
    try:
        Y = cg.spmm(rp, cl, vl, xd, plan=plan, out_dtype=torch.float32)
        assert scaled_error(Y, Yr, Ar) <= tol_for("f32"), (n, mode, F, xk)
    finally:
        plan.close()


@pytest.mark.parametrize("n", [118000, 124000])
@pytest.mark.parametrize("F,xk", [(33, "bf16"), (65, "bf16"), (127, "f16"), (33, "f32"), (63, "f32")])
def test_ragged_rows_past_the_element_lanes(cg, n, F, xk):
    """Max (with its edge ids), add and the sums at widths of no whole vector around the size
    (3 2^18 edges) from where max and add of a plan stop running an element per lane."""
    import torch
    g = _graph(F, n=n, m=3000)
    assert (g.nnz >= 3 << 18) == (n == 124000)
    say(f"max and add n={n} F={F} {xk}")
    rp, cl, vl = graph_to_dev(g)
    xh, xc, xd = features((g.n_cols, F), 5 + F, xk)
    Mr, _, Er = oracle.gspmm(g.rowptr, g.col, g.val, xh, "max", x_dtype=xc)
    Sr, Ar, _ = oracle.gspmm(g.rowptr, g.col, g.val, xh, "sum", compute="add", x_dtype=xc)
    Yr, Yar = oracle.spmm(g.rowptr, g.col, g.val, xh, x_dtype=xc)
    for kw in (None, {}, {"mode": "row_split"}, {"mode": "neighbor_group", "group_size": 40}):
        plan = None if kw is None else cg.Plan(rp, g.nnz, max_feat=F, **kw)
        try:
            top, arg = cg.gspmm(rp, cl, vl, xd, "max", plan=plan, out_dtype=torch.float32, return_arg=True)
            assert np.array_equal(to_f64(top), oracle.decode(oracle.round_to(Mr, oracle.F32), oracle.F32).reshape(Mr.shape))
            assert np.array_equal(arg.cpu().numpy(), Er)
            add = cg.gspmm(rp, cl, vl, xd, "sum", compute="add", plan=plan, out_dtype=torch.float32)
            assert scaled_error(add, Sr, Ar) <= TOL_F32, (n, F, xk, kw)
            Y = cg.spmm(rp, cl, vl, xd, plan=plan, out_dtype=torch.float32)
            assert scaled_error(Y, Yr, Yar) <= TOL_F32, (n, F, xk, kw)
        finally:
            if plan is not None:
                plan.close()


@pytest.mark.parametrize("H,D,xk", [(3, 35, "bf16"), (3, 40, "bf16"), (3, 18, "f32"), (5, 20, "bf16"), (16, 3, "f32"),
                                    (12, 3, "bf16"), (6, 10, "f32")])
def test_head_maps_of_odd_lane_counts(cg, H, D, xk):
    """Heads of vectors on a lane count that is no power of two, and heads whose lanes are padded to
    one where scores are shared but not on given weights."""
    test_head_maps_forward(cg, H, D, xk)
    test_head_maps_backward(cg, H, D, xk)


@pytest.mark.parametrize("H,D,xk", [(1, 41, "bf16"), (1, 5, "f32"), (2, 3, "bf16"), (4, 16, "bf16"), (8, 16, "f32"),
                                    (8, 8, "bf16"), (3, 35, "bf16"), (4, 64, "bf16"), (8, 51, "f32")])
def test_masked_sources_open_a_row(cg, H, D, xk):
    """Sources masked out by a score of -inf weigh nothing, however many of them open a row or a
    group: rows of 1 to 40 edges whose first edges but one, two or five are masked."""
    import torch
    m = 64
    deg = np.repeat(np.arange(1, 41), 3)
    keep = np.minimum(np.tile([1, 2, 5], 40), deg)
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    col = np.concatenate([np.concatenate([np.arange(d - k), 40 + np.arange(k)]) for d, k in zip(deg, keep)]).astype(np.int32)
    g = synth.Graph(rowptr, col, None, deg.size, m)
    say(f"masked sources H={H} D={D} {xk}")
    rng = np.random.default_rng(H * D)
    sd, ss = rng.standard_normal((g.n_rows, H)).astype(np.float32), rng.standard_normal((m, H)).astype(np.float32)
    ss[:40] = -np.inf
    xh, xc, xd = features((m, H, D), 60 + D, xk)
    Yr, Ar = oracle.gat(rowptr, col, sd, ss, xh.reshape(m, H * D), H, D, slope=0.2, x_dtype=xc)
    rp, cl = dev(rowptr), dev(col)
    for plan in _plans(cg, rp, cl, g, H * D, H):
        Y = cg.gat_aggregate(rp, cl, dev(sd), dev(ss), xd, 0.2, plan=plan, out_dtype=torch.float32)
        assert scaled_error(Y.reshape(Yr.shape), Yr, Ar) <= TOL_F32, (H, D, xk)
    for G in (3, 16):
        plan = cg.Plan(rp, g.nnz, max_feat=H * D, max_heads=H, mode="neighbor_group", group_size=G)
        try:
            Y = cg.gat_aggregate(rp, cl, dev(sd), dev(ss), xd, 0.2, plan=plan, out_dtype=torch.float32)
            assert scaled_error(Y.reshape(Yr.shape), Yr, Ar) <= TOL_F32, (H, D, xk, G)
        finally:
            plan.close()


@pytest.mark.parametrize("n", [118000, 124000])
@pytest.mark.parametrize("H,D,xk", [(1, 3, "bf16"), (2, 5, "f32"), (4, 7, "bf16"), (5, 7, "f16"), (2, 9, "f32")])
def test_dots_of_short_heads(cg, n, H, D, xk):
    """Dot products of short ragged heads around the size (3 2^18 edges) from where a plan's run
    the feature-parallel kernel, and heads of one too many or one too wide for the other."""
    import torch
    g = _graph(D, n=n, m=3000)
    assert (g.nnz >= 3 << 18) == (n == 124000)
    say(f"dot n={n} H={H} D={D} {xk}")
    rp, cl, _ = graph_to_dev(g)
    xh, xc, xd = features((g.n_cols, H, D), 70 + D, xk)
    ph, pc, pd = features((g.n_rows, H, D), 71 + D, xk)
    ref, ab = oracle.sddmm_dot(g.rowptr, g.col, ph.reshape(g.n_rows, H * D), xh.reshape(g.n_cols, H * D), H, D,
                               p_dtype=pc, q_dtype=xc)
    for kw in (None, {}, {"mode": "neighbor_group", "group_size": 40}):
        plan = None if kw is None else cg.Plan(rp, g.nnz, max_feat=H * D, max_heads=H, **kw)
        try:
            out, buf = _guarded((g.nnz, H), torch.float32, 0)
            cg.sddmm_dot(rp, cl, pd, xd, plan=plan, out=out)
            assert scaled_error(out, ref, ab) <= TOL_F32, (n, H, D, xk, kw)
            _untouched(buf, g.nnz * H, 0)
        finally:
            if plan is not None:
                plan.close()


def test_bf16_rounding_of_every_class(cg):
    """fp32 to bf16 in an epilogue: every upper half of an fp32 pattern with lower halves below,
    at and above the tie, so all exponents, subnormals, overflow to infinity, infinities and NaN."""
    import torch
    n, low = 1 << 16, np.array([0x0000, 0x0001, 0x7fff, 0x8000, 0x8001, 0xffff], np.uint32)
    bits = (np.arange(n, dtype=np.uint32)[:, None] << 16) | low[None, :]
    x = bits.view(np.float32)
    rp, cl = dev(np.arange(n + 1, dtype=np.int32)), dev(np.arange(n, dtype=np.int32))
    Y = cg.spmm(rp, cl, None, dev(x), out_dtype=torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
    nan = np.isnan(x)
    with np.errstate(over="ignore"):
        want = oracle.round_to(np.where(nan, 0.0, x).astype(np.float64) + 0.0, oracle.BF16).reshape(x.shape)
    assert np.array_equal(Y[~nan], want[~nan])
    assert np.all((Y[nan] & 0x7fc0) == 0x7fc0), "a NaN stays a quiet NaN"


@pytest.mark.parametrize("k", [9, 11, 15, 67])
@pytest.mark.parametrize("xk", ["bf16", "f16"])
def test_linear_tail_keeps_infinities_apart(cg, k, xk):
    """The streaming kernel's overlapped last slot: an infinity in any feature of one row, or of one
    output's weights, gives that row or output its infinity and leaves the others finite."""
    import torch
    n, m = 2080, 41
    dt = torch.bfloat16 if xk == "bf16" else torch.float16
    for d in range(k):
        X, W = torch.ones((n, k), dtype=dt, device="cuda"), torch.ones((m, k), dtype=dt, device="cuda")
        X[7, d] = X[n - 1, d] = W[3, d] = W[m - 1, d] = float("inf")
        want = torch.full((n, m), float(k), device="cuda")
        want[[7, n - 1], :] = float("inf")
        want[:, [3, m - 1]] = float("inf")
        assert torch.equal(cg.linear(X, W, out_dtype=torch.float32), want), d


@pytest.mark.timeout(300)
@pytest.mark.parametrize("n,H,D,xk", [(1_050_000, 7, 293, "bf16"), (40_000_000, 1, 54, "bf16"), (40_000_000, 3, 9, "f32")])
def test_ragged_tables_beyond_4gib(cg, n, H, D, xk):
    """Widths and heads of no whole vector in tables past the 32-bit offsets of the buffer gathers:
    the sums, max, the aggregation with its weights, dot products and the backward against fp64
    over the edges, which reach the tables' last rows."""
    import torch
    W = H * D
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[xk]
    say(f"ragged tables: {n} x {H} x {D} {xk}")
    assert n * W * (4 if xk == "f32" else 2) > 0xffffff00
    rng = np.random.default_rng(W)
    deg = np.zeros(n, np.int64)
    rows = np.unique(np.concatenate([[0, n - 1, n - 2], rng.choice(n, 200)]))
    deg[rows] = rng.integers(1, 30, rows.size)
    deg[n - 2] = 700
    rowptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    nnz = int(rowptr[-1])
    cols = np.unique(np.concatenate([[0, n - 1, n - 2], rng.choice(n, 900)]))
    col = np.concatenate([np.sort(rng.choice(cols, int(deg[r]), replace=False)) for r in rows]).astype(np.int32)
    g = torch.Generator(device="cuda")
    g.manual_seed(W)
    X, G = (torch.randn((n, H, D), dtype=dt, device="cuda", generator=g) for _ in range(2))
    sd, ss = (torch.randn((n, H), device="cuda", generator=g) for _ in range(2))
    val = torch.randn(nnz, device="cuda", generator=g)
    rp, cl = dev(rowptr), dev(col)
    ri, ci = torch.from_numpy(np.repeat(rows, deg[rows])).cuda(), cl.long()
    at = torch.from_numpy(rows).cuda()
    seg = torch.from_numpy(np.repeat(np.arange(rows.size), deg[rows])).cuda()

    def over_rows(t):                                  # sums of per-edge values over the rows with edges
        return torch.zeros((rows.size,) + tuple(t.shape[1:]), dtype=torch.float64, device="cuda").index_add_(0, seg, t)

    x, p = X[ci].double(), G[ri].double()              # [nnz, H, D]
    e = torch.nn.functional.leaky_relu((sd[ri] + ss[ci]).double(), 0.2)
    top = torch.full((rows.size, H), -float("inf"), dtype=torch.float64, device="cuda")
    top = top.index_reduce_(0, seg, e, "amax")
    al = torch.exp(e - top[seg])
    al = al / over_rows(al)[seg]
    msg = val.double()[:, None, None] * x
    da, dab = (p * x).sum(-1), (p * x).abs().sum(-1)
    c, cab = over_rows(al * da), over_rows(al * dab)
    f = torch.where((sd[ri] + ss[ci]) > 0, 1.0, 0.2).double()
    ds, dsab = f * al * (da - c[seg]), f * al * (dab + cab[seg])
    colptr, row_t, _, perm = cg.csr_to_csc(rp, cl, None, n)

    def close(got, want, scale, what, tol=TOL_F32):
        err = ((got.double() - want).abs() / scale.clamp_min(1e-30)).max().item()
        assert err <= tol, (n, H, D, xk, what, err)

    for kw in (None, {"mode": "neighbor_group", "group_size": 64}):
        plan = None if kw is None else cg.Plan(rp, nnz, max_feat=W, max_heads=H, **kw)
        try:
            Y = cg.spmm(rp, cl, val, X.view(n, W), plan=plan, out_dtype=torch.float32)
            close(Y[at], over_rows(msg).view(-1, W), over_rows(msg.abs()).view(-1, W), "sum")
            del Y
            M, A = cg.gspmm(rp, cl, val, X.view(n, W), "max", plan=plan, out_dtype=torch.float32, return_arg=True)
            a = A[at].long()
            assert torch.all(seg[a] == torch.arange(rows.size, device="cuda")[:, None])
            picked = (val[a] * X.view(n, W)[ci[a], torch.arange(W, device="cuda")].float())
            assert torch.equal(M[at], picked)
            best = torch.full((rows.size, W), -float("inf"), device="cuda")
            best.index_reduce_(0, seg, (val[:, None] * X.view(n, W)[ci].float()), "amax")
            assert torch.equal(M[at], best)
            del M, A
            Y, alpha = cg.gat_aggregate(rp, cl, sd, ss, X, 0.2, return_alpha=True, plan=plan, out_dtype=torch.float32)
            want = al[:, :, None] * x
            close(Y[at].view(-1, W), over_rows(want).view(-1, W), over_rows(want.abs()).view(-1, W), "gat")
            close(alpha, al, al, "alpha")
            del Y
            close(cg.sddmm_dot(rp, cl, G, X, plan=plan), da, dab, "dot")
            o = cg.gat_backward(rp, cl, colptr, row_t, perm, sd, ss, alpha, X, G, 0.2, plan=plan)
            close(o["dscore"], ds, dsab, "dscore", 2 * TOL_F32)      # (on the aggregation's own alpha)
            close(o["ds_dst"][at], over_rows(ds), over_rows(dsab), "ds_dst", 2 * TOL_F32)
            used = torch.unique(ci)
            slot = torch.searchsorted(used, ci)
            wx = torch.zeros((used.numel(), H, D), dtype=torch.float64, device="cuda")
            dx = wx.clone().index_add_(0, slot, al[:, :, None] * p)
            dxab = wx.index_add_(0, slot, (al[:, :, None] * p).abs())
            # (dX in X's format: its half unit in the last place beside the sums' error)
            close(o["dX"][used].double(), dx, dxab, "dX", 2 * TOL_F32 + (2.0 ** -8 if xk == "bf16" else 0))
            del o, alpha
        finally:
            if plan is not None:
                plan.close()
    del X, G
    torch.cuda.empty_cache()
