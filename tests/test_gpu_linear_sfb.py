"""GPU parity: sharded linear fwd / bwd and SFB rebuild against the CPU oracle, through the C ABI.

Tolerances (max|err| / max|ref| per output tensor): 1e-5 for fp32, 2e-2 for bf16 inputs with fp32
accumulation; shard index ranges are compared bit-exactly.
"""
import numpy as np
import pytest

import hapgen
from hapgen import TensorId as T
from oracle import linear as olin, sfb as osfb, lp as olp, rounding as ornd

pytestmark = pytest.mark.gpu

from gpu_util import gen, empty, host, check, relerr, torch_mod  # noqa: E402


@pytest.fixture(scope="module")
def hap():
    import paper_2401_05965_amd as h
    return h


DT = {"bf16": 1, "f32": 0}


def run_linear_case(hap, dtype, tokens, in_f, out_f, mode, offsets, act, bias, full, dw_dtype=None, pad=0, seed=7):
    """Runs every shard of one layer on the GPU and checks each against the oracle.  Returns max error."""
    torch = torch_mod()
    dw_dtype = dw_dtype or dtype
    if mode == olin.REDUCTION:
        bias = False          # bias is applied once, after the all-reduce of the partials
    Xh, Xd = gen(seed, T.X, (tokens, in_f), 1.0, dtype)
    Wh, Wd = gen(seed, T.W, (in_f, out_f), 0.05, dtype)
    bh, bd = gen(seed, T.BIAS, (out_f,), 0.5, dtype) if bias else (None, None)
    dYh, dYd = gen(seed, T.DY, (tokens, out_f), 1.0, dtype)
    m = len(offsets) - 1
    worst = 0.0
    Yfull, prefull = olin.linear_fwd(Xh, Wh, bh, act)
    dXsum = np.zeros_like(Xh); dWsum = np.zeros_like(Wh); dbsum = np.zeros(out_f)
    Psum = np.zeros_like(Yfull)
    for j in range(m):
        lo, hi = offsets[j], offsets[j + 1]
        n = hi - lo
        Yo, preo = olin.sharded_linear_fwd(mode, offsets, j, Xh, Wh, bh, act)
        # the oracle's backward takes the full-precision pre-activation; the device uses what it saved
        dXo, dWo, dbo = olin.sharded_linear_bwd(mode, offsets, j, Xh, Wh, prefull if mode != olin.REDUCTION else None, dYh, act)
        if full:
            ldx, ldw, ldy = in_f, out_f, out_f
            Xj, Wj, bj, dYj = Xd, Wd, bd, dYd
            Yj = empty((tokens, out_f), dtype, 0); Pj = empty((tokens, out_f), dtype, 0) if act else None
            dXj = empty((tokens, in_f), dtype, 0); dWj = empty((in_f, out_f), dw_dtype, 0); dbj = empty((out_f,), "f32", 0)
        else:
            # compact slices with padded leading dimensions (pad extra columns filled with NaN poison)
            def compact(t, rows, cols, fill=float("nan")):
                buf = empty((t.shape[0] if rows is None else rows.stop - rows.start, (cols.stop - cols.start if cols else t.shape[1]) + pad), dtype, fill)
                src = t[rows if rows is not None else slice(None), cols if cols is not None else slice(None)]
                buf[:, :src.shape[1]] = src
                return buf
            r = slice(lo, hi)
            if mode == olin.BATCH:
                Xj, Wj, bj, dYj = compact(Xd, r, None), compact(Wd, None, None), bd, compact(dYd, r, None)
                shapeY, shapeX, shapeW = (n, out_f), (n, in_f), (in_f, out_f)
            elif mode == olin.FEATURE:
                Xj, Wj, dYj = compact(Xd, None, None), compact(Wd, None, r), compact(dYd, None, r)
                bj = bd[lo:hi].clone() if bias else None
                shapeY, shapeX, shapeW = (tokens, n), (tokens, in_f), (in_f, n)
            elif mode == olin.REDUCTION:
                Xj, Wj, bj, dYj = compact(Xd, None, r), compact(Wd, r, None), None, compact(dYd, None, None)
                shapeY, shapeX, shapeW = (tokens, out_f), (tokens, n), (n, out_f)
            else:
                Xj, Wj, bj, dYj = compact(Xd, None, None), compact(Wd, None, None), bd, compact(dYd, None, None)
                shapeY, shapeX, shapeW = (tokens, out_f), (tokens, in_f), (in_f, out_f)
            ldx, ldw, ldy = shapeX[1] + pad, shapeW[1] + pad, shapeY[1] + pad
            Yj = empty((shapeY[0], ldy), dtype, 0); Pj = empty((shapeY[0], ldy), dtype, 0) if act else None
            dXj = empty((shapeX[0], ldx), dtype, 0); dWj = empty((shapeW[0], ldw), dw_dtype, 0)
            dbj = empty((shapeY[1],), "f32", 0)
        desc = hap.LinearDesc(tokens, in_f, out_f, mode, offsets, DT[dtype], act=int(act), has_bias=bias and mode != olin.REDUCTION,
                              ldx=ldx, ldw=ldw, ldy=ldy, operands_are_full=full)
        ws = empty((max(hap.hap_linear_bwd_workspace(desc, j), 16),), "u8")
        hap.hap_sharded_linear_fwd(desc, j, Xj, Wj, bj if mode != olin.REDUCTION else None, Yj, Pj, None)
        want_db = mode != olin.REDUCTION
        hap.hap_sharded_linear_bwd(desc, j, Xj, Wj, Pj, dYj, dXj, dWj, DT[dw_dtype], dbj if want_db else None, ws)
        Yg, dXg, dWg, dbg = host(Yj), host(dXj), host(dWj), host(dbj)
        # carve the device's slice out of what came back
        if full:
            if mode == olin.BATCH:
                Ys, dXs, dWs, dbs = Yg[lo:hi], dXg[lo:hi], dWg, dbg
                assert not Yg[:lo].any() and not Yg[hi:].any(), "rows outside the shard were written"
            elif mode == olin.FEATURE:
                Ys, dXs, dWs, dbs = Yg[:, lo:hi], dXg, dWg[:, lo:hi], dbg[lo:hi]
                assert not Yg[:, :lo].any() and not Yg[:, hi:].any(), "columns outside the shard were written"
                assert not dWg[:, :lo].any() and not dWg[:, hi:].any()
            elif mode == olin.REDUCTION:
                Ys, dXs, dWs, dbs = Yg, dXg[:, lo:hi], dWg[lo:hi], None
                assert not dXg[:, :lo].any() and not dXg[:, hi:].any()
                assert not dWg[:lo].any() and not dWg[hi:].any()
            else:
                Ys, dXs, dWs, dbs = Yg, dXg, dWg, dbg
        else:
            Ys, dXs, dWs = Yg[:, :shapeY[1]], dXg[:, :shapeX[1]], dWg[:, :shapeW[1]]
            dbs = dbg if want_db else None
        if n == 0 and mode in (olin.BATCH, olin.FEATURE):
            assert Ys.size == 0 or mode == olin.FEATURE
        tag = f"{dtype} mode{mode} shard{j} full{int(full)}"
        worst = max(worst, check(tag + " Y", Ys, Yo, dtype), check(tag + " dX", dXs, dXo, dtype), check(tag + " dW", dWs, dWo, dw_dtype if dw_dtype == "bf16" else dtype))
        if want_db:
            worst = max(worst, check(tag + " db", dbs, dbo, dtype))
        if mode == olin.REDUCTION:
            Psum += Ys
        if mode == olin.FEATURE:
            dXsum += dXs
        if mode == olin.BATCH:
            dWsum += dWs; dbsum += dbs
    # the rules of Fig. "semantics": partials sum to the unsharded result
    _, dWfull, dbfull = olin.linear_bwd(Xh, Wh, prefull, dYh, act)
    dXfull = olin.linear_bwd(Xh, Wh, prefull, dYh, act)[0]
    big = 4e-2 if dtype == "bf16" else 1e-5
    if mode == olin.REDUCTION:
        assert relerr(Psum, Yfull) <= big
    if mode == olin.FEATURE:
        assert relerr(dXsum, dXfull) <= big
    if mode == olin.BATCH:
        assert relerr(dWsum, dWfull) <= big and relerr(dbsum, dbfull) <= big
    return worst


def test_cfg1_fc_fp32_two_devices(hap):
    """Single fully-connected layer, fp32, batch rows split by the LP ratios of speeds (1, 0.67)."""
    w = hapgen.WORKLOADS["cfg1_fc_f32"]
    d = w.dims
    ratios, _ = hap.hap_shard_ratios(w.speeds, [(1.0, 0, 0, 0)])
    oratios, _ = olp.shard_ratios(w.speeds, [(1.0, 0, 0, 0)])
    assert np.allclose(ratios, oratios, atol=1e-12)
    sizes, offs = hap.hap_round_shards(ratios, d["tokens"])
    osizes, ooffs = ornd.round_shards(oratios, d["tokens"])
    assert sizes == osizes == [38, 26] and offs == ooffs
    # the workload's own scales: X ~ N(0,1), W ~ N(0,0.02), dY ~ N(0,1); seed 0
    torch = torch_mod()
    Xh, Xd = gen(0, T.X, (64, 1024), 1.0, "f32"); Wh, Wd = gen(0, T.W, (1024, 1024), 0.02, "f32"); dYh, dYd = gen(0, T.DY, (64, 1024), 1.0, "f32")
    desc = hap.LinearDesc(64, 1024, 1024, hap.SHARD_BATCH, offs, hap.F32)
    Y = empty((64, 1024), "f32", 0); dX = empty((64, 1024), "f32", 0)
    Xs, dYs = [], []
    for j in range(2):
        dW = empty((1024, 1024), "f32", 0)
        hap.hap_sharded_linear_fwd(desc, j, Xd, Wd, None, Y, None)
        hap.hap_sharded_linear_bwd(desc, j, Xd, Wd, None, dYd, dX, dW, hap.F32, None)
        _, dWo, _ = olin.sharded_linear_bwd(olin.BATCH, offs, j, Xh, Wh, None, dYh)
        check(f"cfg1 dW_{j}", host(dW), dWo, "f32")
        Xs.append(Xd[offs[j]:offs[j + 1]]); dYs.append(dYd[offs[j]:offs[j + 1]])
    Yo, _ = olin.linear_fwd(Xh, Wh); dXo, dWo, _ = olin.linear_bwd(Xh, Wh, None, dYh)
    check("cfg1 Y", host(Y), Yo, "f32"); check("cfg1 dX", host(dX), dXo, "f32")
    # SFB rebuild from the two devices' gathered factors equals the all-reduced gradient
    dW = empty((1024, 1024), "f32", float("nan"))
    hap.hap_sfb_grad(Xs, dYs, sizes, 1024, 1024, 1024, 1024, hap.F32, dW, 1024)
    check("cfg1 SFB dW", host(dW), osfb.sfb_grad([Xh[:38], Xh[38:]], [dYh[:38], dYh[38:]], sizes), "f32")
    check("cfg1 SFB dW vs unsharded", host(dW), dWo, "f32")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode", [0, 1, 2, 3])
@pytest.mark.parametrize("full", [True, False])
def test_linear_modes_ragged(hap, dtype, mode, full):
    tokens, in_f, out_f = 300, 264, 520
    dim = {0: tokens, 1: out_f, 2: in_f, 3: 1}[mode]
    offsets = {0: [0, 131, 131, 257, 300], 1: [0, 137, 137, 391, 520], 2: [0, 99, 99, 200, 264], 3: [0, 1]}[mode]
    assert offsets[-1] == dim
    act = mode in (0, 1, 3)
    run_linear_case(hap, dtype, tokens, in_f, out_f, mode, offsets, act=act, bias=True, full=full)


@pytest.mark.parametrize("full", [True, False])
def test_linear_deep_ragged_contractions(hap, full):
    """Contracted ranges that start off the 16-byte grid and span many K tiles: first / last tiles of a range take the
    general tile body (per-chunk validity, zeroing of out-of-range k), the ones between the branch-free one."""
    run_linear_case(hap, "bf16", 260, 1000, 272, 2, [0, 333, 1000], act=False, bias=False, full=full)      # K ranges 333 | 667 of X columns
    run_linear_case(hap, "bf16", 1100, 200, 264, 0, [0, 451, 1100], act=True, bias=True, full=full)        # bwd-weight contracts 451 | 649 rows
    run_linear_case(hap, "bf16", 150, 264, 1210, 1, [0, 603, 1210], act=True, bias=True, full=full)        # bwd-data contracts 603 | 607 columns


@pytest.mark.parametrize("tokens,in_f,out_f", [(1, 300, 257), (8, 256, 64), (9, 288, 31), (38, 1024, 1024), (64, 292, 1000), (65, 256, 272), (113, 512, 260), (256, 264, 256),
                                               (257, 512, 96), (449, 512, 512), (70, 2080, 1040), (40, 33, 4100)])
@pytest.mark.parametrize("pad", [0, 1])
def test_fp32_layers_of_few_rows(hap, tokens, in_f, out_f, pad):
    """fp32 weight gradients over few rows (k chunks of 8 and 16, one or four waves per 32 x 32 tile), with and without the data gradient
    of few rows in the same launch, the bias gradient from the same registers; pitches off the 16-byte grid take other kernels for dX."""
    run_linear_case(hap, "f32", tokens, in_f, out_f, 3, [0, 1], act=False, bias=True, full=False, pad=pad)
    run_linear_case(hap, "f32", tokens, in_f, out_f, 1, [0, out_f // 3 + 1, out_f], act=True, bias=True, full=True)


@pytest.mark.parametrize("rows", [[38, 26], [0, 1, 17, 0, 64, 33], [0, 0], [200, 311]])
@pytest.mark.parametrize("in_f,out_f", [(1024, 1024), (100, 95), (2049, 2080)])
def test_fp32_sfb_over_few_rows(hap, rows, in_f, out_f):
    """Segments that end inside a chunk, empty ones among them; the sums join what is there with accumulate, and padding is never read."""
    cap = max(rows) + 2
    Xh, Xd, dYh, dYd = [], [], [], []
    for i in range(len(rows)):
        a, b = gen(2, T.SFB_X + i, (cap, in_f), 1.0, "f32"); Xh.append(a); Xd.append(b)
        a, b = gen(2, T.SFB_DY + i, (cap, out_f), 1.0, "f32"); dYh.append(a); dYd.append(b)
        Xd[i][rows[i]:] = float("nan"); dYd[i][rows[i]:] = float("nan")
    ref = osfb.sfb_grad(Xh, dYh, rows)
    dW = empty((in_f, out_f + 3), "f32", 7)
    for accumulate in (False, True):
        hap.hap_sfb_grad(Xd, dYd, rows, in_f, out_f, in_f, out_f, hap.F32, dW, out_f + 3, accumulate=accumulate)
        got = host(dW)
        assert (got[:, out_f:] == 7).all(), "the pitch's padding was written"
        if any(rows): check("fp32 sfb", got[:, :out_f], ref * (2 if accumulate else 1), "f32")
        else: assert not got[:, :out_f].any()


def test_fp32_backward_into_its_own_operands_keeps_the_order(hap):
    """The weight gradient may overwrite the weight that the data gradient has read, the bias gradient a row of X that the weight gradient
    has read: as by products that run one after the other."""
    Xh, Xd = gen(5, T.X, (38, 1024), 1.0, "f32"); Wh, Wd = gen(5, T.W, (1024, 1024), 0.05, "f32"); Gh, Gd = gen(5, T.DY, (38, 1024), 1.0, "f32")
    desc = hap.LinearDesc(38, 1024, 1024, hap.REPLICATED, [0, 1], hap.F32, m=1)
    ws = empty((hap.hap_linear_bwd_workspace(desc, 0),), "u8")
    dXo, dWo, dbo = olin.linear_bwd(Xh, Wh, None, Gh)
    dX = empty((38, 1024), "f32", 0)
    hap.hap_sharded_linear_bwd(desc, 0, Xd, Wd, None, Gd, dX, Wd, hap.F32, Xd[3], ws)
    check("dX", host(dX), dXo, "f32"); check("dW over W", host(Wd), dWo, "f32"); check("db over X", host(Xd)[3], dbo, "f32")


@pytest.mark.parametrize("k", [304, 384, 392, 448, 712])
def test_linear_big_tiles_over_short_contractions(hap, k):
    """Outputs that fill the chip with 256-tiles over 5 to 12 K tiles of 64: the two-stage kernel up to six of them, the ping-pong kernel
    (ring of four stages) beyond; the forward contracts k features, bwd-weight k rows of the first shard and 150 of the second."""
    run_linear_case(hap, "bf16", 3900, k, 4040, 3, [0, 1], act=True, bias=True, full=False)
    run_linear_case(hap, "bf16", k + 150, 3904, 4040, 0, [0, k, k + 150], act=False, bias=True, full=True)


def kernel_counts(hap):
    """Products so far in gemm_kpair_kernel, gemm_small_kernel and gemm_trio_kernel."""
    return np.array([hap.hap_debug_kpair_products(), hap.hap_debug_small_products(), hap.hap_debug_trio_products()])


@pytest.mark.parametrize("k", [193, 256, 257, 385, 449, 768])
def test_linear_smallest_outputs_over_ranges_inside_a_k_tile(hap, k):
    """The smallest outputs over ranges that start and end inside a K tile: the eight waves of a workgroup contract the same and different
    numbers of K steps (7 to 32 of 32), in all three products, without a workspace (forward) and with one (backward)."""
    def reached(*args, **kw):
        before = kernel_counts(hap)
        run_linear_case(hap, "bf16", *args, full=True, **kw)
        assert (kernel_counts(hap) - before == [0, 6, 0]).all(), args
    reached(130, 1000, 200, 2, [0, k, 1000], act=False, bias=False)
    reached(1000, 136, 264, 0, [0, k, 1000], act=True, bias=True, dw_dtype="f32")
    reached(130, 136, 1000, 1, [0, k, 1000], act=False, bias=True)
    reached(130, 136, 1000, 1, [0, k, 1000], act=True, bias=True)


@pytest.mark.parametrize("k", [193, 256, 257, 320, 385, 449, 768])
def test_linear_few_tiles_share_their_contraction_between_wave_groups(hap, k):
    """Outputs of few 128-tiles, but more than 256 tiles of 64 x 64 (the smallest outputs have a kernel of their own), over ranges that start
    and end inside a K tile: the two wave groups of a workgroup contract the same and different numbers of K tiles (4 to 13 of 64, odd
    and even).  Per shard one product contracts k or 1000 - k and has an output of 88 tiles; the others take this kernel or that of the
    smallest outputs.  (A group without any K tile needs a contraction that is shortened on the device: test_moe_few_tiles_per_expert.)"""
    def reached(*args, **kw):
        before = kernel_counts(hap)
        run_linear_case(hap, "bf16", *args, full=True, **kw)
        pair, small, trio = kernel_counts(hap) - before
        assert pair >= 2 and pair + small == 6, (args, pair, small, trio)
    reached(1300, 1000, 1016, 2, [0, k, 1000], act=False, bias=False)      # forward over k features
    reached(1300, 1016, 1000, 1, [0, k, 1000], act=True, bias=True)        # dX over k columns of the activation backward's copy
    reached(1300, 1016, 1000, 1, [0, k, 1000], act=False, bias=True)       # ... of the whole dY
    reached(1000, 1304, 1016, 0, [0, k, 1000], act=True, bias=True, dw_dtype="f32")    # dW over k rows


@pytest.mark.parametrize("k", [200, 264, 520, 1000])
def test_linear_paired_wave_groups_with_bias_gelu_and_preactivation(hap, k):
    """The forward's epilogue in the kernel of the paired wave groups: bias, GeLU and the pre-activation copy of unsplit contractions of 4 to 16
    K tiles, into columns on and off the output's 16-byte grid and into a compact slice."""
    for args, kw in [((1300, k, 2040, 1, [0, 1003, 2040]), dict(full=True)), ((1300, k, 2040, 1, [0, 1000, 2040]), dict(full=True)), ((1300, k, 1016, 3, [0, 1]), dict(full=False))]:
        shards = len(args[4]) - 1
        before = kernel_counts(hap)
        run_linear_case(hap, "bf16", *args, act=True, bias=True, **kw)
        assert kernel_counts(hap)[0] - before[0] >= shards, (args, kernel_counts(hap) - before)


@pytest.mark.parametrize("k", [8, 24, 32, 40, 96, 104, 200, 328, 520])
def test_linear_short_contractions_of_many_tiles(hap, k):
    """More than 512 tiles of 128 x 128 over one to seventeen K steps of 32 (fewer than the ring has stages, as many, more), interior and cut
    at both ends: bwd-data over the first third of k columns, the rest and all, the forward over either half of k features and all, with GeLU,
    its backward and without."""
    before = hap.hap_debug_trio_products()
    run_linear_case(hap, "bf16", 4300, 2104, k, 1, [0, k // 3, k], act=True, bias=True, full=True)        # dX over k // 3, k - k // 3
    run_linear_case(hap, "bf16", 4300, k, 2104, 2, [0, k // 2, k], act=False, bias=False, full=True)      # Y over k // 2
    run_linear_case(hap, "bf16", 4300, k, 2104, 3, [0, 1], act=True, bias=True, full=False)
    assert hap.hap_debug_trio_products() - before >= 5
    # the fused activation backward into columns that start on and off the output's 16-byte grid
    from oracle import pointwise as opw
    Xh, Xd = gen(13, T.X, (4300, 2104), 1.0, "bf16"); Wh, Wd = gen(13, T.W, (2104, k), 0.05, "bf16")
    dYh, dYd = gen(13, T.DY, (4300, k), 1.0, "bf16"); Ph, Pd = gen(13, T.MISC, (4300, 2104), 1.5, "bf16")
    for lo in (0, 3, 8):
        desc = hap.LinearDesc(4300, 2104, k, olin.REDUCTION, [0, lo, 2104], hap.BF16)
        want, _, _ = olin.sharded_linear_bwd(olin.REDUCTION, [0, lo, 2104], 1, Xh, Wh, None, dYh, False)
        dX = empty((4300, 2104), "bf16", float("nan"))
        hap.hap_sharded_linear_bwd_dact(desc, 1, Xd, Wd, None, dYd, dX, None, hap.BF16, None, Pd, hap.ACT_GELU_ERF, None)
        got = host(dX)
        check(f"dP k{k} lo{lo}", got[:, lo:], want * opw.gelu_grad(Ph[:, lo:]), "bf16")
        assert np.isnan(got[:, :lo]).all()


@pytest.mark.parametrize("k", [8, 24, 33, 64, 95, 104, 200, 329, 520, 770])
def test_linear_weight_gradients_of_many_tiles_over_few_rows(hap, k):
    """bf16 weight gradients of more than 512 tiles of 128 x 128 over one to 25 K steps of 32, into a compact slice and into a whole tensor's
    columns off the 16-byte grid: both operands M- / N-contiguous, three workgroups to a compute unit."""
    in_f, out_f = 2104, 4304
    Xh, Xd = gen(4, T.X, (k, in_f), 1.0, "bf16"); dYh, dYd = gen(4, T.DY, (k, out_f), 1.0, "bf16")
    W = empty((in_f, out_f), "bf16", 0)
    for mode, offsets, j in ((hap.REPLICATED, [0, 1], 0), (olin.FEATURE, [0, 3, out_f], 1)):
        lo = 3 if j else 0
        desc = hap.LinearDesc(k, in_f, out_f, mode, offsets, hap.BF16, m=len(offsets) - 1)
        dW = empty((in_f, out_f), "bf16", 9)
        before = hap.hap_debug_trio_products()
        hap.hap_sharded_linear_bwd(desc, j, Xd, W, None, dYd, None, dW, hap.BF16, None, empty((hap.hap_linear_bwd_workspace(desc, j),), "u8"))
        assert hap.hap_debug_trio_products() - before == 1
        assert (host(dW)[:, :lo] == 9).all()
        check("dW", host(dW)[:, lo:], Xh.T @ dYh[:, lo:], "bf16")


@pytest.mark.parametrize("tokens,in_f,out_f", [(1, 40, 24), (31, 72, 64), (33, 520, 65), (64, 32, 200), (65, 1000, 63), (197, 1024, 315), (250, 248, 1001), (450, 130, 1030), (1000, 3900, 260)])
def test_linear_smallest_outputs(hap, tokens, in_f, out_f):
    """Outputs of at most 256 tiles of 32 x 64 or 64 x 64 around the tiles' edges, over contractions from less than one K step of 32 (waves
    without any) to sixteen per wave, from whole tensors at odd columns and rows and from compact slices."""
    for mode, dim in [(0, tokens), (1, out_f), (2, in_f)]:
        before = hap.hap_debug_small_products()
        run_linear_case(hap, "bf16", tokens, in_f, out_f, mode, [0, dim // 3, dim], act=mode != 2, bias=True, full=True)
        if in_f % 8 == 0 and out_f % 8 == 0:      # (other pitches are not on the 16-byte grid: the scalar kernel)
            assert hap.hap_debug_small_products() - before >= 4, mode
    run_linear_case(hap, "bf16", tokens, in_f + 7 & ~7, out_f + 7 & ~7, 3, [0, 1], act=True, bias=True, full=False, dw_dtype="f32")


def test_linear_smallest_outputs_route(hap):
    """One tile per compute unit is the most: 256 tiles of 32 x 64, then of 64 x 64, then another kernel; the contraction has its limits."""
    torch = torch_mod()
    assert hap.hap_device_info()[0] == 256
    for tokens, in_f, out_f, want in [(512, 256, 1024, 1), (513, 256, 1024, 1), (1024, 256, 1024, 1), (1025, 256, 1024, 0), (1024, 3968, 1024, 1), (1024, 3976, 1024, 0),
                                      (128, 5120, 64, 1), (128, 5128, 64, 0), (40, 8, 8, 1)]:
        X, W, Y = empty((tokens, in_f), "bf16", 0), empty((in_f, out_f), "bf16", 0), empty((tokens, out_f), "bf16", 1)
        X[:, 0] = 1; W[0] = 2
        desc = hap.LinearDesc(tokens, in_f, out_f, hap.REPLICATED, [0, 1], hap.BF16, m=1)
        before = hap.hap_debug_small_products()
        hap.hap_sharded_linear_fwd(desc, 0, X, W, None, Y, None, empty((1 << 20,), "u8"))
        assert hap.hap_debug_small_products() - before == want, (tokens, in_f, out_f)
        assert (host(Y) == 2).all()


@pytest.mark.parametrize("product,tokens,in_f,out_f,most,alone", [("fwd", 320, None, 512, 136, 160), ("fwd", 256, None, 512, 160, 160), ("fwd", 512, None, 1024, 124, 124),
                                                                  ("fwd", 1024, None, 1024, 95, 124), ("dX", 320, 512, None, 136, 160), ("dX", 1024, 1024, None, 87, 124),
                                                                  ("dW", None, 256, 256, 144, 160), ("dW", None, 512, 512, 112, 160), ("dW", None, 768, 1024, 124, 124)])
def test_linear_smallest_outputs_end_where_others_split(hap, product, tokens, in_f, out_f, most, alone):
    """How many K steps of 32 the kernel of the smallest outputs takes where another kernel could split its contraction, by tile height,
    product and tile count, and without a workspace (`alone`).  Right on both sides of each line."""
    torch = torch_mod()
    for steps, scratch, want in ((most, True, 1), (most + 1, True, 0), (alone, False, 1), (alone + 1, False, 0)):
        k = steps * 32
        t, i, o = tokens or k, in_f or k, out_f or k
        X, W, dY = empty((t, i), "bf16", 0), empty((i, o), "bf16", 0), empty((t, o), "bf16", 0)
        X[:, 0] = 1; W[0] = 2; W[:, 0] = 2; dY[:, 0] = 3      # one feature, one column, all rows
        desc = hap.LinearDesc(t, i, o, hap.REPLICATED, [0, 1], hap.BF16, m=1)
        ws = empty((hap.hap_linear_bwd_workspace(desc, 0),), "u8") if scratch else None
        out = empty({"fwd": (t, o), "dX": (t, i), "dW": (i, o)}[product], "f32" if product == "dW" else "bf16", 1)
        before = hap.hap_debug_small_products()
        if product == "fwd": hap.hap_sharded_linear_fwd(desc, 0, X, W, None, out, None, ws)
        elif product == "dX": hap.hap_sharded_linear_bwd(desc, 0, X, W, None, dY, out, None, hap.BF16, None, ws)
        else: hap.hap_sharded_linear_bwd(desc, 0, X, W, None, dY, None, out, hap.F32, None, ws)
        assert hap.hap_debug_small_products() - before == want, (steps, scratch)
        got = host(out)
        if product == "fwd": assert (got == 2).all()
        elif product == "dX": assert (got == 6).all()
        else: assert got[0, 0] == 3 * k and not got[1:].any() and not got[:, 1:].any()


@pytest.mark.parametrize("scratch", [True, False])
@pytest.mark.parametrize("tokens,in_f,cut", [(130, 1000, 128), (130, 1000, 333), (130, 1000, 517), (1000, 1000, 128), (1000, 1000, 333), (1000, 1000, 517),
                                             (1300, 2040, 1000), (1300, 2040, 1003), (1300, 2040, 1037)])
@pytest.mark.parametrize("out_f", [264, 1104, 1600])
def test_linear_bwd_data_into_column_ranges(hap, tokens, in_f, cut, out_f, scratch):
    """bwd-data of a reduction shard of whole tensors: its columns of dX start on and off the output's 16-byte grid (`cut`), its rows of W
    with them; contractions of 5, 18 and 25 K tiles, plain and with the producer's gelu' in the epilogue.  1300 tokens (11 x 8 and 11 x 9 tiles of 128)
    take the kernel of the paired wave groups, fewer that of the smallest outputs, with a workspace and without."""
    from oracle import pointwise as opw
    offsets = [0, cut, in_f]
    Xh, Xd = gen(13, T.X, (tokens, in_f), 1.0, "bf16"); Wh, Wd = gen(13, T.W, (in_f, out_f), 0.05, "bf16")
    dYh, dYd = gen(13, T.DY, (tokens, out_f), 1.0, "bf16"); Ph, Pd = gen(13, T.MISC, (tokens, in_f), 1.5, "bf16")
    desc = hap.LinearDesc(tokens, in_f, out_f, olin.REDUCTION, offsets, hap.BF16)
    for j in range(2):
        lo, hi = offsets[j], offsets[j + 1]
        want, _, _ = olin.sharded_linear_bwd(olin.REDUCTION, offsets, j, Xh, Wh, None, dYh, False)
        ws = empty((hap.hap_linear_bwd_workspace(desc, j),), "u8") if scratch else None
        for act in (False, True):
            dX = empty((tokens, in_f), "bf16", float("nan"))
            before = kernel_counts(hap)
            hap.hap_sharded_linear_bwd_dact(desc, j, Xd, Wd, None, dYd, dX, None, hap.BF16, None, Pd if act else None, hap.ACT_GELU_ERF if act else hap.ACT_NONE, ws)
            taken = kernel_counts(hap) - before
            got = host(dX)
            check(f"dX act{int(act)} shard {j}", got[:, lo:hi], want * opw.gelu_grad(Ph[:, lo:hi]) if act else want, "bf16")
            assert np.isnan(got[:, :lo]).all() and np.isnan(got[:, hi:]).all(), "columns outside the shard were written"
            assert (taken == ([1, 0, 0] if tokens == 1300 else [0, 1, 0])).all(), (lo, hi, taken)


@pytest.mark.parametrize("scratch", [0, 1 << 16, None])
def test_linear_route_to_the_paired_wave_groups(hap, scratch):
    """Products of at most one 128-tile per compute unit and at least four K tiles take the kernel with two wave groups, whatever the
    workspace holds (nothing, too little for a single split, everything): few tiles over a short contraction, poorly filled tile counts
    over a long one.  Fewer K tiles or more output tiles do not, and neither do the smallest outputs."""
    torch = torch_mod()
    cus, _ = hap.hap_device_info()
    assert cus == 256
    for tokens, in_f, out_f, want in [(250, 880, 500, [0, 0, 0]),         # at most 14 x 8 tiles of 64
                                      (1300, 1016, 1104, [1, 1, 1]),       # 11 x 9 output tiles over 16 K tiles, 11 x 8 over 18, 8 x 9 over 21
                                      (1270, 4090, 1140, [1, 0, 0])]:      # 10 x 9 over 64; 10 x 32 and 32 x 9 tiles are too many
        Xh, Xd = gen(3, T.X, (tokens, in_f), 1.0, "bf16"); Wh, Wd = gen(3, T.W, (in_f, out_f), 0.05, "bf16"); Gh, Gd = gen(3, T.DY, (tokens, out_f), 1.0, "bf16")
        ld = lambda n: (n + 7) // 8 * 8
        wide = lambda t: torch.nn.functional.pad(t, (0, ld(t.shape[1]) - t.shape[1]))
        Xd, Wd, Gd = wide(Xd), wide(Wd), wide(Gd)
        desc = hap.LinearDesc(tokens, in_f, out_f, hap.REPLICATED, [0, 1], hap.BF16, ldx=ld(in_f), ldw=ld(out_f), ldy=ld(out_f), m=1)
        ws = empty((scratch if scratch else hap.hap_linear_bwd_workspace(desc, 0),), "u8") if scratch != 0 else None
        Y, dX, dW = empty(Gd.shape, "bf16", 0), empty(Xd.shape, "bf16", 0), empty(Wd.shape, "bf16", 0)
        Yo, _ = olin.linear_fwd(Xh, Wh); dXo, dWo, _ = olin.linear_bwd(Xh, Wh, None, Gh)
        n = [hap.hap_debug_kpair_products()]
        hap.hap_sharded_linear_fwd(desc, 0, Xd, Wd, None, Y, None, ws); n.append(hap.hap_debug_kpair_products())
        hap.hap_sharded_linear_bwd(desc, 0, Xd, Wd, None, Gd, dX, None, hap.BF16, None, ws); n.append(hap.hap_debug_kpair_products())
        hap.hap_sharded_linear_bwd(desc, 0, Xd, Wd, None, Gd, None, dW, hap.BF16, None, ws); n.append(hap.hap_debug_kpair_products())
        check("route Y", host(Y)[:, :out_f], Yo, "bf16"); check("route dX", host(dX)[:, :in_f], dXo, "bf16"); check("route dW", host(dW)[:, :out_f], dWo, "bf16")
        assert [b - a for a, b in zip(n, n[1:])] == want, (tokens, in_f, out_f, n)
    for tokens, in_f, out_f in [(1300, 190, 1000), (17 * 128, 256, 16 * 128)]:  # 3 K tiles; 17 x 16 output tiles
        Xd, Wd, Y = empty((tokens, 256), "bf16", 0), empty((in_f, 2048), "bf16", 0), empty((tokens, 2048), "bf16", 1)
        desc = hap.LinearDesc(tokens, in_f, out_f, hap.REPLICATED, [0, 1], hap.BF16, ldx=256, ldw=2048, ldy=2048, m=1)
        before = hap.hap_debug_kpair_products()
        hap.hap_sharded_linear_fwd(desc, 0, Xd, Wd, None, Y, None)
        assert hap.hap_debug_kpair_products() == before and not host(Y)[:, :out_f].any()


def test_linear_unaligned_leading_dimensions_take_the_scalar_kernel(hap):
    # compact slices whose leading dimension is not a multiple of 16 bytes
    run_linear_case(hap, "bf16", 70, 50, 90, 1, [0, 37, 90], act=True, bias=True, full=False, pad=3)
    run_linear_case(hap, "f32", 70, 50, 90, 2, [0, 21, 50], act=False, bias=False, full=False, pad=1)


def test_linear_bf16_fp32_weight_gradient(hap):
    run_linear_case(hap, "bf16", 515, 256, 384, 1, [0, 129, 384], act=True, bias=True, full=True, dw_dtype="f32")


def test_index_ranges_bit_exact_through_identity(hap):
    """An iota tensor pushed through an identity weight: each shard must reproduce exactly its own rows / columns."""
    torch = torch_mod()
    n = 160
    ratios, _ = hap.hap_shard_ratios([1.0, 0.6, 0.35], [(1.0, 0, 0, 0)])
    sizes, offs = hap.hap_round_shards(ratios, n)
    assert (sizes, offs) == ornd.round_shards(olp.shard_ratios([1.0, 0.6, 0.35], [(1.0, 0, 0, 0)])[0], n)
    iota = torch.arange(n * n, dtype=torch.float32, device="cuda").reshape(n, n) % 251   # exact in bf16
    eye = torch.eye(n, dtype=torch.float32, device="cuda")
    for dtype, td in (("f32", torch.float32), ("bf16", torch.bfloat16)):
        X, W = iota.to(td), eye.to(td)
        for mode in (0, 1):
            desc = hap.LinearDesc(n, n, n, mode, offs, DT[dtype])
            for j in range(3):
                Y = empty((n, n), dtype, -1)
                hap.hap_sharded_linear_fwd(desc, j, X, W, None, Y, None)
                got = host(Y); ref = host(X)
                mask = np.zeros((n, n), bool)
                if mode == 0:
                    mask[offs[j]:offs[j + 1], :] = True
                else:
                    mask[:, offs[j]:offs[j + 1]] = True
                assert np.array_equal(got[mask], ref[mask]) and (got[~mask] == -1).all()


def test_sfb_ragged_segments_padding_never_read(hap):
    rows = [70, 0, 33, 128, 1]
    cap, in_f, out_f = 128, 200, 328
    Xh, Xd, dYh, dYd = [], [], [], []
    for i in range(len(rows)):
        a, b = gen(1, T.SFB_X + i, (cap, in_f), 1.0, "bf16"); Xh.append(a); Xd.append(b)
        a, b = gen(1, T.SFB_DY + i, (cap, out_f), 1.0, "bf16"); dYh.append(a); dYd.append(b)
        Xd[i][rows[i]:] = float("nan"); dYd[i][rows[i]:] = float("nan")     # poison the padded All-Gather rows
    ref = osfb.sfb_grad(Xh, dYh, rows)
    dW = empty((in_f, out_f), "f32", float("nan"))
    hap.hap_sfb_grad(Xd, dYd, rows, in_f, out_f, in_f, out_f, hap.BF16, dW, out_f)
    check("sfb", host(dW), ref, "bf16")
    hap.hap_sfb_grad(Xd, dYd, rows, in_f, out_f, in_f, out_f, hap.BF16, dW, out_f, accumulate=True)
    check("sfb accumulate", host(dW), 2 * ref, "bf16")
    # grouped-Broadcast layout: compact factors (cap_i == rows_i), one device only -> plain X^T dY
    dW1 = empty((in_f, out_f), "f32", 0)
    hap.hap_sfb_grad([Xd[3]], [dYd[3]], [128], in_f, out_f, in_f, out_f, hap.BF16, dW1, out_f)
    check("sfb m=1", host(dW1), Xh[3].T @ dYh[3], "bf16")
    # all devices empty -> zeros
    hap.hap_sfb_grad(Xd, dYd, [0] * 5, in_f, out_f, in_f, out_f, hap.BF16, dW1, out_f)
    assert not host(dW1).any()


# Outputs (rows, columns) and contractions that are split over workgroups where there is a workspace: the K-pair kernel in three, 128-tiles in
# five (eight wave groups short of a full chip otherwise), 256-tiles in three.
SPLITS = [(1000, 1096, 4104), (1000, 1304, 8200), (1800, 2200, 4104)]


def run_sfb_case(hap, rows, in_f, out_f, splits):
    cap = max(rows)
    Xh, Xd, dYh, dYd = [], [], [], []
    for i in range(len(rows)):
        a, b = gen(9, T.SFB_X + i, (cap, in_f), 1.0, "bf16"); Xh.append(a); Xd.append(b)
        a, b = gen(9, T.SFB_DY + i, (cap, out_f), 1.0, "bf16"); dYh.append(a); dYd.append(b)
        Xd[i][rows[i]:] = float("nan"); dYd[i][rows[i]:] = float("nan")
    ref = osfb.sfb_grad(Xh, dYh, rows)
    ws = empty((hap.hap_sfb_workspace(len(rows), rows, in_f, out_f),), "u8")
    n = [hap.hap_debug_split_products()]
    dW = empty((in_f, out_f), "f32", float("nan"))
    hap.hap_sfb_grad(Xd, dYd, rows, in_f, out_f, in_f, out_f, hap.BF16, dW, out_f, ws=ws); n.append(hap.hap_debug_split_products())
    check("sfb with a workspace", host(dW), ref, "bf16")
    dW1 = empty((in_f, out_f), "f32", float("nan"))
    hap.hap_sfb_grad(Xd, dYd, rows, in_f, out_f, in_f, out_f, hap.BF16, dW1, out_f); n.append(hap.hap_debug_split_products())
    assert np.abs(host(dW1) - host(dW)).max() <= 1e-5 * np.abs(ref).max()      # fp32 partial sums, different order only
    hap.hap_sfb_grad(Xd, dYd, rows, in_f, out_f, in_f, out_f, hap.BF16, dW, out_f, accumulate=True, ws=ws); n.append(hap.hap_debug_split_products())
    check("sfb accumulate", host(dW), 2 * ref, "bf16")
    # a pitch and a base off the 16-byte grid: element by element
    flat = empty((in_f * (out_f + 3) + 1,), "f32", 5)
    hap.hap_sfb_grad(Xd, dYd, rows, in_f, out_f, in_f, out_f, hap.BF16, flat.data_ptr() + 4, out_f + 3, accumulate=True, ws=ws); n.append(hap.hap_debug_split_products())
    got = host(flat)
    assert got[0] == 5 and (got[1:].reshape(in_f, out_f + 3)[:, out_f:] == 5).all()
    check("sfb off the grid", got[1:].reshape(in_f, out_f + 3)[:, :out_f], 5 + ref, "bf16")
    assert [b - a for a, b in zip(n, n[1:])] == ([1, 0, 1, 1] if splits else [0, 0, 0, 0])


@pytest.mark.parametrize("in_f,out_f,k", SPLITS)
def test_sfb_split_k_over_segment_boundaries(hap, in_f, out_f, k):
    """With workspace the engine splits the contracted axis over idle compute units; the split points fall
    inside and between the devices' ragged segments.  Result must equal the one-pass result."""
    run_sfb_case(hap, [k // 3 + 5, 0, 77, k // 2, k - k // 3 - k // 2 - 82], in_f, out_f, True)


def test_sfb_of_the_smallest_outputs_over_ragged_segments(hap):
    """Eight waves share a tile's contraction; their ranges start and end inside and between the segments, whatever the workspace."""
    run_sfb_case(hap, [300, 0, 77, 512, 130], 264, 392, False)


@pytest.mark.parametrize("m,n,k", SPLITS)
@pytest.mark.parametrize("dn", [0, 2, 5])
@pytest.mark.parametrize("y_phase,p_phase", [(0, 0), (4, 4), (3, 3), (0, 2)])
def test_linear_split_k_with_bias_gelu_and_preactivation(hap, m, n, k, dn, y_phase, p_phase):
    """The reduction behind a forward that is split over workgroups: bias, GeLU and the saved pre-activation, with columns that are and are not
    a multiple of four and output rows that start on the 8-byte grid (whole quads) and off it (elements)."""
    n -= dn
    Xh, Xd = gen(5, T.X, (m, k), 1.0, "bf16"); Wh, Wd = gen(5, T.W, (k, n), 0.05, "bf16"); bh, bd = gen(5, T.BIAS, (n,), 0.5, "bf16")
    ld = (n + 7) // 8 * 8
    Wd = torch_mod().nn.functional.pad(Wd, (0, ld - n), value=float("nan"))
    desc = hap.LinearDesc(m, k, n, hap.REPLICATED, [0, 1], hap.BF16, act=hap.ACT_GELU_ERF, has_bias=True, ldx=k, ldw=ld, ldy=ld, m=1)
    ws = empty((hap.lib.hap_linear_fwd_workspace(None, 0),), "u8")
    Y, P = empty((m * ld + 8,), "bf16", 9), empty((m * ld + 8,), "bf16", 9)
    before = hap.hap_debug_split_products()
    hap.hap_sharded_linear_fwd(desc, 0, Xd, Wd, bd, Y.data_ptr() + 2 * y_phase, P.data_ptr() + 2 * p_phase, ws)
    assert hap.hap_debug_split_products() - before == 1
    Yo, preo = olin.linear_fwd(Xh, Wh, bh, True)
    for name, t, phase, want in (("Y", Y, y_phase, Yo), ("preact", P, p_phase, preo)):
        got = host(t)
        assert (got[:phase] == 9).all() and (got[phase + m * ld:] == 9).all(), name
        got = got[phase:phase + m * ld].reshape(m, ld)
        assert (got[:, n:] == 9).all(), "the pitch's padding was written"
        check("split-k " + name, got[:, :n], want, "bf16")


@pytest.mark.parametrize("m,n,k", SPLITS[:2])
@pytest.mark.parametrize("cut", [0, 3, 8])
def test_linear_split_k_with_activation_backward_into_column_ranges(hap, m, n, k, cut):
    """The reduction behind a split bwd-data with the producer's gelu', into columns of a whole tensor that start on and off the 16-byte grid;
    without a workspace the same product in one pass, and the weight gradient of the same shard split over the same rows."""
    from oracle import pointwise as opw
    Xh, Xd = gen(13, T.X, (m, n), 1.0, "bf16"); Wh, Wd = gen(13, T.W, (n, k), 0.05, "bf16")
    dYh, dYd = gen(13, T.DY, (m, k), 1.0, "bf16"); Ph, Pd = gen(13, T.MISC, (m, n), 1.5, "bf16")
    desc = hap.LinearDesc(m, n, k, olin.REDUCTION, [0, cut, n], hap.BF16)
    want, _, _ = olin.sharded_linear_bwd(olin.REDUCTION, [0, cut, n], 1, Xh, Wh, None, dYh, False)
    for scratch in (True, False):
        dX = empty((m, n), "bf16", float("nan"))
        before = hap.hap_debug_split_products()
        hap.hap_sharded_linear_bwd_dact(desc, 1, Xd, Wd, None, dYd, dX, None, hap.BF16, None, Pd, hap.ACT_GELU_ERF,
                                        empty((hap.hap_linear_bwd_workspace(desc, 1),), "u8") if scratch else None)
        assert hap.hap_debug_split_products() - before == int(scratch)
        got = host(dX)
        assert np.isnan(got[:, :cut]).all()
        check(f"dP scratch {scratch}", got[:, cut:], want * opw.gelu_grad(Ph[:, cut:]), "bf16")


@pytest.mark.parametrize("m,n,k", SPLITS)
@pytest.mark.parametrize("dw_dtype", ["bf16", "f32"])
def test_linear_split_k_weight_gradient_into_column_ranges(hap, m, n, k, dw_dtype):
    """Weight gradients split over workgroups, into a whole tensor's columns off the 16-byte grid."""
    Xh, Xd = gen(4, T.X, (k, m), 1.0, "bf16"); dYh, dYd = gen(4, T.DY, (k, n), 1.0, "bf16")
    W = empty((m, n), "bf16", 0)
    desc = hap.LinearDesc(k, m, n, olin.FEATURE, [0, 3, n], hap.BF16)
    dW = empty((m, n), dw_dtype, 9)
    before = hap.hap_debug_split_products()
    hap.hap_sharded_linear_bwd(desc, 1, Xd, W, None, dYd, None, dW, DT[dw_dtype], None, empty((hap.hap_linear_bwd_workspace(desc, 1),), "u8"))
    assert hap.hap_debug_split_products() - before == 1
    assert (host(dW)[:, :3] == 9).all()
    check("dW", host(dW)[:, 3:], Xh.T @ dYh[:, 3:], dw_dtype if dw_dtype == "bf16" else "bf16")


@pytest.mark.parametrize("scratch", [True, False])
def test_fp32_split_k_with_workspace(hap, scratch):
    """fp32 products whose 64-tiles cannot occupy the chip and whose rows are too many for the kernels of the few-row layers: split over
    workgroups where there is a workspace (forward with bias + GeLU, bwd-data, a weight gradient over many rows); same 1e-5 bar."""
    for tokens, in_f, out_f, want in [(512, 2048, 512, (1, 1, 0)), (700, 3000, 520, (1, 0, 0)), (4100, 264, 260, (1, 1, 1))]:
        Xh, Xd = gen(0, T.X, (tokens, in_f), 1.0, "f32"); Wh, Wd = gen(0, T.W, (in_f, out_f), 0.02, "f32"); dYh, dYd = gen(0, T.DY, (tokens, out_f), 1.0, "f32")
        bh, bd = gen(0, T.BIAS, (out_f,), 0.5, "f32")
        fwd = hap.LinearDesc(tokens, in_f, out_f, hap.REPLICATED, [0, 1], hap.F32, act=hap.ACT_GELU_ERF, has_bias=True, m=1)
        bwd = hap.LinearDesc(tokens, in_f, out_f, hap.REPLICATED, [0, 1], hap.F32, m=1)
        ws = empty((hap.hap_linear_bwd_workspace(bwd, 0),), "u8") if scratch else None
        nan = float("nan")
        Y, P, dX, dW = empty((tokens, out_f), "f32", nan), empty((tokens, out_f), "f32", nan), empty((tokens, in_f), "f32", nan), empty((in_f, out_f), "f32", nan)
        n = [hap.hap_debug_split_products()]
        hap.hap_sharded_linear_fwd(fwd, 0, Xd, Wd, bd, Y, P, ws); n.append(hap.hap_debug_split_products())
        hap.hap_sharded_linear_bwd(bwd, 0, Xd, Wd, None, dYd, dX, None, hap.F32, None, ws); n.append(hap.hap_debug_split_products())
        hap.hap_sharded_linear_bwd(bwd, 0, Xd, Wd, None, dYd, None, dW, hap.F32, None, ws); n.append(hap.hap_debug_split_products())
        Yo, Po = olin.linear_fwd(Xh, Wh, bh, True); dXo, dWo, _ = olin.linear_bwd(Xh, Wh, None, dYh)
        check("Y", host(Y), Yo, "f32"); check("preact", host(P), Po, "f32"); check("dX", host(dX), dXo, "f32"); check("dW", host(dW), dWo, "f32")
        assert tuple(b - a for a, b in zip(n, n[1:])) == (want if scratch else (0, 0, 0)), (tokens, in_f, out_f, n)


@pytest.mark.parametrize("tokens,out_f,most", [(128, 256, 5120), (104, 688, 2048), (192, 688, 1364), (256, 1024, 1024)])
def test_fp32_rows_beyond_64_split_k_where_that_is_faster(hap, tokens, out_f, most):
    """Up to `most` features the contraction is shared by the waves of a workgroup, beyond it is split over workgroups if the workspace allows;
    a weight whose rows are off the 16-byte grid has no kernel that could.  fp32 bar on both sides."""
    torch = torch_mod()
    for in_f, pad, scratch, want in ((most, 0, True, 0), (most + 4, 0, True, 1), (most + 4, 0, False, 0), (most + 4, 1, True, 0)):
        Xh, Xd = gen(3, T.X, (tokens, in_f), 1.0, "f32"); Wh, Wd = gen(3, T.W, (in_f, out_f), 0.05, "f32"); bh, bd = gen(3, T.BIAS, (out_f,), 0.5, "f32")
        Wd = torch.nn.functional.pad(Wd, (0, pad), value=float("nan"))
        desc = hap.LinearDesc(tokens, in_f, out_f, hap.REPLICATED, [0, 1], hap.F32, act=hap.ACT_GELU_ERF, has_bias=True, ldx=in_f, ldw=out_f + pad, ldy=out_f, m=1)
        Y, P = empty((tokens, out_f), "f32", float("nan")), empty((tokens, out_f), "f32", float("nan"))
        before = hap.hap_debug_split_products()
        hap.hap_sharded_linear_fwd(desc, 0, Xd, Wd, bd, Y, P, empty((64 << 20,), "u8") if scratch else None)
        assert hap.hap_debug_split_products() - before == want, (in_f, pad, scratch)
        Yo, Po = olin.linear_fwd(Xh, Wh, bh, True)
        check("Y", host(Y), Yo, "f32"); check("preact", host(P), Po, "f32")


def test_linear_smallest_outputs_with_bias_gelu_and_ragged_view(hap):
    """Deep contraction, few output tiles, bias + GeLU + saved pre-activation, misaligned column range, into one pair of whole tensors."""
    tokens, in_f, out_f = 200, 1024, 520
    offs = [0, 137, 391, 520]
    Xh, Xd = gen(5, T.X, (tokens, in_f), 1.0, "bf16"); Wh, Wd = gen(5, T.W, (in_f, out_f), 0.05, "bf16")
    bh, bd = gen(5, T.BIAS, (out_f,), 0.5, "bf16")
    desc = hap.LinearDesc(tokens, in_f, out_f, hap.SHARD_FEATURE, offs, hap.BF16, act=hap.ACT_GELU_ERF, has_bias=True)
    ws = empty((hap.lib.hap_linear_fwd_workspace(None, 0),), "u8")
    Yo, preo = olin.linear_fwd(Xh, Wh, bh, True)
    Y = empty((tokens, out_f), "bf16", 0); P = empty((tokens, out_f), "bf16", 0)
    for j in range(3):
        hap.hap_sharded_linear_fwd(desc, j, Xd, Wd, bd, Y, P, ws)
    check("Y", host(Y), Yo, "bf16"); check("preact", host(P), preo, "bf16")


def test_cfg1_fp32_with_workspace(hap):
    """Config 1 again with workspace, which neither the kernel of few rows nor the one launch of the backward needs; same 1e-5 bar, forward
    with bias + GeLU and all gradients."""
    offs = [0, 38, 64]
    Xh, Xd = gen(0, T.X, (64, 1024), 1.0, "f32"); Wh, Wd = gen(0, T.W, (1024, 1024), 0.02, "f32"); dYh, dYd = gen(0, T.DY, (64, 1024), 1.0, "f32")
    bh, bd = gen(0, T.BIAS, (1024,), 0.5, "f32")
    desc = hap.LinearDesc(64, 1024, 1024, hap.SHARD_BATCH, offs, hap.F32, act=hap.ACT_GELU_ERF, has_bias=True)
    Y = empty((64, 1024), "f32", 0); P = empty((64, 1024), "f32", 0); dX = empty((64, 1024), "f32", 0); db = empty((1024,), "f32", 0)
    wsf = empty((hap.lib.hap_linear_fwd_workspace(None, 0),), "u8")
    Yo, Po = olin.linear_fwd(Xh, Wh, bh, True)
    dW_sum = np.zeros((1024, 1024)); db_sum = np.zeros(1024)
    for j in range(2):
        hap.hap_sharded_linear_fwd(desc, j, Xd, Wd, bd, Y, P, wsf)
        wsb = empty((hap.hap_linear_bwd_workspace(desc, j),), "u8")
        dW = empty((1024, 1024), "f32", float("nan"))
        hap.hap_sharded_linear_bwd(desc, j, Xd, Wd, P, dYd, dX, dW, hap.F32, db, wsb)
        dW_sum += host(dW); db_sum += host(db)
    dXo, dWo, dbo = olin.linear_bwd(Xh, Wh, Po, dYh, act=True)
    check("cfg1 Y", host(Y), Yo, "f32"); check("cfg1 preact", host(P), Po, "f32")
    check("cfg1 dX", host(dX), dXo, "f32"); check("cfg1 dW", dW_sum, dWo, "f32"); check("cfg1 db", db_sum, dbo, "f32")


def test_linear_seeded_random_sweep(hap):
    """A seeded sweep over shapes, rules, layouts and options nobody hand-picked: tiny to multi-tile extents, ragged everything,
    random shard boundaries (including empty shards), compact and whole-tensor operands, odd pads."""
    rng = np.random.default_rng(20240105)
    for trial in range(28):
        dtype = "bf16" if trial % 3 else "f32"
        tokens = int(rng.choice([1, 7, 33, 130, 257, 515, 700]))
        in_f = int(rng.choice([1, 8, 24, 100, 264, 513]))
        out_f = int(rng.choice([1, 8, 40, 136, 300, 520]))
        mode = int(rng.choice([olin.BATCH, olin.FEATURE, olin.REDUCTION, olin.REPLICATED]))
        axis = {olin.BATCH: tokens, olin.FEATURE: out_f, olin.REDUCTION: in_f, olin.REPLICATED: 1}[mode]
        m = int(rng.integers(1, 4))
        cuts = sorted(int(c) for c in rng.integers(0, axis + 1, m - 1))
        offsets = [0] + cuts + [axis] if mode != olin.REPLICATED else [0, 1]
        act = bool(rng.integers(0, 2)) and mode != olin.REDUCTION
        bias = bool(rng.integers(0, 2))
        full = bool(rng.integers(0, 2))
        pad = int(rng.choice([0, 0, 1, 8])) if not full else 0
        dw_dtype = "f32" if (dtype == "f32" or rng.integers(0, 2)) else "bf16"
        run_linear_case(hap, dtype, tokens, in_f, out_f, mode, offsets, act, bias, full, dw_dtype=dw_dtype, pad=pad, seed=100 + trial)


def test_cfg1_step_replays_from_a_hip_graph(hap):
    """The library's calls only launch kernels on the given stream (no allocation, no memset, no host synchronisation), so a
    whole latency-bound step - config 1: forward + backward of both devices and the SFB rebuild - can be captured once and
    replayed.  Every replay, with eager work and synchronisations in between, must reproduce the eager results bit for bit."""
    torch = torch_mod()
    offs = [0, 38, 64]
    _, Xd = gen(0, T.X, (64, 1024), 1.0, "f32"); _, Wd = gen(0, T.W, (1024, 1024), 0.02, "f32"); _, dYd = gen(0, T.DY, (64, 1024), 1.0, "f32")
    desc = hap.LinearDesc(64, 1024, 1024, hap.SHARD_BATCH, offs, hap.F32)
    ws = empty((hap.hap_linear_bwd_workspace(desc, 0),), "u8")
    out = {k: empty(s, "f32", 0) for k, s in (("Y", (64, 1024)), ("dX", (64, 1024)), ("dW0", (1024, 1024)), ("dW1", (1024, 1024)), ("dWs", (1024, 1024)))}

    def step():
        for j in range(2):
            hap.hap_sharded_linear_fwd(desc, j, Xd, Wd, None, out["Y"], None, ws)
            hap.hap_sharded_linear_bwd(desc, j, Xd, Wd, None, dYd, out["dX"], out[f"dW{j}"], hap.F32, None, ws)
        hap.hap_sfb_grad([Xd[:38], Xd[38:]], [dYd[:38], dYd[38:]], [38, 26], 1024, 1024, 1024, 1024, hap.F32, out["dWs"], 1024, ws=ws)
    step()
    torch.cuda.synchronize()
    want = {k: v.clone() for k, v in out.items()}
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        step()                      # warm the capture stream's state
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    for rep in range(3):
        for v in out.values():
            v.fill_(float(rep + 1))                      # eager work between replays: results must come from the replay
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in out:
            assert torch.equal(out[k], want[k]), (rep, k)
        step()                                           # and an eager step in between
        torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode,full", [("batch", True), ("batch", False), ("reduction", True), ("reduction", False), ("replicated", False)])
@pytest.mark.parametrize("shape", [(300, 200, 130), (64, 96, 4200), (1031, 517, 263)])
def test_linear_bwd_with_producer_activation_backward(hap, dtype, mode, full, shape):
    """hap_sharded_linear_bwd_dact: dX * gelu'(x_preact) in the dX product's epilogue equals the oracle's dX times the oracle's
    gelu', for every shard of the modes whose dX is complete on the device; shapes take the tiled kernels, the split
    contraction (64 x 96 outputs over 4200) and ragged tiles with odd leading dimensions (the element-wise stores)."""
    from oracle import pointwise as opw
    tokens, in_f, out_f = shape
    code = {"batch": olin.BATCH, "reduction": olin.REDUCTION, "replicated": olin.REPLICATED}[mode]
    axis = {"batch": tokens, "reduction": in_f, "replicated": 1}[mode]
    offsets = [0, axis * 2 // 5, axis * 2 // 5, axis] if mode != "replicated" else [0, 1]
    Xh, Xd = gen(11, T.X, (tokens, in_f), 1.0, dtype); Wh, Wd = gen(11, T.W, (in_f, out_f), 0.05, dtype)
    dYh, dYd = gen(11, T.DY, (tokens, out_f), 1.0, dtype); Ph, Pd = gen(11, T.MISC, (tokens, in_f), 1.5, dtype)   # the producer's pre-activation
    for j in range(len(offsets) - 1):
        lo, hi = offsets[j], offsets[j + 1]
        dXo, dWo, _ = olin.sharded_linear_bwd(code, offsets, j, Xh, Wh, None, dYh, False)
        rs = slice(lo, hi) if mode == "batch" else slice(None)
        cs = slice(lo, hi) if mode == "reduction" else slice(None)
        want = dXo * opw.gelu_grad(Ph[rs, cs])
        if full or mode == "replicated":
            Xj, Wj, dYj, Pj = Xd, Wd, dYd, Pd
            ldx, ldw, ldy = in_f, out_f, out_f
            dXj = empty((tokens, in_f), dtype, float("nan"))
        else:
            Xj, Pj = Xd[rs, cs].contiguous(), Pd[rs, cs].contiguous()
            Wj = Wd[cs].contiguous() if mode == "reduction" else Wd
            dYj = dYd[rs].contiguous()
            ldx, ldw, ldy = Xj.shape[1], out_f, out_f
            dXj = empty(tuple(Xj.shape), dtype, float("nan"))
        if Xj.numel() == 0:
            Xj = Pj = dXj = empty((8, max(ldx, 8)), dtype, 0); ldx = max(ldx, 8)
        desc = hap.LinearDesc(tokens, in_f, out_f, code, offsets, DT[dtype], ldx=ldx, ldw=ldw, ldy=ldy, operands_are_full=full, m=len(offsets) - 1)
        ws = empty((max(hap.hap_linear_bwd_workspace(desc, j), 16),), "u8")
        dWj = empty((Wj.shape[0], ldw), "f32", 0)
        hap.hap_sharded_linear_bwd_dact(desc, j, Xj, Wj, None, dYj, dXj, dWj, hap.F32, None, Pj, hap.ACT_GELU_ERF, ws)
        got = host(dXj)
        if full and mode != "replicated":
            inside = got[rs, cs]
            outside = np.ones(got.shape, bool); outside[rs, cs] = False
            assert np.isnan(got[outside]).all(), "elements outside the shard were written"
            got = inside
        elif hi == lo and mode != "replicated":
            continue
        if want.size:
            e = check(f"{dtype} {mode} full{int(full)} shard {j} dX*gelu'", got, want, dtype)
            # and it is the two-step result: the plain backward followed by the element-wise pass, same roundings
            dX2 = empty(tuple(dXj.shape), dtype, float("nan"))
            hap.hap_sharded_linear_bwd(desc, j, Xj, Wj, None, dYj, dX2, None, hap.F32, None, ws)
            if full and mode != "replicated":
                v2, vp = dX2[rs, cs].contiguous(), Pd[rs, cs].contiguous()
            else:
                v2, vp = dX2, Pj
            two = empty(tuple(v2.shape), dtype, 0)
            hap.hap_gelu_bwd(v2.shape[0], v2.shape[1], DT[dtype], vp, vp.stride(0), v2, v2.stride(0), two, two.stride(0))
            assert relerr(got, host(two)) <= (1e-2 if dtype == "bf16" else 1e-5)


def test_linear_bwd_dact_rejects_partial_sums(hap):
    """In feature mode dX is a partial sum: an activation backward applied before the All-Reduce would be wrong, so the call refuses."""
    desc = hap.LinearDesc(64, 32, 48, olin.FEATURE, [0, 20, 48], hap.F32, ldx=32, ldw=48, ldy=48, operands_are_full=True)
    X, W, dY, dX, P = (empty(s, "f32", 0) for s in ((64, 32), (32, 48), (64, 48), (64, 32), (64, 32)))
    ws = empty((hap.hap_linear_bwd_workspace(desc, 0),), "u8")
    with pytest.raises(hap.HapError):
        hap.hap_sharded_linear_bwd_dact(desc, 0, X, W, None, dY, dX, None, hap.F32, None, P, hap.ACT_GELU_ERF, ws)
    with pytest.raises(hap.HapError):
        d2 = hap.LinearDesc(64, 32, 48, olin.BATCH, [0, 20, 64], hap.F32, ldx=32, ldw=48, ldy=48, operands_are_full=True)
        hap.hap_sharded_linear_bwd_dact(d2, 0, X, W, None, dY, dX, None, hap.F32, None, None, hap.ACT_GELU_ERF, ws)


@pytest.mark.parametrize("tokens", [1, 16, 38, 64])
@pytest.mark.parametrize("in_f,out_f", [(1024, 1024), (256, 1000), (4100, 17), (2048, 8000), (4100, 264), (1600, 1600)])
def test_fp32_layer_with_few_rows(hap, tokens, in_f, out_f):
    """fp32 layers of at most 64 rows (config 1's shards are 38 and 26 rows) run forward and bwd-data in a kernel that splits the
    contraction over the waves of a workgroup and sums the partial tiles through LDS: all row-block counts, ragged column tiles,
    contractions that do not divide by the 16 waves, bias + GeLU + saved pre-activation, and dX through the K-contiguous weight.
    (8000 columns are 125 tiles of 64: just below where the tiled kernel takes over.  4100 columns of dX take all rows in one workgroup, and so
    does the forward of 38 rows over 1600 features, whose dX takes three row blocks.)"""
    Xh, Xd = gen(3, T.X, (tokens, in_f), 1.0, "f32"); Wh, Wd = gen(3, T.W, (in_f, out_f), 0.05, "f32")
    bh, bd = gen(3, T.BIAS, (out_f,), 0.5, "f32"); dYh, dYd = gen(3, T.DY, (tokens, out_f), 1.0, "f32")
    desc = hap.LinearDesc(tokens, in_f, out_f, olin.REPLICATED, [0, 1], hap.F32, act=hap.ACT_GELU_ERF, has_bias=True, m=1)
    Y = empty((tokens, out_f), "f32", float("nan")); P = empty((tokens, out_f), "f32", float("nan"))
    ws = empty((max(hap.hap_linear_bwd_workspace(desc, 0), 16),), "u8")
    hap.hap_sharded_linear_fwd(desc, 0, Xd, Wd, bd, Y, P, ws)
    Yo, preo = olin.linear_fwd(Xh, Wh, bh, True)
    check("Y", host(Y), Yo, "f32"); check("preact", host(P), preo, "f32")
    dX = empty((tokens, in_f), "f32", float("nan")); dW = empty((in_f, out_f), "f32", float("nan")); db = empty((out_f,), "f32", float("nan"))
    hap.hap_sharded_linear_bwd(desc, 0, Xd, Wd, P, dYd, dX, dW, hap.F32, db, ws)
    dXo, dWo, dbo = olin.linear_bwd(Xh, Wh, preo, dYh, True)
    check("dX", host(dX), dXo, "f32"); check("dW", host(dW), dWo, "f32"); check("db", host(db), dbo, "f32")
