"""GPU: kernels at the sizes where their partitioning can go wrong -- one tile, runs that end inside a wave, the
first size that needs a second pass of a loop -- against the oracle or against an independent kernel of the
library that the oracle pins elsewhere."""
import numpy as np
import pytest
import torch

from oracle import fgmp_oracle as orc
from paper_2504_14152_amd import build, fgmp, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


# ------------------------------------------------------------------ packing weights

def _run_lengths(mask: torch.Tensor, rows: int, K: int) -> torch.Tensor:
    """FP8 slots per 8 x 128 tile, in tile order, from a canonical mask."""
    n_rt, n_kt = -(-rows // 8), -(-(K // 16) // 8)
    m = torch.zeros((n_rt * 8, n_kt * 8), dtype=torch.int64, device=mask.device)
    m[:rows, : K // 16] = mask.to(torch.int64)
    return m.view(n_rt, 8, n_kt, 8).sum((1, 3)).flatten()


# (rows, K): one tile; fewer tiles than waves; tiles per wave that leave a ragged last run; 2 per wave; and, with
# one block per row, more than 512 x 16 x 64 tiles, where a wave walks its run in two batches
@pytest.mark.parametrize("rows,K", [(1, 16), (8, 144), (520, 2064), (70000, 144), (4200000, 16)])
@pytest.mark.parametrize("p", [0.0, 0.1, 1.0])
def test_packed_weights_hold_the_same_blocks_as_the_one_pass_layout(rows, K, p):
    g = torch.Generator(device=DEV).manual_seed(rows + K)
    w = torch.randn(rows, K, generator=g, device=DEV).to(torch.bfloat16)
    f = torch.exp(torch.randn(K, generator=g, device=DEV))
    s = float(w.abs().max()) / 448.0
    _, scores = fgmp.quantize_weights(w, f, float("inf"), s, want_scores=True)
    T = fgmp.threshold_for_fraction(scores, p)
    pw = fgmp.quantize_weights(w, f, T, s)
    px = fgmp.quantize_activations(w, f, T, s)       # strided layout: nothing shared with the packing pass
    for a, b in zip(fgmp.unpack_canonical(pw), fgmp.unpack_canonical(px)):
        assert torch.equal(a, b)
    mask = fgmp.unpack_canonical(px)[2]
    counts = _run_lengths(mask, rows, K)
    info = fgmp.packed_info(pw)
    assert info["n_fp8_blocks"] == int(counts.sum())
    n_tiles = counts.numel()
    off_T = 256 + n_tiles * 512                       # planes L, S, M precede T, each 256-byte aligned
    off_T = -(-off_T // 256) * 256 + n_tiles * 64
    off_T = -(-off_T // 256) * 256 + n_tiles * 8
    off_T = -(-off_T // 256) * 256
    plane_t = pw.buf[off_T: off_T + 4 * n_tiles].view(torch.int32).to(torch.int64)
    assert torch.equal(plane_t, torch.cumsum(counts, 0) - counts)
    off_H = -(-(off_T + 4 * n_tiles) // 256) * 256
    assert info["bytes_used"] == off_H + 8 * max(1, int(counts.sum()))


# ------------------------------------------------------------------ products of 20 .. 1024 rows

def _product(M, K, N, dtype, p, seed):
    x = synth.activations(M, K, seed, 1)
    w = synth.weights(N, K, seed, 2)
    fx, fw = synth.fisher_per_channel(K, seed, 3), synth.fisher_per_channel(K, seed, 4)
    xd = torch.from_numpy(x).to(DEV).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    wd = torch.from_numpy(w).to(DEV)
    xref = xd.float().cpu().numpy()
    fxd, fwd = torch.from_numpy(fx).to(DEV), torch.from_numpy(fw).to(DEV)
    sx, sw = float(synth.default_tensor_scale(xref)), float(synth.default_tensor_scale(w))
    Tx = fgmp.threshold_for_fraction(fgmp.quantize_activations(xd, fxd, float("inf"), sx, want_scores=True)[1], p)
    Tw = fgmp.threshold_for_fraction(fgmp.quantize_weights(wd, fwd, float("inf"), sw, want_scores=True)[1], p)
    pW = fgmp.quantize_weights(wd, fwd, Tw, sw)
    qx, qw = orc.quantize(xref, fx, Tx, sx), orc.quantize(w, fw, Tw, sw)
    want, tol = orc.gemm(orc.dequantize(qx["codes"], qx["scales"], qx["mask"]), sx,
                         orc.dequantize(qw["codes"], qw["scales"], qw["mask"]), sw)
    return xd, fxd, Tx, sx, pW, want, tol


# (M, K, N): rows one past a tile; columns that end inside a lane group, an odd number of 8-row weight tiles; K groups
# without a K-tile in the last round, K in several parts across workgroups; long products of 20 to 32 rows and, with 19 rows or
# just below N K^2 = 2^38, their neighbours on the decode kernels; and the neighbours on the prefill kernel, with K of one block, one
# and two K-tiles
MID_SHAPES = [(33, 16, 24, "f32", 0.1), (48, 128, 264, "bf16", 0.1), (64, 4096, 136, "bf16", 0.2), (77, 2064, 503, "f32", 0.2),
              (96, 640, 72, "bf16", 0.0), (112, 1168, 1000, "bf16", 1.0), (129, 384, 40, "f32", 0.3), (200, 8192, 200, "bf16", 0.1),
              (300, 1040, 264, "bf16", 0.1), (512, 2816, 328, "bf16", 0.1), (700, 144, 136, "bf16", 0.1), (1024, 272, 72, "f32", 0.1),
              (40, 256, 34000, "bf16", 0.1), (20, 65536, 256, "bf16", 0.1), (19, 65536, 128, "bf16", 0.1), (32, 32768, 264, "f32", 0.1),
              (32, 32768, 248, "f32", 0.1), (27, 11008, 2400, "bf16", 0.1)]


@pytest.mark.parametrize("M,K,N,dtype,p", MID_SHAPES)
def test_products_of_a_few_dozen_to_a_few_hundred_rows_match_oracle(M, K, N, dtype, p):
    """Within 1e-5 of the sum of magnitudes (FP32 accumulation), equal to the product of the packed activations and to a
    second call bit for bit, counters left zero, and equal to the build in which every hand-counted wait is a full one."""
    from paper_2504_14152_amd import build
    xd, fxd, Tx, sx, pW, want, tol = _product(M, K, N, dtype, p, 70 + M)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(M, N, K), DEV)
    ws[fgmp.WORKSPACE_CONTROL_BYTES:] = 0xFF       # partial sums and rows beyond M start as NaN patterns
    Y = fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, workspace=ws)
    err = np.abs(Y.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= tol), (err / tol).max()
    assert int(ws[: fgmp.WORKSPACE_CONTROL_BYTES].sum()) == 0
    assert torch.equal(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, workspace=ws), Y)
    assert torch.equal(fgmp.gemm(fgmp.quantize_activations(xd, fxd, Tx, sx), pW), Y)
    with fgmp.use_library(build.lib_path("fullwait")):
        assert torch.equal(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW), Y)


# (M, K, N), (16-row groups, 16-column groups of a wave), K shared among workgroups: every instantiation that the planner
# uses, with and without a shared K where it uses both; the last one has 411 workgroups, more than run at once
MID_PLANS = [((49, 160, 10), (2, 2), False), ((49, 5008, 8), (2, 2), True), ((23, 4368, 17911), (2, 3), False),
             ((32, 7184, 6183), (2, 3), True), ((21, 3360, 26570), (2, 4), False), ((24, 12704, 6355), (2, 4), True),
             ((40, 144, 8), (3, 2), False), ((39, 4512, 8), (3, 2), True), ((33, 160, 16503), (3, 3), False),
             ((65, 5616, 2751), (3, 3), True), ((65, 272, 12409), (3, 4), False), ((36, 9472, 6289), (3, 4), True),
             ((199, 160, 8), (4, 2), False), ((195, 3632, 9), (4, 2), True), ((153, 272, 5647), (4, 3), False),
             ((194, 4128, 1347), (4, 3), True), ((160, 416, 8215), (4, 4), False), ((195, 8016, 1579), (4, 4), True),
             ((331, 144, 8), (5, 2), False), ((327, 1856, 8), (5, 2), True), ((210, 416, 10897), (5, 3), False),
             ((327, 2416, 1541), (5, 3), True), ((506, 144, 8), (6, 2), False), ((482, 1616, 8), (6, 2), True),
             ((248, 416, 10953), (6, 3), False), ((482, 2432, 1388), (6, 3), True), ((875, 144, 8), (7, 2), False),
             ((889, 1344, 8), (7, 2), True), ((297, 1952, 12322), (7, 3), False), ((963, 1600, 1054), (7, 3), True),
             ((1017, 432, 3224), (8, 2), False), ((1011, 1552, 841), (8, 2), True), ((228, 3792, 17051), (8, 3), False),
             ((1019, 1552, 1211), (8, 3), True), ((267, 2544, 17421), (6, 2), False)]


@pytest.mark.parametrize("shape,groups,shared", MID_PLANS)
def test_every_arrangement_of_the_mid_size_kernel_matches_oracle(shape, groups, shared):
    """On 96 columns, first and last among them, within 1e-5 of the sum of magnitudes; whole results equal to a second
    call and to the build in which every hand-counted wait is a full one, bit for bit."""
    from paper_2504_14152_amd import build
    M, K, N = shape
    route = fgmp.selftest_gemm_route(M, N, K)
    assert route[0] == 2 and route[1:3] == groups and (route[5] > 1) == shared
    gen = torch.Generator(device=DEV).manual_seed(M + N)
    dtype = torch.float32 if M % 2 else torch.bfloat16
    xd = torch.randn(M, K, generator=gen, device=DEV).to(dtype)
    wd = (torch.randn(N, K, generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
    fx, fw = torch.exp(torch.randn(K, generator=gen, device=DEV)), torch.exp(torch.randn(K, generator=gen, device=DEV))
    sx, sw = float(xd.abs().max()) / 448.0, float(wd.abs().max()) / 448.0
    Tx = fgmp.threshold_for_fraction(fgmp.quantize_activations(xd, fx, float("inf"), sx, want_scores=True)[1], 0.2)
    Tw = fgmp.threshold_for_fraction(fgmp.quantize_weights(wd, fw, float("inf"), sw, want_scores=True)[1], 0.2)
    pW = fgmp.quantize_weights(wd, fw, Tw, sw)
    Y = fgmp.quant_gemm_fused(xd, fx, Tx, sx, pW)
    cols = np.unique(np.linspace(0, N - 1, min(N, 96)).astype(np.int64))
    qx = orc.quantize(xd.float().cpu().numpy(), fx.cpu().numpy(), Tx, sx)
    qw = orc.quantize(wd[torch.from_numpy(cols).to(DEV)].float().cpu().numpy(), fw.cpu().numpy(), Tw, sw)
    want, tol = orc.gemm(orc.dequantize(qx["codes"], qx["scales"], qx["mask"]), sx, orc.dequantize(qw["codes"], qw["scales"], qw["mask"]), sw)
    err = np.abs(Y[:, torch.from_numpy(cols).to(DEV)].cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= tol), (err / tol).max()
    assert torch.equal(fgmp.quant_gemm_fused(xd, fx, Tx, sx, pW), Y)
    with fgmp.use_library(build.lib_path("fullwait")):
        assert torch.equal(fgmp.quant_gemm_fused(xd, fx, Tx, sx, pW), Y)


def test_products_between_decode_and_prefill_replay_in_a_graph():
    """K in parts (partial sums, counters that the kernel puts back to zero), replayed with other work between."""
    xd, fxd, Tx, sx, pW, _, _ = _product(64, 8192, 200, "bf16", 0.1, 91)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(64, 200, 8192), DEV)
    Y = torch.empty(64, 200, device=DEV)
    fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, out=Y, workspace=ws)
    want = Y.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, out=Y, workspace=ws)
    for _ in range(4):
        Y.fill_(float("nan"))
        ws[fgmp.WORKSPACE_CONTROL_BYTES:] = 0xFF
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want)


# (M, K, N), workgroups that hold a share: a last chunk of 64 blocks that ends inside the tensor, rows in K-tiles of which part lies
# beyond K, fewer chunks than workgroups and more, shares for some of the workgroups, most and all of them, 256 workgroups, one
# block per thread almost and exactly, and more (none hold a share: two launches), partial sums across workgroups, 24 rows
@pytest.mark.parametrize("M,K,N,holders", [(33, 144, 136, 3), (33, 160, 16503, 3), (65, 272, 12409, 7), (77, 2064, 5003, 41), (77, 2064, 503, 0),
                                           (64, 4096, 12288, 64), (120, 368, 603, 30), (96, 640, 700, 22), (96, 640, 72, 0), (512, 4096, 4096, 256),
                                           (516, 4096, 4096, 0), (49, 7696, 5491, 94), (154, 10976, 4810, 208), (24, 11008, 4096, 65)])
@pytest.mark.parametrize("dtype,mode", [("bf16", None), ("f32", "delta")])
@pytest.mark.parametrize("switch", [None, ("FGMP_MID_PATIENCE", "0"), ("FGMP_MID_ABSENT", "1"), ("FGMP_MID_ABSENT", "999")])
def test_products_that_quantize_in_their_launch_are_those_of_packed_activations(M, K, N, holders, dtype, mode, switch, monkeypatch):
    """Against the product of activations packed beforehand, which the oracle pins above: the same kernel over the same values, so
    every bit agrees.  Without patience (a switch of the build with measurement hooks, as the next) every workgroup makes the shares
    that it finds missing; with the last holder absent, or all of them, the others make theirs."""
    assert fgmp.selftest_gemm_route(M, N, K)[0] == 2 and fgmp.selftest_quantizing_workgroups(M, N, K) == holders
    g = torch.Generator(device=DEV).manual_seed(M + K + N)
    w = torch.randn(N, K, generator=g, device=DEV) * 0.02
    f = torch.exp(torch.randn(K, generator=g, device=DEV))
    pW = fgmp.quantize_weights(w, f, 1e-5, float(w.abs().max()) / 448.0)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(M, N, K), DEV)
    if switch is not None:
        monkeypatch.setenv(*switch)
    with fgmp.use_library(build.lib_path("hooks" if switch is not None else None)):
        for call in range(3):   # other inputs each time, in the place where the earlier ones' values lie
            x = torch.randn(M, K, generator=g, device=DEV).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
            s = float(x.float().abs().max()) / 448.0
            ws[fgmp.WORKSPACE_CONTROL_BYTES:].fill_(0xFF)   # NaN wherever nothing is written
            got = fgmp.quant_gemm_fused(x, f, 0.5, s, pW, workspace=ws, score_mode=mode)
            want = fgmp.gemm(fgmp.quantize_activations(x, f, 0.5, s, score_mode=mode), pW)
            assert torch.equal(got, want), call
            assert int(ws[: fgmp.WORKSPACE_CONTROL_BYTES].count_nonzero()) == 0


def test_products_that_quantize_in_their_launch_replay_in_a_graph_with_other_inputs():
    """Three launches one behind the other on one workspace, nothing between them: each finds the words as the one before left them and,
    where its values go, other ones, which the chip's caches may hold from the replay before.  Inputs change between replays."""
    g = torch.Generator(device=DEV).manual_seed(17)
    shapes = [(64, 4096, 12288), (64, 4096, 12288), (77, 2064, 5003)]
    assert all(fgmp.selftest_quantizing_workgroups(M, N, K) > 0 for M, K, N in shapes)
    weights, calls = {}, []
    for M, K, N in shapes:
        f = torch.exp(torch.randn(K, generator=g, device=DEV))
        if (K, N) not in weights:
            w = torch.randn(N, K, generator=g, device=DEV) * 0.02
            weights[K, N] = fgmp.quantize_weights(w, f, 1e-5, float(w.abs().max()) / 448.0)
        calls.append((torch.empty(M, K, dtype=torch.bfloat16, device=DEV), f, weights[K, N], torch.empty(M, N, device=DEV)))
    ws = fgmp.new_workspace(max(fgmp.workspace_bytes(M, N, K) for M, K, N in shapes), DEV)

    def step():
        for x, f, pw, y in calls:
            fgmp.quant_gemm_fused(x, f, 0.5, 0.011, pw, out=y, workspace=ws)

    def fresh():
        for x, _, _, _ in calls:
            x.copy_(torch.randn(x.shape, generator=g, device=DEV))

    fresh()
    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for replay in range(5):
        fresh()
        graph.replay()
        torch.cuda.synchronize()
        for x, f, pw, y in calls:
            assert torch.equal(y, fgmp.gemm(fgmp.quantize_activations(x, f, 0.5, 0.011), pw)), replay
        assert int(ws[: fgmp.WORKSPACE_CONTROL_BYTES].count_nonzero()) == 0


# (runs of one, two, three and more K-tiles, the last one shorter; a single run and several; an odd number of row-tiles; parts of K)
@pytest.mark.parametrize("M,K,N", [(3, 128, 4096), (5, 256, 22016), (1, 4096, 4096), (1, 4096, 12288), (1, 11008, 1032), (8, 384, 6168), (2, 640, 72),
                                   (20, 4096, 4104), (32, 11008, 520)])
@pytest.mark.parametrize("source", ["bf16", "packed"])
def test_decode_steps_over_weights_that_are_not_compact(M, K, N, source):
    """The same codes with the upper halves where the activation quantizer puts them: every tile's plane-T word is needed, not a run's
    first one only.  Every bit as from the compact tensor."""
    assert fgmp.selftest_gemm_route(M, N, K)[0] == 0
    g = torch.Generator(device=DEV).manual_seed(M + K + N)
    w = torch.randn(N, K, generator=g, device=DEV) * 0.02
    f = torch.exp(torch.randn(K, generator=g, device=DEV))
    x = torch.randn(M, K, generator=g, device=DEV).bfloat16()
    sw, sx = float(w.abs().max()) / 448.0, float(x.abs().max()) / 448.0
    _, scores = fgmp.quantize_activations(w, f, float("inf"), sw, want_scores=True)
    for fraction in (0.1, 0.6):
        T = fgmp.threshold_for_fraction(scores, fraction)
        compact, strided = fgmp.quantize_weights(w, f, T, sw), fgmp.quantize_activations(w, f, T, sw)
        assert (fgmp.packed_info(compact)["compact"], fgmp.packed_info(strided)["compact"]) == (1, 0)
        if source == "packed":
            px = fgmp.quantize_activations(x, f, 0.5, sx)
            got, want = fgmp.gemm(px, strided), fgmp.gemm(px, compact)
        else:
            got, want = (fgmp.quant_gemm_fused(x, f, 0.5, sx, p) for p in (strided, compact))
        assert torch.equal(got, want) and bool(got.any())


# (launches that hold half of the chip, most of it and all of it; shares for a third of the workgroups, most and all)
@pytest.mark.parametrize("M,K,N", [(36, 5920, 1759), (64, 4096, 12288), (200, 4096, 22016), (207, 6496, 720)])
def test_products_that_quantize_in_their_launch_overlap_on_four_streams(M, K, N):
    """A workspace each, started together and followed by more, other inputs every time: launches that share the chip find shares
    whose workgroups have not started, and make them.  Every result is that of packed activations, bit for bit."""
    assert fgmp.selftest_quantizing_workgroups(M, N, K) > 0
    g = torch.Generator(device=DEV).manual_seed(M + K + N)
    w = torch.randn(N, K, generator=g, device=DEV) * 0.02
    f = torch.exp(torch.randn(K, generator=g, device=DEV))
    pW = fgmp.quantize_weights(w, f, 1e-5, float(w.abs().max()) / 448.0)
    streams = [torch.cuda.Stream() for _ in range(4)]
    spaces = [fgmp.new_workspace(fgmp.workspace_bytes(M, N, K), DEV) for _ in streams]
    xs = [[torch.randn(M, K, generator=g, device=DEV).bfloat16() for _ in range(3)] for _ in streams]
    scales = [[float(x.abs().max()) / 448.0 for x in row] for row in xs]
    want = [[fgmp.gemm(fgmp.quantize_activations(x, f, 0.5, s), pW) for x, s in zip(*row)] for row in zip(xs, scales)]
    out = [[torch.empty(M, N, device=DEV) for _ in range(3)] for _ in streams]
    torch.cuda.synchronize()
    for call in range(3):
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                fgmp.quant_gemm_fused(xs[i][call], f, 0.5, scales[i][call], pW, out=out[i][call], workspace=spaces[i])
    torch.cuda.synchronize()
    for i in range(len(streams)):
        assert all(torch.equal(got, y) for got, y in zip(out[i], want[i])), i
        assert int(spaces[i][: fgmp.WORKSPACE_CONTROL_BYTES].count_nonzero()) == 0


def test_long_products_of_few_rows_quantize_the_results_of_the_plain_call():
    M, K, N = 28, 16384, 2048
    xd, fxd, Tx, sx, pW, _, _ = _product(M, K, N, "bf16", 0.1, 93)
    Y = fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW)
    f_n = torch.from_numpy(synth.fisher_per_channel(N, 93, 5)).to(DEV)
    sy = float(Y.abs().max()) / 448.0
    T_y = fgmp.threshold_for_fraction(fgmp.quantize_activations(Y, f_n, float("inf"), sy, want_scores=True)[1], 0.1)
    want = fgmp.unpack_canonical(fgmp.quantize_activations(Y, f_n, T_y, sy))
    for epilogue in (fgmp.EPILOGUE_NONE, fgmp.EPILOGUE_ONE_LAUNCH):
        got = fgmp.unpack_canonical(fgmp.quant_gemm_fused_packed_out(xd, fxd, Tx, sx, pW, f_n, T_y, sy, epilogue=epilogue))
        assert all(torch.equal(a, b) for a, b in zip(got, want))
    got = torch.empty(M, N, device=DEV)
    fgmp.quant_gemm_fused_static_scratch(xd, fxd, Tx, sx, pW, out=got)
    assert torch.equal(got, Y)


def test_static_scratch_takes_products_of_more_than_32_rows():
    # (the last one: prefill tiles split along K, whose partial sums fit right behind the activations only, or the kernel for fewer rows)
    for M, K, N in ((64, 4096, 1024), (300, 1040, 264), (200, 16, 24), (1100, 256, 264)):
        xd, fxd, Tx, sx, pW, _, _ = _product(M, K, N, "bf16", 0.1, 92)
        got = torch.full((M, N), float("nan"), device=DEV)
        fgmp.quant_gemm_fused_static_scratch(xd, fxd, Tx, sx, pW, out=got)
        assert torch.equal(got, fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW))


# ------------------------------------------------------------------ products on the prefill kernel

# (M, K, N), all on the 256 x 256 tiles: a round of 85 to 119 tiles, each computed in two parts of K whose sums meet in
# memory, with 4, 6, 8, 10, 16 and 18 K-steps of 64 -- of which the main loop turns over 6 at a time -- and ragged ends
@pytest.mark.parametrize("M,K,N", [(4100, 256, 1200), (4097, 272, 1280), (4200, 512, 1100), (4100, 640, 1500), (4352, 1024, 1030), (4100, 1040, 1700)])
def test_products_in_two_parts_match_oracle(M, K, N):
    """Within 1e-5 of the sum of magnitudes, and the same bits every time, whichever part comes first."""
    route = fgmp.selftest_gemm_route(M, N, K)
    assert route[0] == 3 and route[2] == 0 and 64 < route[3] <= 128 and route[4] == 2
    xd, fxd, Tx, sx, pW, want, tol = _product(M, K, N, "bf16", 0.1, 95)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(M, N, K), DEV)
    ws[fgmp.WORKSPACE_CONTROL_BYTES:] = 0xFF
    Y = fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, workspace=ws)
    err = np.abs(Y.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= tol), (err / tol).max()
    px = fgmp.quantize_activations(xd, fxd, Tx, sx)
    for _ in range(8):
        assert torch.equal(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, workspace=ws), Y)
        assert torch.equal(fgmp.gemm(px, pW, workspace=ws), Y)


@pytest.mark.parametrize("K,N", [(4096, 4096), (11008, 4096)])
def test_one_workspace_serves_every_batch_up_to_the_one_it_was_sized_for(K, N):
    """64 rows use less than 20 or 32 rows, whose K is shared among workgroups; the size of 64 rows is enough for all of them."""
    xd, fxd, Tx, sx, pW, _, _ = _product(64, K, N, "bf16", 0.1, 94)
    f_n = torch.ones(N, device=DEV)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(64, N, K), DEV)
    ws_packed = fgmp.new_workspace(fgmp.workspace_bytes_packed_out(64, N, K), DEV)
    for M in (64, 33, 32, 20, 16, 1):
        want = fgmp.quant_gemm_fused(xd[:M], fxd, Tx, sx, pW)
        assert torch.equal(fgmp.quant_gemm_fused(xd[:M], fxd, Tx, sx, pW, workspace=ws), want)
        assert torch.equal(fgmp.gemm(fgmp.quantize_activations(xd[:M], fxd, Tx, sx), pW, workspace=ws), want)
        got = fgmp.quant_gemm_fused_packed_out(xd[:M], fxd, Tx, sx, pW, f_n, 0.0, 1.0, workspace=ws_packed)
        for a, b in zip(fgmp.unpack_canonical(got), fgmp.unpack_canonical(fgmp.quantize_activations(want, f_n, 0.0, 1.0))):
            assert torch.equal(a, b)


# ------------------------------------------------------------------ clipping: the candidates that are left out

@pytest.mark.parametrize("what", ["ordinary", "heavy tails", "sparse sensitivities", "huge range", "negative", "tiny", "small scale", "large scale", "uneven"])
def test_clipped_scales_are_the_brute_force_ones(what):
    """The kernel tries only the codes whose error can be the smallest; the oracle tries all 127."""
    rng = synth.rng_for(33, len(what))
    N, K = 72, 528
    w = rng.standard_normal((N, K)).astype(np.float32) * np.float32(0.02)
    f = np.exp(rng.standard_normal((N, K))).astype(np.float32)
    scale = 1.0
    if what == "heavy tails":
        w *= np.exp(1.5 * rng.standard_normal((N, K))).astype(np.float32)
    elif what == "sparse sensitivities":
        f[rng.random((N, K)) < 0.8] = 0.0          # blocks decided by a few elements, some by none
        w[:, :16] = 0.0
        w[:, 16:32] = np.float32(0.0125)           # all elements equal: ties
    elif what == "huge range":
        f = np.exp(12.0 * rng.standard_normal((N, K))).astype(np.float32)
    elif what == "negative":
        f *= np.where(rng.random((N, K)) < 0.1, -1.0, 1.0).astype(np.float32)
    elif what == "tiny":
        w *= np.float32(1e-12)
        f *= np.float32(1e-10)
    elif what == "small scale":
        scale = 1.0 / 64.0                          # blocks beyond the largest code
    elif what == "large scale":
        scale = 300.0                               # every block among the first few codes
    elif what == "uneven":                          # a wave's ranges from empty (zeros) over a few codes to most of them
        f = np.exp(np.repeat(rng.uniform(0.0, 4.0, (N, K // 16)), 16, axis=1) * rng.standard_normal((N, K))).astype(np.float32)
        w *= np.repeat(rng.random((N, K // 16)) < 0.8, 16, axis=1)
        w[:, 64:80] *= np.arange(16) == 5           # one element each
    S = float(synth.default_tensor_scale(w)) * scale
    want = orc.quantize(w, f, float("inf"), S, clip=True)
    pk, scores = fgmp.quantize_weights_clip(torch.from_numpy(w).to(DEV), torch.from_numpy(f).to(DEV), float("inf"), S, want_scores=True)
    codes, scales, mask = (t.cpu().numpy() for t in fgmp.unpack_canonical(pk))
    assert np.array_equal(scales, want["scales"]) and np.array_equal(codes, want["codes"]) and np.array_equal(mask, want["mask"])
    assert np.array_equal(scores.cpu().numpy().view(np.uint32), want["scores"].view(np.uint32))


@pytest.mark.parametrize("what", ["three values", "codes already", "across code 8", "wide ranges", "close seconds", "vanishing sensitivities"])
def test_clipped_scales_found_by_estimates_are_the_brute_force_ones(what):
    """Candidates are ranked by an estimate of their error; equal and nearly equal errors, errors of zero and scales that are not
    normal numbers are where that could show."""
    rng = synth.rng_for(37, len(what))
    N, K = 136, 656
    w = rng.standard_normal((N, K)).astype(np.float32) * np.float32(0.02)
    f = np.exp(rng.standard_normal((N, K))).astype(np.float32)
    scale = 1.0
    if what == "three values":                      # many codes with the same error: every code is compared
        w = (np.sign(w) * (np.abs(w) > 0.01) * 0.03).astype(np.float32)
    elif what == "codes already":                   # reconstructed exactly under some code (S is a power of two)
        grid = np.array([0, 0.5, 1, 1.5, 2, 3, 4, 6], np.float32)
        w = grid[rng.integers(0, 8, (N, K))] * np.where(rng.random((N, K)) < 0.5, -1, 1) * np.repeat(2.0 ** rng.integers(-3, 3, (N, K // 16)), 16, axis=1)
        w = w.astype(np.float32)
        w[0, 0] = 448.0
    elif what == "across code 8":
        w *= np.repeat(2.0 ** -rng.uniform(0.0, 6.0, (N, K // 16)), 16, axis=1).astype(np.float32)
        scale = 12.0
    elif what == "wide ranges":
        f = np.exp(3.0 * rng.standard_normal((N, K))).astype(np.float32)
        f[:, ::3] *= np.float32(1e-6)
    elif what == "close seconds":                   # two halves that trade places from code to code
        w[:, 1::2] = w[:, ::2] * np.float32(1.0 + 2.0 ** -22)
        f[:, 1::2] = f[:, ::2]
    elif what == "vanishing sensitivities":         # on both sides of where the estimate is not used
        f[: N // 2] *= np.where(rng.random((N // 2, K)) < 0.02, 1e-33, 1.0).astype(np.float32)
        f[N // 2:] *= np.float32(1e-26)
    S = float(synth.default_tensor_scale(w)) * scale
    want = orc.quantize(w, f, float("inf"), S, clip=True)
    pk, scores = fgmp.quantize_weights_clip(torch.from_numpy(w).to(DEV), torch.from_numpy(f).to(DEV), float("inf"), S, want_scores=True)
    codes, scales, mask = (t.cpu().numpy() for t in fgmp.unpack_canonical(pk))
    assert np.array_equal(scales, want["scales"]) and np.array_equal(codes, want["codes"]) and np.array_equal(mask, want["mask"])
    assert np.array_equal(scores.cpu().numpy().view(np.uint32), want["scores"].view(np.uint32))


def _assert_clipped_as_by_the_oracle(w, f, S):
    want = orc.quantize(w, f, float("inf"), S, clip=True)
    pk, scores = fgmp.quantize_weights_clip(torch.from_numpy(w).to(DEV), torch.from_numpy(f).to(DEV), float("inf"), S, want_scores=True)
    codes, scales, mask = (t.cpu().numpy() for t in fgmp.unpack_canonical(pk))
    assert np.array_equal(scales, want["scales"]), f"{int((scales != want['scales']).sum())} of {scales.size} scales"
    assert np.array_equal(codes, want["codes"]) and np.array_equal(mask, want["mask"])
    assert np.array_equal(scores.cpu().numpy().view(np.uint32), want["scores"].view(np.uint32))


@pytest.mark.parametrize("what", ["one in a block", "beside zero weights", "one in each short block", "per channel"])
def test_clipped_scales_with_sensitivities_of_minus_zero_are_the_brute_force_ones(what):
    """-0.0 compares equal to zero and weighs nothing, as zero does; its root and its reciprocal are negative, though."""
    rng = synth.rng_for(38, len(what))
    N, K = 72, 528
    w = rng.standard_normal((N, K)).astype(np.float32) * np.float32(0.02)
    f = np.exp(rng.standard_normal((N, K))).astype(np.float32)
    at = 16 * np.arange(K // 16) + rng.integers(0, 16, (N, K // 16))
    scale = 1.0
    if what == "beside zero weights":
        w[np.arange(N)[:, None], at ^ 1] = 0.0
        w[: N // 2][np.arange(N // 2)[:, None], at[: N // 2]] = 0.0
    elif what == "one in each short block":         # ranges too short for estimates
        scale = 300.0
    if what == "per channel":
        f = f[0].copy()
        f[at[0]] = np.float32(-0.0)
    else:
        some = rng.random((N, K // 16)) < 0.5       # blocks with and without one in the same wave
        np.put_along_axis(f, at, np.where(some, np.float32(-0.0), np.take_along_axis(f, at, 1)), 1)
        f[:, 32:48] = np.float32(-0.0)              # a whole block
    assert (np.signbit(f) & (f == 0)).any()
    _assert_clipped_as_by_the_oracle(w, f, float(synth.default_tensor_scale(w)) * scale)


@pytest.mark.parametrize("sensitivity", [1.0, 1e-14, 1e-16, 1e-18])
@pytest.mark.parametrize("noise", [1e-3, 1e-4])
def test_clipped_scales_of_nearly_reproduced_blocks_are_the_brute_force_ones(noise, sensitivity):
    """Values nearly 4, 2 and 1 times some scale: codes an octave apart are all off by the noise alone, far below the error under
    code 0 that an estimate's distance grows with; with small sensitivities the product of the two errors is no FP32 number."""
    rng = synth.rng_for(39, int(-np.log10(noise)))
    N, K = 128, 1024
    code = rng.integers(40, 100, (N, K // 16))
    S = np.float32(0.015)
    base = np.repeat(4.0 * (1.0 + code % 8 / 8.0) * 2.0 ** (code // 8 - 7.0) * float(S), 16, axis=1)
    w = base * rng.choice([1.0, 0.5, 0.25, -1.0, -0.5, -0.25], (N, K)) * (1.0 + noise * rng.standard_normal((N, K)))
    f = np.exp(rng.standard_normal((N, K))) * sensitivity
    _assert_clipped_as_by_the_oracle(w.astype(np.float32), f.astype(np.float32), float(S))


@pytest.mark.parametrize("share", [1.0, 0.98, 0.5, 0.02])
def test_clipped_scales_of_blocks_with_equal_errors_are_the_brute_force_ones(share):
    """Values of +-12 times a power of two and one small one: seven scales of the same error, more than are compared one by one.
    All 64 blocks of a wave, nearly all of them, half and one of them; the others are ordinary ones."""
    rng = synth.rng_for(40, int(100 * share))
    N, K = 72, 528
    w = 6.0 * rng.standard_normal((N, K))
    f = np.exp(rng.standard_normal((N, K)))
    tied = np.repeat(rng.random((N, K // 16)) < share, 16, axis=1)
    w[tied] = (12.0 * 2.0 ** np.repeat(rng.integers(-2, 3, (N, K // 16)), 16, axis=1) * rng.choice([-1.0, 1.0], (N, K)))[tied]
    w[:, 5::16] = 0.01
    _assert_clipped_as_by_the_oracle(w.astype(np.float32), f.astype(np.float32), 2.0 ** -3)


# ------------------------------------------------------------------ decode steps: the last row group with one row-tile

# (M, K, N), N / 8 rounded up odd: one, eight, sixteen and 32 rows; K in one part and in several; a last row-tile of one row
@pytest.mark.parametrize("M,K,N,dtype,p", [(1, 5840, 40, "bf16", 0.2), (8, 4112, 1001, "f32", 0.1), (16, 1040, 1000, "bf16", 1.0),
                                           (5, 272, 4353, "bf16", 0.0), (32, 4832, 1315, "f32", 0.2), (9, 8192, 72, "bf16", 0.1),
                                           (25, 14816, 1287, "bf16", 0.1)])
def test_decode_steps_with_an_odd_number_of_row_tiles_match_oracle(M, K, N, dtype, p):
    """Within 1e-5 of the sum of magnitudes; whatever lies behind the last row-tile's bytes must not show."""
    from paper_2504_14152_amd import build
    assert fgmp.selftest_gemm_route(M, N, K)[0] == 0
    xd, fxd, Tx, sx, pW, want, tol = _product(M, K, N, dtype, p, 96 + M)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(M, N, K), DEV)
    ws[fgmp.WORKSPACE_CONTROL_BYTES:] = 0xFF
    out = torch.full((M + 1, N + 3), 7.0, device=DEV)
    Y = fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, out=out[:M, :N], workspace=ws).clone()
    err = np.abs(Y.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= tol), (err / tol).max()
    assert bool((out[M] == 7.0).all()) and bool((out[:, N:] == 7.0).all())
    assert int(ws[: fgmp.WORKSPACE_CONTROL_BYTES].sum()) == 0
    assert torch.equal(fgmp.gemm(fgmp.quantize_activations(xd, fxd, Tx, sx), pW), Y)
    used = fgmp.packed_info(pW)["bytes_used"]
    exact = torch.full((-(-used // 16) * 16 + 4096,), 0xFF, dtype=torch.uint8, device=DEV)   # poison right behind the tensor
    exact[:used] = pW.buf[:used]
    assert torch.equal(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, fgmp.Packed(exact[:used], N, K)), Y)
    with fgmp.use_library(build.lib_path("fullwait")):
        assert torch.equal(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW), Y)


# one row-tile and three, the last of one row and of eight; the smallest K, K in one part and in several
@pytest.mark.parametrize("M,K,N", [(1, 16, 1), (8, 1024, 24), (1, 5840, 8), (16, 8192, 17), (32, 4832, 24), (5, 272, 3)])
def test_decode_steps_over_one_and_three_row_tiles_match_oracle(M, K, N):
    assert fgmp.selftest_gemm_route(M, N, K)[0] == 0
    xd, fxd, Tx, sx, pW, want, tol = _product(M, K, N, "f32", 0.2, 101)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(M, N, K), DEV)
    ws[fgmp.WORKSPACE_CONTROL_BYTES:] = 0xFF
    Y = fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, workspace=ws).clone()
    err = np.abs(Y.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= tol), (err / tol).max()
    assert int(ws[: fgmp.WORKSPACE_CONTROL_BYTES].sum()) == 0
    assert torch.equal(fgmp.gemm(fgmp.quantize_activations(xd, fxd, Tx, sx), pW), Y)
    got = torch.full((M, N), float("nan"), device=DEV)
    fgmp.quant_gemm_fused_static_scratch(xd, fxd, Tx, sx, pW, out=got)
    assert torch.equal(got, Y)
    used = fgmp.packed_info(pW)["bytes_used"]
    exact = torch.full((-(-used // 16) * 16 + 4096,), 0xFF, dtype=torch.uint8, device=DEV)   # poison right behind the tensor
    exact[:used] = pW.buf[:used]
    assert torch.equal(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, fgmp.Packed(exact[:used], N, K)), Y)


# ------------------------------------------------------------------ prefill results whose rows do not start on a cache line

# more than 16 MB of results (ordinary stores) and less (streaming ones), both with rows that start anywhere
@pytest.mark.parametrize("M,K,N", [(4100, 48, 1033), (4100, 48, 777)])
def test_prefill_results_in_rows_of_any_alignment_match_oracle(M, K, N):
    xd, fxd, Tx, sx, pW, want, tol = _product(M, K, N, "bf16", 0.1, 97)
    assert fgmp.selftest_gemm_route(M, N, K)[0] == 3
    out = torch.full((M, N + 1), 7.0, device=DEV)
    Y = fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, out=out[:, :N])
    err = np.abs(Y.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= tol), (err / tol).max()
    assert bool((out[:, N] == 7.0).all())
    assert torch.equal(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW), Y)


# rows that start on half lines, up to 40 MB (streaming stores) and beyond (ordinary ones)
@pytest.mark.parametrize("M,K,N", [(2257, 320, 3888), (2947, 256, 4016)])
def test_prefill_results_in_rows_on_half_lines_are_those_of_whole_lines(M, K, N):
    assert fgmp.selftest_gemm_route(M, N, K)[0] == 3 and N % 32 == 16
    g = torch.Generator(device=DEV).manual_seed(M)
    x, w = torch.randn(M, K, generator=g, device=DEV), torch.randn(N, K, generator=g, device=DEV)
    f = torch.ones(K, device=DEV)
    pW = fgmp.quantize_weights(w, f, 0.1, 0.01)
    whole, half = torch.full((M, N + 16), 7.0, device=DEV), torch.full((M, N + 32), 7.0, device=DEV)
    Y = fgmp.quant_gemm_fused(x, f, 0.1, 0.01, pW, out=whole[:, :N])
    assert torch.equal(fgmp.quant_gemm_fused(x, f, 0.1, 0.01, pW, out=half[:, :N]), Y) and float(Y.std()) > 1.0
    assert bool((whole[:, N:] == 7.0).all()) and bool((half[:, N:] == 7.0).all())


# ------------------------------------------------------------------ selecting thresholds: states that calls borrow

def test_more_selections_at_a_time_than_there_are_states_are_exact():
    """Twelve threads on streams of their own, eight states; and a selection refused under capture leaves everything usable."""
    import threading
    gen = torch.Generator(device=DEV).manual_seed(98)
    scores = [torch.randn(20011 + 4096 * i, generator=gen, device=DEV) ** 2 for i in range(12)]
    want = [orc.threshold(s.cpu().numpy(), 0.1) for s in scores]
    got = [[] for _ in scores]

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                got[i].append(fgmp.threshold_for_fraction(scores[i], 0.1))

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(scores))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(g == [w] * 20 for g, w in zip(got, want))
    g, x = torch.cuda.CUDAGraph(), torch.zeros(4, device=DEV)
    with torch.cuda.graph(g):
        x.add_(1.0)
        with pytest.raises(fgmp.FgmpError):
            fgmp.threshold_for_fraction(scores[0], 0.1)
    g.replay()
    torch.cuda.synchronize()
    assert bool((x == 1.0).all()) and fgmp.threshold_for_fraction(scores[0], 0.1) == want[0]


# ------------------------------------------------------------------ packing weights with no block in FP8

@pytest.mark.parametrize("rows,K", [(1, 16), (9, 144), (520, 2064)])
@pytest.mark.parametrize("clip", [False, True])
def test_weights_packed_with_an_infinite_threshold_hold_no_upper_half(rows, K, clip):
    """Written in one pass; the same bytes as with a threshold that no score exceeds, in a buffer that held something else."""
    g = torch.Generator(device=DEV).manual_seed(rows + K)
    w = torch.randn(rows, K, generator=g, device=DEV)
    f = torch.exp(torch.randn(rows, K, generator=g, device=DEV))
    s = float(w.abs().max()) / 448.0
    pack = fgmp.quantize_weights_clip if clip else fgmp.quantize_weights
    bufs = [torch.full((fgmp.packed_bytes(rows, K),), v, dtype=torch.uint8, device=DEV) for v in (0xA5, 0xA5)]
    for buf, T in zip(bufs, (float("inf"), 3.0e38)):
        pack(w, f, T, s, out=fgmp.Packed(buf, rows, K))
    assert torch.equal(*bufs)
    assert fgmp.packed_info(fgmp.Packed(bufs[0], rows, K))["n_fp8_blocks"] == 0


# ------------------------------------------------------------------ the same with K in fewer parts than would be fastest

@pytest.mark.parametrize("M,K,N", [(497, 9744, 385), (439, 9616, 507)])
def test_long_products_in_the_parts_that_have_room_match_oracle(M, K, N):
    """In a workspace of the size a call is told, and on the static scratch array; with its control region left zero."""
    assert fgmp.selftest_gemm_route(M, N, K)[0] == 2
    xd, fxd, Tx, sx, pW, want, tol = _product(M, K, N, "bf16", 0.1, 98)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(M, N, K), DEV)
    ws[fgmp.WORKSPACE_CONTROL_BYTES:] = 0xFF
    Y = fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, workspace=ws).clone()
    err = np.abs(Y.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= tol), (err / tol).max()
    assert int(ws[: fgmp.WORKSPACE_CONTROL_BYTES].sum()) == 0
    assert torch.equal(fgmp.gemm(fgmp.quantize_activations(xd, fxd, Tx, sx), pW, workspace=ws), Y)
    got = torch.full((M, N), float("nan"), device=DEV)
    fgmp.quant_gemm_fused_static_scratch(xd, fxd, Tx, sx, pW, out=got)
    assert torch.equal(got, Y)


# ------------------------------------------------------------------ the kernel for mid-size products above 1024 rows

# (M, K, N): few columns; a last tile of a few rows, K shared among workgroups;
# more tiles than run at once; the most rows it takes
@pytest.mark.parametrize("M,K,N", [(1301, 272, 264), (1545, 3088, 320), (2500, 144, 1408), (4096, 528, 136)])
def test_mid_size_kernel_above_1024_rows_matches_oracle(M, K, N):
    """Plain, packed and gated calls, in a workspace of the size that a call is told and with its control region left zero."""
    from paper_2504_14152_amd import build
    assert fgmp.selftest_gemm_route(M, N, K)[0] == 2
    xd, fxd, Tx, sx, pW, want, tol = _product(M, K, N, "bf16", 0.1, 99)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(M, N, K), DEV)
    ws[fgmp.WORKSPACE_CONTROL_BYTES:] = 0xFF
    Y = fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, workspace=ws).clone()
    err = np.abs(Y.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= tol), (err / tol).max()
    assert int(ws[: fgmp.WORKSPACE_CONTROL_BYTES].sum()) == 0
    assert torch.equal(fgmp.gemm(fgmp.quantize_activations(xd, fxd, Tx, sx), pW, workspace=ws), Y)
    with fgmp.use_library(build.lib_path("fullwait")):
        assert torch.equal(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW), Y)
    f_n = torch.from_numpy(synth.fisher_per_channel(N, 99, 5)).to(DEV)
    s_y = float(Y.abs().max()) / 448.0
    for epilogue in (fgmp.EPILOGUE_NONE, fgmp.EPILOGUE_SILU_GATE)[: 2 if N % 64 == 0 else 1 if N % 16 == 0 else 0]:
        h = torch.from_numpy(orc.gate_columns(Y.cpu().numpy())).to(DEV) if epilogue else Y
        f_h = f_n[: h.shape[1]].contiguous()
        ref = fgmp.unpack_canonical(fgmp.quantize_activations(h.contiguous(), f_h, 1e-4, s_y))
        got = fgmp.unpack_canonical(fgmp.quant_gemm_fused_packed_out(xd, fxd, Tx, sx, pW, f_h, 1e-4, s_y, epilogue=epilogue))
        assert all(torch.equal(a, b) for a, b in zip(got, ref))


# ------------------------------------------------------------------ gated products in a workspace of just the size

# staged for a decode step, with K in parts, and for the mid-size kernel; in the prefill kernel's epilogue
@pytest.mark.parametrize("M,K,N", [(9, 1024, 192), (16, 8192, 128), (200, 512, 320), (4100, 272, 320)])
def test_gated_products_stay_within_the_workspace_they_are_told(M, K, N):
    xd, fxd, Tx, sx, pW, _, _ = _product(M, K, N, "bf16", 0.1, 102)
    f_h = torch.ones(N // 2, device=DEV)
    size = fgmp.workspace_bytes_packed_out(M, N, K, fgmp.EPILOGUE_SILU_GATE)
    assert size == fgmp.workspace_bytes_packed_out(M, N, K, fgmp.EPILOGUE_NONE)
    room = fgmp.new_workspace(size + 65536, DEV)
    room[fgmp.WORKSPACE_CONTROL_BYTES:] = 0xA5
    got = fgmp.quant_gemm_fused_packed_out(xd, fxd, Tx, sx, pW, f_h, 1e-4, 0.05, workspace=room[:size], epilogue=fgmp.EPILOGUE_SILU_GATE)
    assert bool((room[size:] == 0xA5).all())
    h = torch.from_numpy(orc.gate_columns(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW).cpu().numpy())).to(DEV)
    for a, b in zip(fgmp.unpack_canonical(got), fgmp.unpack_canonical(fgmp.quantize_activations(h.contiguous(), f_h, 1e-4, 0.05))):
        assert torch.equal(a, b)


# ------------------------------------------------------------------ decode steps: K shared among more than four workgroups

# (M, K): 5, 6, 7 and 13 parts, added up six at a time; 5, 8, 11 and 16 parts, four at a time
@pytest.mark.parametrize("M,K", [(16, 10128), (9, 12288), (16, 12304), (13, 26000), (32, 5008), (17, 8192), (32, 11008), (29, 16384)])
def test_decode_steps_in_many_parts_match_oracle(M, K):
    N = 48
    assert fgmp.selftest_gemm_route(M, N, K)[0] == 0
    xd, fxd, Tx, sx, pW, want, tol = _product(M, K, N, "bf16", 0.1, 100 + M)
    ws = fgmp.new_workspace(fgmp.workspace_bytes(M, N, K), DEV)
    ws[fgmp.WORKSPACE_CONTROL_BYTES:] = 0xFF       # partial sums start as NaN patterns
    Y = fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, workspace=ws).clone()
    err = np.abs(Y.cpu().numpy().astype(np.float64) - want)
    assert np.all(err <= tol), (err / tol).max()
    assert int(ws[: fgmp.WORKSPACE_CONTROL_BYTES].sum()) == 0
    for _ in range(4):
        assert torch.equal(fgmp.quant_gemm_fused(xd, fxd, Tx, sx, pW, workspace=ws), Y)
