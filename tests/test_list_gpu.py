"""GPU parity of the streaming list forward (lb_list_init / lb_list_forward).

Lists of linears of at most two tokens run on the look-up-table kernels: every
linear must give bit for bit what the single-launch look-up-table decode kernel
gives for it (lb_linear_forward_kernel(..., LB_KERNEL_DECODE)) and meet the oracle
bar.  Lists with a linear of more than two tokens run on the matrix-core kernels:
every token of every linear meets the oracle bar of the forward (fp32: relative L2
<= 1e-5; bf16 / f16: max relative error <= 1e-2 per token row), and repeated calls
give the same bits.  Lists mix ragged shapes (tails of d_in, r and d_out, ranks that
are not a multiple of 64 or 16, token counts that are not a multiple of 16), runs
of one and of several blocks, empty linears; the plan check, graph replays and the
Llama2-70B layer shapes are covered for both kinds."""
import numpy as np
import pytest

from paper_2506_13771_amd import synth
import lbtest_utils as U
from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch
    import paper_2506_13771_amd as lb

from test_parity_gpu import _check


def _linears(specs, cfg, act="bf16", sc="f16", direct=False):
    out = []
    for i, (T, d_in, d_out, r) in enumerate(specs):
        li = synth.make_linear(d_in, d_out, r, T, act_dtype=act, scale_dtype=sc, cfg=cfg, linear=i,
                               direct_words=direct)
        x, paths, _ = U.to_device(li)
        out.append((li, x, paths))
    return out


def _decode_single(lins):
    out = []
    for li, x, paths in lins:
        out.append(lb.lb_linear_forward(x, paths, li.r, kernel=lb.LB_KERNEL_DECODE))
    torch.cuda.synchronize()
    return out


def _same_bits(a, b):
    if a.numel() == 0:
        return b.numel() == 0
    v = torch.int16 if a.element_size() == 2 else torch.int32
    return torch.equal(a.view(v), b.view(v))


def _run_list(lins):
    L = lb.LittleBitList([(x, paths, li.r, None) for li, x, paths in lins])
    ys = L.forward()
    torch.cuda.synchronize()
    return L, ys


RAGGED = [(1, 100, 77, 19), (2, 33, 200, 50), (1, 257, 130, 16), (2, 31, 64, 1), (1, 70, 45, 33),
          (2, 1000, 999, 96), (1, 96, 4100, 48), (1, 1, 1, 1), (2, 4000, 300, 200), (1, 5000, 700, 80),
          (1, 2048, 640, 130), (2, 700, 64, 64), (1, 6500, 2000, 288), (2, 3000, 1500, 176)]


@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f32", "f32"), ("f16", "bf16"), ("bf16", "bf16")])
def test_list_ragged_bit_identical_to_decode(act, sc):
    lins = _linears(RAGGED, cfg=40, act=act, sc=sc)
    # scales of both signs: nothing may assume positive scales
    for j, (li, x, paths) in enumerate(lins):
        rs = np.random.default_rng(j)
        for p in range(2):
            li.h[p] = synth.quantize(rs.standard_normal(li.d_out), sc)
            li.g[p] = synth.quantize(rs.standard_normal(li.d_in), sc)
            li.l[p] = synth.quantize(rs.standard_normal(li.r), sc)
            paths[p].h.copy_(U.raw_to_torch(li.h[p], sc))
            paths[p].g.copy_(U.raw_to_torch(li.g[p], sc))
            paths[p].l.copy_(U.raw_to_torch(li.l[p], sc))
    ref = _decode_single(lins)
    L, ys = _run_list(lins)
    for i, ((li, _, _), y, r) in enumerate(zip(lins, ys, ref)):
        assert _same_bits(y, r), (i, RAGGED[i], act, sc)
        _check(li, U.torch_to_raw(y, act), label=f"list {RAGGED[i]} {act}/{sc}")
    assert lb.lb_workspace_status(L.workspace) == 0


def test_list_llama2_70b_layer_shapes():
    """One Llama2-70B layer at 0.1 bits per weight (q, k, v, o, gate, up, down), one token."""
    ranks = {(8192, 8192): 176, (8192, 1024): 16, (8192, 28672): 288, (28672, 8192): 288}
    specs = [(1, d_in, d_out, ranks[(d_in, d_out)]) for _, d_in, d_out in synth.LLAMA2_70B]
    lins = _linears(specs, cfg=4, direct=True)
    ref = _decode_single(lins)
    L, ys = _run_list(lins)
    for i, ((li, _, _), y, r) in enumerate(zip(lins, ys, ref)):
        assert _same_bits(y, r), (i, specs[i])
        _check(li, U.torch_to_raw(y, "bf16"), label=f"70b list {specs[i]}")
    # repeated forwards give the same bits
    for _ in range(3):
        again = L.forward()
        torch.cuda.synchronize()
        for y, r in zip(again, ref):
            assert _same_bits(y, r)


def test_list_empty_members():
    specs = [(1, 512, 384, 32), (1, 64, 64, 16), (2, 300, 200, 40)]
    lins = _linears(specs, cfg=41)
    items = [(x, paths, li.r, None) for li, x, paths in lins]
    # an empty reduction (d_in = 0 and r = 0) gives y = 0; T = 0 and d_out = 0 are skipped
    dev = "cuda"
    zx = torch.empty((3, 0), dtype=torch.bfloat16, device=dev)
    zpaths = [lb.LittleBitPath(U=torch.zeros(64, dtype=torch.uint8, device=dev), V=None,
                               h=torch.ones(16, dtype=torch.float16, device=dev), g=None,
                               l=torch.ones(4, dtype=torch.float16, device=dev)) for _ in range(2)]
    y_empty = torch.full((3, 16), 7.0, dtype=torch.bfloat16, device=dev)
    items.insert(1, (zx, zpaths, 4, y_empty))
    t0x = torch.empty((0, 64), dtype=torch.bfloat16, device=dev)
    items.append((t0x, lins[1][2], 16, None))
    L = lb.LittleBitList(items)
    ys = L.forward()
    torch.cuda.synchronize()
    ref = _decode_single(lins)
    assert _same_bits(ys[0], ref[0]) and _same_bits(ys[2], ref[1]) and _same_bits(ys[3], ref[2])
    assert torch.count_nonzero(y_empty.float()) == 0
    assert ys[4].numel() == 0


def test_list_plan_mismatch_computes_nothing():
    lins = _linears([(1, 512, 384, 32), (1, 640, 256, 48)], cfg=42)
    L, ys = _run_list(lins)
    before = [y.clone() for y in ys]
    # a descriptor array whose output pointer differs from the plan's
    other = torch.full_like(ys[0], 3.0)
    arr, _ = lb.make_descs([(x, paths, li.r, other if i == 0 else ys[i]) for i, (li, x, paths) in enumerate(lins)])
    st = lb.load_library().lb_list_forward(arr, 2, L.workspace.data_ptr(), L.workspace.numel(),
                                           torch.cuda.current_stream().cuda_stream)
    assert st == lb.LB_OK
    torch.cuda.synchronize()
    assert torch.all(other == 3.0)
    assert all(torch.equal(a, b) for a, b in zip(before, ys))
    assert lb.lb_workspace_status(L.workspace) == 2
    assert lb.lb_workspace_status(L.workspace) == 0
    # the matching descriptors still work
    again = L.forward()
    torch.cuda.synchronize()
    assert all(_same_bits(a, b) for a, b in zip(again, before))


def test_list_graph_replays_match_eager():
    specs = [(1, 2048, 1536, 64), (1, 1024, 4096, 80), (2, 512, 512, 32), (1, 8192, 1024, 16), (2, 3000, 700, 130)]
    lins = _linears(specs, cfg=43)
    L, ys = _run_list(lins)
    y_eager = [y.clone() for y in ys]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        L.forward()
    for rep in range(4):
        for y in ys:
            y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for i in range(len(lins)):
            assert _same_bits(ys[i], y_eager[i]), (rep, i)
        # eager work on the same workspace between replays
        L.forward()
        torch.cuda.synchronize()
        for i in range(len(lins)):
            assert _same_bits(ys[i], y_eager[i]), (rep, i)


# ---------------------------------------------------------------------------
# lists with linears of more than two tokens: the matrix-core kernels (every
# linear of such a list, whatever its own token count); parity with the oracle
# at the forward's bar, every token compared
# ---------------------------------------------------------------------------
RAGGED_MMA = [(3, 100, 77, 19), (8, 36, 200, 50), (16, 256, 130, 16), (17, 32, 64, 1), (64, 1000, 999, 96),
              (33, 96, 4100, 48), (1, 4, 1, 1), (8, 4000, 300, 200), (5, 5000, 700, 80), (64, 2048, 640, 130),
              (2, 700, 64, 64), (48, 6500, 2000, 288), (8, 3000, 1500, 176), (64, 4096, 4096, 1024)]


@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f32", "f32"), ("f16", "bf16"), ("bf16", "bf16")])
def test_mma_list_ragged_matches_oracle(act, sc):
    lins = _linears(RAGGED_MMA, cfg=44, act=act, sc=sc)
    for j, (li, x, paths) in enumerate(lins):
        rs = np.random.default_rng(100 + j)
        for p in range(2):
            li.h[p] = synth.quantize(rs.standard_normal(li.d_out), sc)
            li.g[p] = synth.quantize(rs.standard_normal(li.d_in), sc)
            li.l[p] = synth.quantize(rs.standard_normal(li.r), sc)
            paths[p].h.copy_(U.raw_to_torch(li.h[p], sc))
            paths[p].g.copy_(U.raw_to_torch(li.g[p], sc))
            paths[p].l.copy_(U.raw_to_torch(li.l[p], sc))
    L, ys = _run_list(lins)
    for i, ((li, _, _), y) in enumerate(zip(lins, ys)):
        _check(li, U.torch_to_raw(y, act), label=f"mma list {RAGGED_MMA[i]} {act}/{sc}")
    assert lb.lb_workspace_status(L.workspace) == 0
    # repeated forwards give the same bits (fixed summation order)
    again = L.forward()
    torch.cuda.synchronize()
    assert all(_same_bits(a, b) for a, b in zip(again, ys))


@pytest.mark.parametrize("T", [8, 64])
def test_mma_list_llama2_70b_layer_shapes(T):
    """One Llama2-70B layer at 0.1 bits per weight (q, k, v, o, gate, up, down), T tokens."""
    ranks = {(8192, 8192): 176, (8192, 1024): 16, (8192, 28672): 288, (28672, 8192): 288}
    specs = [(T, d_in, d_out, ranks[(d_in, d_out)]) for _, d_in, d_out in synth.LLAMA2_70B]
    lins = _linears(specs, cfg=5, direct=True)
    L, ys = _run_list(lins)
    for i, ((li, _, _), y) in enumerate(zip(lins, ys)):
        _check(li, U.torch_to_raw(y, "bf16"), label=f"70b mma list {specs[i]}")
    assert lb.lb_workspace_status(L.workspace) == 0


def test_mma_list_plan_mismatch_and_graph_replays():
    specs = [(8, 2048, 1536, 64), (64, 1024, 4096, 80), (3, 512, 512, 32)]
    lins = _linears(specs, cfg=45)
    L, ys = _run_list(lins)
    y_eager = [y.clone() for y in ys]
    other = torch.full_like(ys[0], 3.0)
    arr, _ = lb.make_descs([(x, paths, li.r, other if i == 0 else ys[i]) for i, (li, x, paths) in enumerate(lins)])
    st = lb.load_library().lb_list_forward(arr, len(specs), L.workspace.data_ptr(), L.workspace.numel(),
                                           torch.cuda.current_stream().cuda_stream)
    assert st == lb.LB_OK
    torch.cuda.synchronize()
    assert torch.all(other == 3.0)
    assert lb.lb_workspace_status(L.workspace) == 2
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        L.forward()
    for rep in range(3):
        for y in ys:
            y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for i in range(len(lins)):
            assert _same_bits(ys[i], y_eager[i]), (rep, i)
        L.forward()
        torch.cuda.synchronize()
        for i in range(len(lins)):
            assert _same_bits(ys[i], y_eager[i]), (rep, i)
    assert lb.lb_workspace_status(L.workspace) == 0


# (T, d_in, d_out, r): ranks at the edges of the 2-, 3-, 5- and 6-or-8-tile classes of a wave and of one and two
# groups of them; output rows around the 256- and 512-row workgroups; tails of d_in of 4, 12, 20 and 28 inputs (rows that
# are and are not whole 16-byte pieces); runs of one block, of a chunk and of several
EDGE_MMA = [(3, 36, 511, 128), (16, 100, 513, 129), (9, 2588, 64, 192), (4, 1000, 36, 193), (16, 268, 20, 320),
            (7, 524, 257, 321), (12, 96, 1, 512), (5, 4092, 40, 513), (32, 316, 255, 384), (17, 64, 256, 640),
            (48, 200, 130, 289), (33, 44, 300, 385), (64, 2060, 257, 577), (49, 24, 12, 1024)]


@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f32", "f16"), ("f16", "f32"), ("f32", "bf16")])
def test_mma_list_tile_edges(act, sc):
    lins = _linears(EDGE_MMA, cfg=45, act=act, sc=sc)
    L, ys = _run_list(lins)
    first = [y.clone() for y in ys]
    for i, ((li, _, _), y) in enumerate(zip(lins, ys)):
        _check(li, U.torch_to_raw(y, act), label=f"mma list {EDGE_MMA[i]} {act}/{sc}")
    # the loads run ahead of their use: a second pass over other buffer contents gives the same bits
    for y in ys:
        y.zero_()
    L.forward()
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(first, ys))


# ---------------------------------------------------------------------------
# matrix-core plans of longer lists: what they choose is computed here as the library's comments state it
# ---------------------------------------------------------------------------
def _classes(T):
    tt = (T + 15) // 16
    return tt, (2, 3, 5, 8 if tt <= 2 else 6)


def _plan(specs):
    """(blocks per run, S1 workgroups, latent tiles computed with a class per linear, with one class per token tile count)"""
    for bpr in (64, 32, 16, 8):
        n1, per, largest = 0, [], {}
        for T, d_in, _, r in specs:
            tt, cls = _classes(T)
            nmf, nbt = -(-r // 16), -(-d_in // 32)
            ng = -(-nmf // (4 * cls[-1]))
            mt = next(c for c in cls if c >= -(-nmf // (4 * ng)))
            n = 2 * ng * -(-nbt // bpr)
            n1 += n
            per.append((n, tt, mt))
            largest[tt] = max(largest.get(tt, 0), mt)
        if n1 >= 1024 or bpr == 8:
            return bpr, n1, sum(n * m for n, _, m in per), sum(n * largest[t] for n, t, _ in per)


# (T, d_in, d_out, r) of every token tile count, rows of d_in past 2048 with tails; the first fills stage 2 (512 workgroups of
# 512 rows) when the list is long
LONG = [(5, 4100, 10000, 100), (16, 2052, 70, 513), (31, 2076, 130, 321), (48, 4108, 65, 385), (64, 2060, 257, 577)]


@pytest.mark.parametrize("bpr,copies", [(64, 27), (32, 20), (16, 12), (8, 2)])
@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f32", "f32")])
def test_mma_list_run_lengths(bpr, copies, act, sc):
    assert _plan(LONG * copies)[0] == bpr
    lins = _linears(LONG, cfg=46, act=act, sc=sc)
    # copies of the linears with outputs of their own: the first is checked, the others have its bits
    L, ys = _run_list(lins * copies)
    for i, (li, _, _) in enumerate(lins):
        tokens = None if li.T <= 16 else np.arange(0, li.T, 5)
        _check(li, U.torch_to_raw(ys[i], act), tokens=tokens, label=f"mma list {LONG[i]} x{copies} {act}/{sc}")
        for c in range(1, copies):
            assert _same_bits(ys[i], ys[c * len(LONG) + i]), (LONG[i], c)


@pytest.mark.parametrize("T", [3, 17, 33, 49])
@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f32", "f32")])
def test_mma_list_class_launches(T, act, sc):
    # many linears of few latents beside some of many: a launch of stage 1 per class; one of them alone: one launch
    wide = [(T, 96, 40, 192), (T, 100, 41, 320), (T, 64, 42, 512 if T <= 32 else 384)]
    for specs, apart in (([(T, 96, 33, 16), (T, 68, 30, 33)] * 4 + wide, True), (wide, False)):
        _, _, tiles, tiles_one = _plan(specs)
        assert (tiles_one > 2 * tiles) == apart
        lins = _linears(specs, cfg=47, act=act, sc=sc)
        _, ys = _run_list(lins)
        for i, ((li, _, _), y) in enumerate(zip(lins, ys)):
            _check(li, U.torch_to_raw(y, act), label=f"mma list {specs[i]} {act}/{sc}")


# runs of 64 blocks at every token tile count
LONG_RUNS = [(5, 8192, 1000, 100), (16, 4096, 640, 513), (31, 4096, 640, 321), (48, 8192, 320, 385), (64, 8192, 320, 385)]


def test_mma_list_long_runs_keep_fp32_sums():
    """A run's length must not cost precision: in fp32 a list of 64-block runs lies at most 1.25
    times as far from the oracle as the prefill kernels, which add the same products in shorter
    sums (measured: 0.8 to 1.17; with the sums of 16 blocks in one accumulator 1.29)."""
    copies = 40
    assert _plan(LONG_RUNS * copies)[0] == 64
    lins = _linears(LONG_RUNS, cfg=48, act="f32", sc="f32")
    _, ys = _run_list(lins * copies)
    for i, (li, x, paths) in enumerate(lins):
        ref = U.oracle_forward(li, None)
        err = U.rel_l2(ys[i].double().cpu().numpy(), ref)
        pre = U.rel_l2(lb.lb_linear_forward(x, paths, li.r, kernel=lb.LB_KERNEL_PREFILL).double().cpu().numpy(), ref)
        assert err <= 1.25 * pre, (LONG_RUNS[i], err, pre)
