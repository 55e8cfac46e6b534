"""GPU parity: the HIP path (through the C ABI) against the fp64 oracle on the
same seeded inputs.

Bars: packing is bit-exact; fp32 activations must reach relative L2 <= 1e-5;
bf16 / f16 activations (fp32 accumulation) must reach max relative error
<= 1e-2 per token row (max_i |y - y*| / max_i |y*|).  Sizes span several
tiles and ragged tails; the benchmark shapes run at full size and every token
of every output is compared with the oracle.
"""
import numpy as np
import pytest

import oracle as O
from paper_2506_13771_amd import synth
import lbtest_utils as U
from conftest import gpu_available

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch
    import paper_2506_13771_amd as lb

KERNELS = {"decode": 1, "prefill": 2, "auto": 0, "mma": 3}
MMA_MAX_T, MMA_MAX_R = 64, 832


def _run(li, kernel="auto", pack_on_gpu=True):
    x, paths, _ = U.to_device(li, pack_on_gpu)
    y = lb.lb_linear_forward(x, paths, li.r, kernel=KERNELS[kernel])
    torch.cuda.synchronize()
    return U.torch_to_raw(y, li.act_dtype)


def _check(li, y_raw, tokens=None, label=""):
    ref = U.oracle_forward(li, tokens)
    y = O.to_f64(y_raw, li.act_dtype)
    if tokens is not None:
        y = y[tokens]
    assert np.all(np.isfinite(y)), label
    if li.act_dtype == "f32":
        err = U.rel_l2(y, ref)
        assert err <= U.TOL_F32_REL_L2, (label, err)
    else:
        err = U.row_inf_rel(y, ref)
        assert err <= U.TOL_BF16_ROW_INF, (label, err, U.rel_l2(y, ref))
    return err


# ---------------------------------------------------------------------------
# packing: bit-exact against the oracle packer
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("rows,r", [(512, 32), (4096, 80), (11008, 128), (4096, 544), (1024, 16), (33, 7),
                                    (40, 50), (100, 17), (1, 1), (64, 31)])
@pytest.mark.parametrize("dt", ["f32", "bf16", "f16"])
def test_pack_bit_exact(rows, r, dt):
    rs = np.random.default_rng(rows * 13 + r)
    src64 = rs.standard_normal((rows, r))
    src64[0, 0] = -0.0
    raw = synth.quantize(src64, dt)
    src_t = U.raw_to_torch(raw, dt)
    src_exact = O.to_f64(raw, dt)
    for role in (lb.LB_ROLE_U, lb.LB_ROLE_V):
        got = lb.lb_pack_signs(src_t, role)
        torch.cuda.synchronize()
        ref, _ = O.pack(src_exact, role)
        assert got.cpu().numpy().tobytes() == ref.tobytes(), (rows, r, dt, role)


@pytest.mark.parametrize("rows,r", [(1, 63), (15, 64), (16, 65), (17, 48), (31, 49), (48, 129), (49, 3)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_pack_tile_edges(rows, r, dt):
    # 16-row and 64-latent wave tiles, the 16- and 32-bit tail planes, NaNs and infinities in the last row and column;
    # the source is a view that starts one element into its buffer
    rs = np.random.default_rng(rows * 131 + r)
    src64 = rs.standard_normal((rows, r))
    src64[-1, -1] = np.nan
    src64[-1, 0] = -np.inf
    raw = synth.quantize(src64, dt)
    buf = torch.zeros(rows * r + 1, dtype=U.torch_dtype(dt), device="cuda")
    src_t = buf[1:].view(rows, r)
    src_t.copy_(U.raw_to_torch(raw, dt))
    for role in (lb.LB_ROLE_U, lb.LB_ROLE_V):
        cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
        got = lb.lb_pack_signs(src_t, role, nan_count=cnt)
        torch.cuda.synchronize()
        ref, nans = O.pack(O.to_f64(raw, dt), role)
        assert got.cpu().numpy().tobytes() == ref.tobytes(), (rows, r, dt, role)
        assert int(cnt.item()) == nans == 1


@pytest.mark.parametrize("rows,r", [(1, 1), (63, 1), (255, 2), (257, 5), (4097, 8), (1000, 15), (513, 16), (513, 17),
                                    (63, 9), (131072, 9), (131073, 16), (131135, 17), (131130, 31), (131136, 32), (131072, 33)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_pack_narrow_rows(rows, r, dt):
    # rows of up to 8 latents, or 32 from 131072 rows on (64 of them as one stream of elements), and the first that are not,
    # NaNs and infinities at the ends of rows
    rs = np.random.default_rng(rows + r)
    src64 = rs.standard_normal((rows, r))
    src64[-1, -1] = np.nan
    src64[0, 0] = -np.inf
    if rows > 2:
        src64[rows // 2, r - 1] = np.nan
    raw = synth.quantize(src64, dt)
    src_t = U.raw_to_torch(raw, dt)
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = lb.lb_pack_signs(src_t, lb.LB_ROLE_U, nan_count=cnt)
    ref, nans = O.pack(O.to_f64(raw, dt), O.ROLE_U)
    assert got.cpu().numpy().tobytes() == ref.tobytes()
    assert int(cnt.item()) == nans


@pytest.mark.parametrize("rows,r", [((1 << 30) + 5, 1), ((1 << 31) - 1, 1), (1, (1 << 31) - 33), (1, (1 << 31) - 1)])
@pytest.mark.parametrize("role", ["U", "V"])
def test_pack_sizes_near_the_limit(rows, r, role):
    # sizes whose tiles or threads do not fit 32 bits: element e of the other dimension's only one is bit e % 32 of word e / 32
    # (rows, r) = (n, 1) in role V and (1, n) in role U; in the other two every entry has one bit, 16 bits wide
    n = rows * r
    src = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
    where = torch.tensor([0, 1, 31, 32, 63, 64, n // 2, n - 65, n - 64, n - 34, n - 33, n - 17, n - 16, n - 2, n - 1], device="cuda")
    src[where] = -1.0
    dst = lb.lb_pack_signs(src.view(rows, r), {"U": lb.LB_ROLE_U, "V": lb.LB_ROLE_V}[role])
    del src
    if (rows == 1) == (role == "U"):
        nb, w = n // 32, n % 32
        full, tail = dst[:4 * nb].view(torch.int32), dst[4 * nb:].view(torch.int16 if w <= 16 else torch.int32)
        bits = [32 * i + b for v in (full,) for i in v.nonzero().flatten().tolist() for b in range(32) if (int(v[i]) >> b) & 1]
        bits += [32 * nb + b for b in range(w) if w and (int(tail[0]) >> b) & 1]
        assert bits == sorted(set(where.tolist()))
    else:
        v = dst.view(torch.int16)
        assert v.numel() == n
        at = torch.cat([s + k for k, s in ((k, v[k:k + (1 << 28)].nonzero().flatten()) for k in range(0, n, 1 << 28))])
        assert torch.equal(at, where.unique()) and bool((v[at] == 1).all())


def test_pack_nan_count():
    src = torch.randn(64, 48, device="cuda")
    src[3, 5] = float("nan")
    src[10, 40] = float("nan")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = lb.lb_pack_signs(src, lb.LB_ROLE_V, nan_count=cnt)
    torch.cuda.synchronize()
    assert int(cnt.item()) == 2
    ref, nans = O.pack(src.cpu().double().numpy(), O.ROLE_V)
    assert nans == 2 and got.cpu().numpy().tobytes() == ref.tobytes()


# ---------------------------------------------------------------------------
# forward: configuration 0 (512x512, r=32, T=4, fp32) on every kernel, and vs dense
# ---------------------------------------------------------------------------
def cfg0():
    return synth.make_linear(512, 512, 32, 4, act_dtype="f32", scale_dtype="f32", cfg=0, l_over_sqrt_r=True)


@pytest.mark.parametrize("kernel", ["decode", "prefill", "mma", "auto"])
def test_cfg0_fp32(kernel):
    li = cfg0()
    y = _run(li, kernel)
    _check(li, y, label=f"cfg0 {kernel}")
    # also against the brute-force dense reconstruction (Proposition 1 identity)
    Us, Vs, _, _ = U.oracle_signs(li)
    h, g, l = U.oracle_scales(li)
    Wd = O.dense_weight(Us, Vs, h, g, l)
    ref = O.dense_forward(O.to_f64(li.x, "f32"), Wd)
    assert U.rel_l2(O.to_f64(y, "f32"), ref) <= U.TOL_F32_REL_L2


def test_dense_reference_weight_cfg0():
    li = cfg0()
    x, paths, _ = U.to_device(li)
    W = lb.lb_dense_reference_weight(paths, li.d_in, li.d_out, li.r)
    torch.cuda.synchronize()
    Us, Vs, _, _ = U.oracle_signs(li)
    h, g, l = U.oracle_scales(li)
    ref = O.dense_weight(Us, Vs, h, g, l)
    err = np.abs(W.cpu().double().numpy() - ref).max() / np.abs(ref).max()
    assert err <= 1e-6, err


# ---------------------------------------------------------------------------
# configuration 1: Llama2-7B q_proj 4096x4096 at 0.1 BPW (r=80), T=1, bf16
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("kernel", ["auto", "prefill", "mma"])
def test_cfg1_q_proj(kernel):
    li = synth.make_linear(4096, 4096, 80, 1, cfg=1)
    _check(li, _run(li, kernel), label=f"cfg1 {kernel}")


# ---------------------------------------------------------------------------
# configuration 2: all 7 linears of a Llama2-7B block at 0.1 / 0.55 BPW, T in {1, 16, 64}
# ---------------------------------------------------------------------------
RANKS_7B = {0.1: {4096: 80, 11008: 128}, 0.55: {4096: 544, 11008: 800}}


def _rank_7b(bpw, d_in, d_out):
    return RANKS_7B[bpw][max(d_in, d_out)]


@pytest.mark.parametrize("bpw", [0.1, 0.55])
@pytest.mark.parametrize("T", [1, 16, 64])
def test_cfg2_llama2_7b_block(bpw, T):
    for li_idx, (name, d_in, d_out) in enumerate(synth.LLAMA2_7B):
        r = _rank_7b(bpw, d_in, d_out)
        assert lb.lb_rank_for_bpw(d_in, d_out, bpw, 16) == r
        li = synth.make_linear(d_in, d_out, r, T, cfg=2, linear=li_idx + (100 if bpw > 0.5 else 0))
        _check(li, _run(li), label=f"cfg2 {name} bpw={bpw} T={T}")


@pytest.mark.parametrize("T", [1, 2, 4])
def test_cfg2_both_kernels_agree_with_oracle(T):
    li = synth.make_linear(11008, 4096, 128, T, cfg=2, linear=50)
    for k in ("decode", "prefill", "mma"):
        _check(li, _run(li, k), label=f"down T={T} {k}")


@pytest.mark.parametrize("d_in,d_out,r", [(4096, 4096, 544), (11008, 4096, 800), (4096, 11008, 800),
                                          (8192, 28672, 288), (28672, 8192, 288), (8192, 1024, 16)])
@pytest.mark.parametrize("T", [1, 3])
def test_decode_large_rank_and_long_inputs(d_in, d_out, r, T):
    """Decode geometry extremes: two-level reduction (many d_in runs), 16 lanes per
    output row, several rows per lane."""
    li = synth.make_linear(d_in, d_out, r, T, cfg=11, linear=d_in + r, direct_words=True)
    _check(li, _run(li, "decode"), label=f"decode {d_in}x{d_out} r={r} T={T}")


@pytest.mark.parametrize("d_in,d_out,r", [(4096, 4096, 544), (11008, 4096, 800), (4096, 11008, 800),
                                          (8192, 28672, 288), (28672, 8192, 288), (8192, 1024, 16),
                                          (4000, 3000, 832)])
@pytest.mark.parametrize("T", [5, 16, 33, 64])
def test_mma_large_rank_and_long_inputs(d_in, d_out, r, T):
    """Matrix-core decode geometry extremes: many d_in runs (two-level sums), the
    largest rank it takes, 1 to 4 token fragments."""
    li = synth.make_linear(d_in, d_out, r, T, cfg=12, linear=d_in + r + T, direct_words=True)
    _check(li, _run(li, "mma"), label=f"mma {d_in}x{d_out} r={r} T={T}")


# ---------------------------------------------------------------------------
# configuration 3: Llama2-13B block shapes at 0.1 BPW, prefill T=2048
# ---------------------------------------------------------------------------
RANKS_13B = {(5120, 5120): 96, (5120, 13824): 160, (13824, 5120): 160}


@pytest.mark.parametrize("which", range(7))
def test_cfg3_llama2_13b_prefill(which):
    name, d_in, d_out = synth.LLAMA2_13B[which]
    r = RANKS_13B[(d_in, d_out)]
    li = synth.make_linear(d_in, d_out, r, 2048, cfg=3, linear=which)
    # every token: all 32 token tiles of 64 and every 16-token subtile of the MFMA path
    _check(li, _run(li), label=f"cfg3 {name}")


# ---------------------------------------------------------------------------
# configuration 4: Llama2-70B linear shapes at 0.1 BPW, T in {1, 8, 64}
# (packed words drawn directly, read by the oracle through its own unpacker)
# ---------------------------------------------------------------------------
RANKS_70B = {(8192, 8192): 176, (8192, 1024): 16, (8192, 28672): 288, (28672, 8192): 288}


@pytest.mark.parametrize("T", [1, 8, 64])
def test_cfg4_llama2_70b_shapes(T):
    for which, (name, d_in, d_out) in enumerate(synth.LLAMA2_70B):
        if name in ("k", "up", "o"):
            continue  # same shapes as v, gate and q
        r = RANKS_70B[(d_in, d_out)]
        li = synth.make_linear(d_in, d_out, r, T, cfg=4, linear=which, direct_words=True)
        _check(li, _run(li), label=f"cfg4 {name} T={T}")


# ---------------------------------------------------------------------------
# ragged shapes, dtypes, edge cases
# ---------------------------------------------------------------------------
RAGGED = [(100, 77, 19, 3), (33, 200, 50, 5), (257, 130, 16, 1), (31, 64, 1, 2), (70, 45, 33, 9),
          (1000, 999, 96, 16), (96, 4100, 48, 70), (1, 1, 1, 1), (5, 3, 2, 130)]


@pytest.mark.parametrize("d_in,d_out,r,T", RAGGED)
@pytest.mark.parametrize("kernel", ["decode", "prefill", "mma"])
@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f32", "f32"), ("f16", "bf16"), ("f16", "f32"),
                                    ("bf16", "bf16")])
def test_ragged(d_in, d_out, r, T, kernel, act, sc):
    if kernel == "decode" and T > lb.lb_decode_max_tokens():
        pytest.skip("decode kernel covers small T only")
    if kernel == "mma" and (T > MMA_MAX_T or r > MMA_MAX_R):
        pytest.skip("matrix-core decode kernel covers T <= 64, r <= 832")
    li = synth.make_linear(d_in, d_out, r, T, act_dtype=act, scale_dtype=sc, cfg=9,
                           linear=d_in * 7 + d_out * 3 + r + T)
    # scales of both signs: nothing in the kernels may assume positive scales
    rs = np.random.default_rng(d_in + d_out)
    for p in range(2):
        li.h[p] = synth.quantize(rs.standard_normal(d_out), sc)
        li.g[p] = synth.quantize(rs.standard_normal(d_in), sc)
        li.l[p] = synth.quantize(rs.standard_normal(r), sc)
    _check(li, _run(li, kernel), label=f"ragged {d_in}x{d_out} r={r} T={T} {kernel} {act}/{sc}")


@pytest.mark.parametrize("T,d_in,d_out,r", [(0, 64, 64, 16), (4, 0, 64, 16), (4, 64, 64, 0), (4, 64, 0, 16)])
@pytest.mark.parametrize("kernel", ["decode", "prefill", "mma", "auto"])
def test_degenerate_sizes(T, d_in, d_out, r, kernel):
    li = synth.make_linear(max(d_in, 1), max(d_out, 1), max(r, 1), max(T, 1), cfg=8)
    x = torch.randn(T, d_in, device="cuda").to(torch.bfloat16)
    paths = []
    for p in range(2):
        paths.append(lb.LittleBitPath(
            U=torch.zeros(max(lb.lb_packed_bytes(lb.LB_ROLE_U, d_out, r), 4), dtype=torch.uint8, device="cuda"),
            V=torch.zeros(max(lb.lb_packed_bytes(lb.LB_ROLE_V, d_in, r), 4), dtype=torch.uint8, device="cuda"),
            h=torch.ones(d_out, dtype=torch.float16, device="cuda"),
            g=torch.ones(d_in, dtype=torch.float16, device="cuda"),
            l=torch.ones(r, dtype=torch.float16, device="cuda")))
    y = torch.full((T, d_out), 7.0, dtype=torch.bfloat16, device="cuda")
    lb.lb_linear_forward(x, paths, r, y=y, kernel=KERNELS[kernel])
    torch.cuda.synchronize()
    assert torch.all(y == 0).item() or y.numel() == 0
    del li


def test_single_path_via_zero_residual_h():
    li = synth.make_linear(256, 192, 32, 3, cfg=7)
    li.h[1] = synth.quantize(np.zeros(192), "f16")
    y = _run(li)
    Us, Vs, _, _ = U.oracle_signs(li)
    h, g, l = U.oracle_scales(li)
    ref = O.forward_factored(O.to_f64(li.x, "bf16"), Us[:1], Vs[:1], h[:1], g[:1], l[:1])
    assert U.row_inf_rel(O.to_f64(y, "bf16"), ref) <= U.TOL_BF16_ROW_INF


def test_fp16_subnormal_scales_exact():
    """fp16 scales include subnormals; they must be widened exactly (fp32 activations)."""
    li = synth.make_linear(128, 128, 16, 2, act_dtype="f32", scale_dtype="f16", cfg=6)
    for p in range(2):
        g = li.g[p].copy()
        g[::7] = 0x0001 + (np.arange(g[::7].size) % 0x3FF).astype(np.uint16)  # subnormal fp16 patterns
        li.g[p] = g
    for k in ("decode", "prefill"):
        _check(li, _run(li, k), label=f"subnormal {k}")


# ---------------------------------------------------------------------------
# determinism and workspace reuse (counters must reset themselves)
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("T,kernel", [(1, "decode"), (1, "mma"), (16, "mma"), (64, "mma")])
def test_decode_bitwise_deterministic(T, kernel):
    li = synth.make_linear(4096, 4096, 80, T, cfg=1)
    x, paths, _ = U.to_device(li)
    ws = lb.alloc_workspace(T, 4096, 4096, 80)
    ys = []
    for _ in range(20):
        ys.append(lb.lb_linear_forward(x, paths, 80, workspace=ws, kernel=KERNELS[kernel]).clone())
    torch.cuda.synchronize()
    for y in ys[1:]:
        assert torch.equal(y.view(torch.int16), ys[0].view(torch.int16))


def test_workspace_reuse_across_shapes():
    shapes = [(1, 4096, 4096, 80), (16, 4096, 11008, 128), (3, 512, 512, 32), (100, 1000, 300, 48),
              (1, 4096, 4096, 80), (8, 11008, 4096, 800), (2, 700, 900, 17), (64, 2048, 2048, 64)]
    max_ws = max(lb.lb_forward_workspace_bytes(*s) for s in shapes)
    ws = torch.zeros(max_ws, dtype=torch.uint8, device="cuda")
    for rep in range(2):
        for i, (T, d_in, d_out, r) in enumerate(shapes):
            li = synth.make_linear(d_in, d_out, r, T, cfg=5, linear=i)
            x, paths, _ = U.to_device(li)
            y = lb.lb_linear_forward(x, paths, r, workspace=ws)
            torch.cuda.synchronize()
            tokens = None if T <= 16 else np.arange(0, T, 9)
            _check(li, U.torch_to_raw(y, "bf16"), tokens=tokens, label=f"reuse {i} rep {rep}")
    # the control block is back to its idle state (word 0 holds the decode call
    # tag; every counter and the error word are zero)
    ctrl_bytes = lb.lb_forward_workspace_bytes(0, 0, 0, 0)
    ctrl = ws[:ctrl_bytes].view(torch.int32)
    assert int(ctrl[0].item()) > 0
    assert int(ctrl[1:].abs().sum().item()) == 0


def test_back_to_back_launches_stress():
    """Many back-to-back decode launches with changing inputs on one workspace; every
    result checked against a GPU-side dense reference built by the checking kernel."""
    d_in, d_out, r, T = 1024, 1024, 48, 2
    li = synth.make_linear(d_in, d_out, r, T, cfg=4, linear=77)
    x0, paths, _ = U.to_device(li)
    W = lb.lb_dense_reference_weight(paths, d_in, d_out, r)
    ws = lb.alloc_workspace(T, d_in, d_out, r)
    g = torch.Generator(device="cuda").manual_seed(5)
    outs, xs = [], []
    for i in range(300):
        x = torch.randn(T, d_in, device="cuda", generator=g).to(torch.bfloat16)
        xs.append(x)
        outs.append(lb.lb_linear_forward(x, paths, r, workspace=ws))
    torch.cuda.synchronize()
    for x, y in zip(xs, outs):
        ref = x.float() @ W.t()
        err = ((y.float() - ref).abs().max(dim=1).values / ref.abs().max(dim=1).values).max().item()
        assert err <= U.TOL_BF16_ROW_INF, err


@pytest.mark.parametrize("T,kernel", [(1, "decode"), (4, "decode"), (16, "mma"), (100, "prefill")])
def test_graph_replays_match_eager(T, kernel):
    """Launches captured in a HIP graph: every replay (with eager work and syncs in
    between) must reproduce the eager result."""
    li = synth.make_linear(2048, 1536, 64, T, cfg=10, linear=T)
    x, paths, _ = U.to_device(li)
    ws = lb.alloc_workspace(T, 2048, 1536, 64)
    y_eager = lb.lb_linear_forward(x, paths, 64, workspace=ws, kernel=KERNELS[kernel]).clone()
    torch.cuda.synchronize()
    y_graph = torch.empty_like(y_eager)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        lb.lb_linear_forward(x, paths, 64, y=y_graph, workspace=ws, kernel=KERNELS[kernel])
    for rep in range(5):
        y_graph.zero_()
        g.replay()
        torch.cuda.synchronize()
        # eager work on the same workspace between replays
        y_mid = lb.lb_linear_forward(x, paths, 64, workspace=ws, kernel=KERNELS[kernel])
        torch.cuda.synchronize()
        if kernel in ("decode", "mma"):
            assert torch.equal(y_graph.view(torch.int16), y_eager.view(torch.int16)), rep
            assert torch.equal(y_mid.view(torch.int16), y_eager.view(torch.int16)), rep
        else:
            _check(li, U.torch_to_raw(y_graph, "bf16"), label=f"graph replay {rep}")
            _check(li, U.torch_to_raw(y_mid, "bf16"), label=f"eager between replays {rep}")


# ---------------------------------------------------------------------------
# the few-token stages (AUTO, 3 to 64 tokens; by sizes: test_auto_rule)
# ---------------------------------------------------------------------------
# tile classes and groups of latents at their edges, one run and several, runs whose wave groups get unequal shares of
# blocks, tails of d_in and r, rows that are not whole 16-byte pieces, outputs around the 64-row workgroups
FEW = [(16, 128, 64, 16), (16, 36, 65, 129), (17, 2092, 63, 33), (31, 4096, 200, 320), (32, 1000, 127, 50),
       (33, 288, 1, 193), (48, 3000, 257, 288), (49, 64, 500, 385), (64, 11008, 96, 800), (64, 260, 1000, 577),
       (20, 4100, 129, 641), (3, 520, 10000, 816)]


@pytest.mark.parametrize("case", FEW, ids=[f"T{c[0]}_{c[1]}x{c[2]}r{c[3]}" for c in FEW])
@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f32", "f32"), ("f16", "bf16")])
def test_few_tokens_edges(case, act, sc):
    T, d_in, d_out, r = case
    li = synth.make_linear(d_in, d_out, r, T, act_dtype=act, scale_dtype=sc, cfg=91, linear=T + d_in, l_over_sqrt_r=True)
    y_raw = _run(li)
    _check(li, y_raw, label=f"{case} {act}/{sc}")


# as above, with sizes that AUTO gives to these stages in fp32 and in 16 bits, in fp32 seen from the result (every kernel adds in
# an order of its own): both tile classes (2 tiles a wave; from r = 961 and 128 blocks of d_in 3), their first and last
# rank, all token tile counts, tails of d_in and r
FEW_TAKEN = [(16, 640, 65, 129), (17, 2092, 63, 33), (31, 4096, 33, 961), (16, 4096, 65, 961), (3, 4100, 127, 976),
             (8, 4124, 1024, 1008), (32, 4108, 130, 1008), (48, 4096, 65, 1024), (64, 4100, 70, 970), (49, 5000, 1, 1009),
             (64, 4092, 70, 961), (64, 2048, 64, 960), (33, 320, 129, 385), (48, 4128, 40, 960)]


@pytest.mark.parametrize("case", FEW_TAKEN, ids=[f"T{c[0]}_{c[1]}x{c[2]}r{c[3]}" for c in FEW_TAKEN])
@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f32", "f32")])
def test_few_tokens_classes(case, act, sc):
    T, d_in, d_out, r = case
    li = synth.make_linear(d_in, d_out, r, T, act_dtype=act, scale_dtype=sc, cfg=95, linear=T + d_in, l_over_sqrt_r=True)
    x, paths, _ = U.to_device(li, True)
    y = lb.lb_linear_forward(x, paths, r)
    _check(li, U.torch_to_raw(y, act), label=f"{case} {act}/{sc}")
    if act == "f32":
        for k in ("mma", "prefill"):
            if k == "prefill" or r <= 832:
                assert not torch.equal(y, lb.lb_linear_forward(x, paths, r, kernel=KERNELS[k])), k


def test_few_tokens_many_and_shared_workspace():
    # alone, among others of one launch, and between calls of other kernels on one workspace: the same bits
    specs = [(16, 1024, 700, 80), (24, 512, 900, 300), (16, 96, 64, 16), (16, 2048, 130, 530), (31, 640, 640, 64),
             (40, 512, 256, 48), (16, 160, 33, 200), (16, 320, 1025, 20), (16, 224, 96, 96), (16, 4096, 64, 128),
             (16, 64, 64, 64)]
    lins = [synth.make_linear(d_in, d_out, r, T, act_dtype="bf16", scale_dtype="f16", cfg=92, linear=i,
                              l_over_sqrt_r=True) for i, (T, d_in, d_out, r) in enumerate(specs)]
    items = []
    for li in lins:
        x, paths, _ = U.to_device(li, True)
        items.append((x, paths, li.r, None))
    alone = [lb.lb_linear_forward(x, paths, r) for x, paths, r, _ in items]
    many = lb.lb_linear_forward_many(items)
    ws = max((lb.alloc_workspace(li.T, li.d_in, li.d_out, li.r) for li in lins), key=lambda t: t.numel())
    for rep in range(2):
        for (x, paths, r, _), y in zip(items, alone):
            assert torch.equal(lb.lb_linear_forward(x, paths, r, workspace=ws), y)
            one = lb.lb_linear_forward(x[:1].contiguous(), paths, r, workspace=ws)  # look-up-table kernel
            assert torch.equal(one, lb.lb_linear_forward(x[:1].contiguous(), paths, r))
    torch.cuda.synchronize()
    for y, z in zip(alone, many):
        assert torch.equal(y, z)


# prefill stage 1: x rows of whole 16-byte chunks, of whole dwords only (d_in a multiple of 2, or any in fp32; x itself 4-byte
# but not 16-byte aligned) and of neither, with tails of the last 32-input step
@pytest.mark.parametrize("d_in", [64, 66, 94, 999, 1000, 4100])
@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f32", "f32"), ("f16", "bf16")])
def test_prefill_row_alignment(d_in, act, sc):
    li = synth.make_linear(d_in, 130, 50, 70, act_dtype=act, scale_dtype=sc, cfg=93, linear=d_in, l_over_sqrt_r=True)
    _check(li, _run(li, "prefill"), label=f"{d_in} {act}/{sc}")
    x, paths, _ = U.to_device(li, True)
    buf = torch.full((x.numel() + 2,), float("nan"), dtype=x.dtype, device="cuda")
    xs = buf[2:].view(x.shape) if act != "f32" else buf[1:-1].view(x.shape)
    xs.copy_(x)
    y = lb.lb_linear_forward(xs, paths, li.r, kernel=KERNELS["prefill"])
    assert torch.equal(y, lb.lb_linear_forward(x, paths, li.r, kernel=KERNELS["prefill"]))


# ---------------------------------------------------------------------------
# one workspace for calls that tag their intermediate values and calls that do not
# ---------------------------------------------------------------------------
TAG_BASE, TAG_COUNT = 0x7F810000, 0x3F0000  # tags of the decode kernels' slots, by epoch
SCRATCH = 4352  # first byte of a workspace's intermediate values


def _call(T, d_in, d_out, r, act="bf16", sc="f16", cfg=94):
    li = synth.make_linear(d_in, d_out, r, T, act_dtype=act, scale_dtype=sc, cfg=cfg, linear=T + r, l_over_sqrt_r=True)
    x, paths, _ = U.to_device(li, True)
    return x, paths, r


def _zeroed(*shapes):
    n = max(lb.lb_forward_workspace_bytes(*s) for s in shapes)
    return lb.lb_workspace_init(torch.empty(n, dtype=torch.uint8, device="cuda"))


def _high_words(ws):
    return ws[SCRATCH:].view(torch.int32)[1::2]


def test_untagged_words_are_no_tags():
    # r % 32 in 1..16: the upper halves of the last latent block's term pairs are zero, so whole words are bare bf16 patterns,
    # which the call counter reaches after some 15000 decode calls
    first, second = (16, 4096, 4096, 80), (15, 11008, 4096, 128)
    a, b = _call(*first), _call(*second)
    ref = lb.lb_linear_forward(b[0], b[1], b[2], kernel=KERNELS["mma"])
    ws = _zeroed(first, second)
    lb.lb_linear_forward(a[0], a[1], a[2], workspace=ws)
    torch.cuda.synchronize()
    left = ws.clone()
    hi = _high_words(ws)
    vals, counts = hi[(hi > 1) & (hi < 65536)].unique(return_counts=True)
    assert len(vals) > 40
    for v in vals[counts.argsort(descending=True)[:40]].tolist():
        ws.copy_(left)
        ws.view(torch.int32)[0] = v - 1
        y = lb.lb_linear_forward(b[0], b[1], b[2], workspace=ws, kernel=KERNELS["mma"])
        assert torch.equal(y, ref), v
    assert lb.lb_workspace_status(ws) == 0


@pytest.mark.parametrize("act,sc", [("bf16", "f16"), ("f16", "bf16"), ("f32", "f32")])
@pytest.mark.parametrize("T", [16, 100])
def test_intermediate_values_hold_no_tag(T, act, sc):
    # the few-token and prefill stages on ordinary values, infinities, NaNs (of every kind: quiet, signalling, of either
    # sign and with payloads) and values near the types' ends
    shape = (T, 1024, 1024, 80)
    x, paths, r = _call(*shape, act=act, sc=sc)
    it, special = {"bf16": (torch.int16, [0x7F80, 0xFF80, 0x7FC0, 0xFFC0, 0x7F81, 0x7FBF, 0xFFA0, 0x7FFF, 0x7F7F, 1]),
                   "f16": (torch.int16, [0x7C00, 0xFC00, 0x7E00, 0xFE00, 0x7C01, 0x7DFF, 0xFD00, 0x7FFF, 0x7BFF, 1]),
                   "f32": (torch.int32, [0x7F800000, 0xFF800000, 0x7FC00000, 0xFFC00000, 0x7F810000, 0x7FBFFFFF,
                                         0xFFA00000, 0x7FFFFFFF, 0x7F7FFFFF, 1])}[act]
    wrap = 16 if it == torch.int16 else 32
    ws = _zeroed(shape)
    for fill in [None] + special:
        xs = x.clone()
        if fill is not None:
            xs.view(it)[::3, 7] = fill - (1 << wrap) if fill >> (wrap - 1) else fill
        ws[SCRATCH:].zero_()
        lb.lb_linear_forward(xs, paths, r, workspace=ws)
        hi = _high_words(ws)
        assert int((hi != 0).sum()) > 1000
        assert not bool(((hi >= TAG_BASE) & (hi < TAG_BASE + TAG_COUNT)).any()), fill


@pytest.mark.parametrize("kernel,T", [("decode", 1), ("mma", 8)])
def test_tags_come_round(kernel, T):
    # the epoch word moves on to 0 after the last tag; the call in the middle of either half takes the other half's tags out
    # of the workspace, so a value left from a call with the same tag is not taken for a fresh one
    big, small = (T, 4096, 1024, 144), (T, 512, 512, 80)
    b, s = _call(*big), _call(*small)
    ref_b, ref_s = (lb.lb_linear_forward(c[0], c[1], c[2], kernel=KERNELS[kernel]) for c in (b, s))
    ws = _zeroed(big, small)
    ctrl = ws.view(torch.int32)
    half = TAG_COUNT // 2

    def tags(lo, hi):
        h = _high_words(ws)
        return int(((h >= TAG_BASE + lo) & (h < TAG_BASE + hi)).sum())

    ctrl[0] = TAG_COUNT - 1
    for after in (0, 1, 2):
        assert torch.equal(lb.lb_linear_forward(s[0], s[1], s[2], workspace=ws, kernel=KERNELS[kernel]), ref_s)
        assert int(ctrl[0]) == after
    x0 = b[0].clone()
    for mine, other in ((0, half), (half, 0)):
        b[0].copy_(-2 * x0)
        ctrl[0] = mine + 5
        lb.lb_linear_forward(b[0], b[1], b[2], workspace=ws, kernel=KERNELS[kernel])
        assert int(ctrl[0]) == mine + 6 and tags(mine + 5, mine + 6) > 0
        for turn in (other + half // 2 - 1, other + half // 2):
            ctrl[0] = turn
            assert torch.equal(lb.lb_linear_forward(s[0], s[1], s[2], workspace=ws, kernel=KERNELS[kernel]), ref_s)
            assert (tags(mine, mine + half) == 0) == (turn == other + half // 2)
        b[0].copy_(x0)
        ctrl[0] = mine + 5
        assert torch.equal(lb.lb_linear_forward(b[0], b[1], b[2], workspace=ws, kernel=KERNELS[kernel]), ref_b)
    assert lb.lb_workspace_status(ws) == 0


# AUTO's rule for 3 to 64 tokens, at both sides of each of its lines: the few-token stages, the kernel above them, or (None)
# whatever a wide layer without aligned groups of four inputs takes.  Each kernel has bits of its own on these inputs, so the
# one that ran is told by them.
RULE = [(3, 5120, 13824, 160, "mma"), (3, 8192, 8192, 256, "few"), (7, 4096, 4096, 544, "few"), (7, 4096, 11008, 128, "mma"),
        (8, 4096, 4096, 80, "few"), (8, 4096, 4096, 64, "mma"), (8, 2048, 2048, 80, "mma"), (8, 2048, 16384, 64, "few"),
        (15, 4096, 1024, 128, "mma"), (15, 4096, 11008, 128, "few"), (16, 1024, 1024, 80, "few"), (16, 1024, 1024, 48, "mma"),
        (16, 512, 2048, 64, "mma"), (17, 512, 512, 64, "few"), (23, 512, 512, 32, "mma"), (24, 512, 512, 32, "few"),
        (31, 256, 256, 32, "mma"), (32, 512, 512, 32, "few"), (32, 384, 384, 32, "prefill"), (48, 1024, 16640, 64, "few"),
        (49, 1024, 16640, 64, "prefill"), (64, 1024, 16384, 64, "few"), (20, 1022, 1024, 80, "mma"), (40, 1022, 1024, 80, "prefill")]
RULE_F32 = [(24, 512, 512, 64, "mma"), (28, 512, 512, 64, "few"), (24, 1000, 1000, 40, "few"), (32, 384, 384, 32, "few"),
            (49, 384, 384, 32, "prefill"), (64, 10240, 512, 256, "prefill"), (64, 10240, 512, 272, "few"),
            (48, 10240, 512, 256, "few")]


@pytest.mark.parametrize("case,act,sc", [(c, "bf16", "f16") for c in RULE] + [(c, "f32", "f32") for c in RULE_F32],
                         ids=lambda v: f"T{v[0]}_{v[1]}x{v[2]}r{v[3]}" if isinstance(v, tuple) else v)
def test_auto_rule(case, act, sc):
    T, d_in, d_out, r, want = case
    x, paths, _ = _call(T, d_in, d_out, r, act=act, sc=sc)
    y = lb.lb_linear_forward(x, paths, r)
    ran = [k for k in ("mma", "prefill") if torch.equal(y, lb.lb_linear_forward(x, paths, r, kernel=KERNELS[k]))]
    # (16-bit outputs of two kernels may all agree where sums are short)
    if want == "few":
        ran = ran or ["few"]
    assert want in ran, (ran, case)
