"""GPU parity of the Dual-SVID conversion (lb_dual_svid) against the oracle's
Dual-SVID (O7) on the same seeded weights: Sec. 3.2 "Dual-SVID Initialization"
and the residual path of Sec. 3.3.

Bars.  The GPU path computes in fp64 and rounds its outputs to fp32 once; the
oracle computes an exact SVD (one-sided Jacobi), the GPU path a truncated one
by subspace iteration, whose error for singular pair k decays like
(sigma_{b+1} / sigma_k)^(2 iters + 1).  The parity cases run enough rounds for
that term to vanish against fp32 rounding, so:
  - latent factors U', V': max |GPU - oracle| <= 1e-5 max |oracle| per factor;
  - h0, g0, l0 and sigma: max relative error <= 1e-5 (sigma from the oracle as
    the squared column norms of U', since U' = U_r diag(sqrt(sigma)));
  - the sign bits (what the packed path keeps): identical wherever
    |oracle| > 1e-5 max |oracle| (smaller entries may round either way);
  - W_res: max |GPU - oracle| <= 1e-5 max |W|.
Path 1 is compared with the oracle's path 1 run on the oracle's own W_res.
At the full Llama2-7B q_proj shape the oracle's Jacobi SVD is out of reach,
so properties that hold at any size are checked instead."""
import numpy as np
import pytest

import oracle as O
from paper_2506_13771_amd import synth
from conftest import gpu_available
from test_svid_oracle import exact_family

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch
    import paper_2506_13771_amd as lb

TOL = 1e-5


def _run(W, r, **kw):
    Wd = torch.from_numpy(np.ascontiguousarray(W)).cuda()
    out = lb.lb_dual_svid(Wd, r, residual=True, **kw)
    torch.cuda.synchronize()
    return {k: ([t.double().cpu().numpy() for t in v] if isinstance(v, list) else v.double().cpu().numpy())
            for k, v in out.items()}


def _maxrel(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


def _check_path(got, ref, p, label, align=False):
    Ul, Vl, h, g, l = (ref[k][p] for k in ("U", "V", "h", "g", "l"))
    if align:
        # weights whose left vectors have several entries of equal largest magnitude: the sign
        # convention's choice is then decided by rounding, so pairs are matched up to a joint flip
        f = np.where(np.sum(got["U"][p] * Ul, axis=0) < 0, -1.0, 1.0)
        got = dict(got, U=list(got["U"]), V=list(got["V"]))
        got["U"][p] = got["U"][p] * f
        got["V"][p] = got["V"][p] * f
    assert _maxrel(got["U"][p], Ul) <= TOL, (label, "U", _maxrel(got["U"][p], Ul))
    assert _maxrel(got["V"][p], Vl) <= TOL, (label, "V", _maxrel(got["V"][p], Vl))
    for name, ref_v in (("h", h), ("g", g), ("l", l)):
        err = _maxrel(got[name][p], ref_v)
        assert err <= TOL, (label, name, err)
    sig = np.sum(Ul * Ul, axis=0)
    assert _maxrel(got["sigma"][p], sig) <= TOL, (label, "sigma")
    for name, ref_v in (("U", Ul), ("V", Vl)):
        big = np.abs(ref_v) > TOL * np.abs(ref_v).max()
        assert np.array_equal(got[name][p][big] < 0, ref_v[big] < 0), (label, name, "signs")


# (d_out, d_in, r, rank of the signal part, noise)
CASES = [
    (192, 160, 16, 24, 0.05),
    (160, 224, 24, 32, 0.05),   # wide
    (320, 256, 32, 48, 0.02),   # several 64-row tiles and split-K Gram sums
    (70, 50, 50, 40, 0.1),      # r = min(d_out, d_in): the block is the whole space
    (33, 65, 7, 5, 0.1),        # ragged tiles everywhere
    (384, 320, 120, 124, 0.05),  # block b = 136 > 128: one triangle of each small matrix in LDS
    (290, 250, 113, 118, 0.05),  # odd block b = 129 (the round-robin ordering's dummy index)
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}x{c[1]}r{c[2]}" for c in CASES])
def test_dual_svid_matches_oracle(case):
    d_out, d_in, r, k, noise = case
    W = synth.dense_weight(d_out, d_in, k, noise, cfg=70, linear=d_out + d_in)
    ref = O.dual_svid(W.astype(np.float64), r)
    got = _run(W, r, oversample=16, iters=40)
    _check_path(got, ref, 0, f"{case} path 0")
    assert np.abs(got["W_res"] - ref["Wres"]).max() <= TOL * np.abs(W).max()
    _check_path(got, ref, 1, f"{case} path 1")


# (d_out, d_in, r, oversample): blocks b = r + oversample at the edges of the 16-wide tiles of the tiled
# Cholesky and triangular solve, the smallest, and the largest of each of their two sizes (128, 192)
EDGES = [(40, 30, 1, 0), (40, 30, 15, 0), (30, 40, 16, 0), (40, 35, 16, 1), (70, 65, 48, 1), (150, 128, 112, 16),
         (208, 192, 176, 16)]


@pytest.mark.parametrize("case", EDGES, ids=[f"b{c[2] + c[3]}" for c in EDGES])
def test_dual_svid_block_edges(case):
    d_out, d_in, r, over = case
    W = synth.dense_weight(d_out, d_in, r, 0.002, cfg=71, linear=d_out + d_in)
    ref = O.dual_svid(W.astype(np.float64), r)
    got = _run(W, r, oversample=over, iters=40)
    _check_path(got, ref, 0, f"{case} path 0")
    assert np.abs(got["W_res"] - ref["Wres"]).max() <= TOL * np.abs(W).max()


@pytest.mark.parametrize("d_out,d_in,r", [(64, 32, 4), (128, 128, 16), (32, 128, 8)])
def test_dual_svid_exact_family(d_out, d_in, r):
    # Dual-SVID recovers a weight built as one LittleBit path exactly; the residual is ~0
    W, SU, SV, h, g, l = exact_family(d_out, d_in, r, d_out + d_in + r)
    Wf = W.astype(np.float32)
    ref = O.dual_svid(Wf.astype(np.float64), r)
    got = _run(Wf, r, oversample=8, iters=10)
    _check_path(got, ref, 0, "exact family path 0", align=True)
    flip = np.sign(np.sum(np.sign(got["U"][0]) * SU, axis=0))
    assert np.array_equal(np.sign(got["U"][0]), SU * flip)
    assert np.array_equal(np.sign(got["V"][0]), SV * flip)
    assert np.abs(got["W_res"]).max() <= 1e-5 * np.abs(W).max()


def test_dual_svid_steep_spectrum():
    # every block is orthonormalised through its Gram matrix, which squares its condition
    # number: top-16 singular values falling geometrically from 1 to 1e-4, then 8 near 1e-8
    # (a gap of 1e-4) and nothing else, so the 32-column block is rank-deficient and its
    # kept part has a condition number near 1e4; the bars of the other cases still hold
    d_out, d_in, r, k = 160, 128, 16, 24
    rng = np.random.default_rng(7401)
    Uo, _ = np.linalg.qr(rng.standard_normal((d_out, k)))
    Vo, _ = np.linalg.qr(rng.standard_normal((d_in, k)))
    s = np.concatenate([10.0 ** (-4.0 * np.arange(r) / (r - 1)), 1e-8 * 10.0 ** (-np.arange(k - r) / 8.0)])
    W = ((Uo * s) @ Vo.T).astype(np.float32)
    ref = O.dual_svid(W.astype(np.float64), r)
    got = _run(W, r, oversample=16, iters=10)
    _check_path(got, ref, 0, "steep spectrum path 0")
    assert np.abs(got["W_res"] - ref["Wres"]).max() <= TOL * np.abs(W).max()
    _check_path(got, ref, 1, "steep spectrum path 1")


def test_dual_svid_bf16_weight_and_determinism():
    d_out, d_in, r = 128, 96, 12
    W = synth.dense_weight(d_out, d_in, 16, 0.05, cfg=71)
    Wb = torch.from_numpy(W).to(torch.bfloat16)
    ref = O.dual_svid(Wb.double().numpy(), r)
    a = lb.lb_dual_svid(Wb.cuda(), r, oversample=16, iters=40, residual=True)
    b = lb.lb_dual_svid(Wb.cuda(), r, oversample=16, iters=40, residual=True)
    torch.cuda.synchronize()
    for key in ("U", "V", "h", "g", "l", "sigma"):
        for p in range(2):
            assert torch.equal(a[key][p], b[key][p]), key
    assert torch.equal(a["W_res"], b["W_res"])
    got = {k: ([t.double().cpu().numpy() for t in v] if isinstance(v, list) else v.double().cpu().numpy())
           for k, v in a.items()}
    _check_path(got, ref, 0, "bf16 path 0")
    _check_path(got, ref, 1, "bf16 path 1")


def test_dual_svid_zero_weight():
    # every singular value is 0: all outputs are zero (the oracle's too), nothing is NaN
    W = np.zeros((48, 40), dtype=np.float32)
    ref = O.dual_svid(W.astype(np.float64), 8)
    got = _run(W, 8, oversample=8, iters=3)
    for key in ("U", "V", "h", "g", "l", "sigma"):
        for p in range(2):
            assert np.all(got[key][p] == 0.0), key
    for key in ("U", "V", "h", "g", "l"):
        assert np.all(ref[key][0] == 0.0)
    assert np.all(got["W_res"] == 0.0)


def test_dual_svid_feeds_the_forward():
    # the converted linear, packed and run by lb_linear_forward, approximates W x: its error is
    # that of the two-path effective weight, which is below the primary path's alone
    d_out, d_in, r = 256, 192, 32
    W = synth.dense_weight(d_out, d_in, 24, 0.02, cfg=72)
    Wd = torch.from_numpy(W).cuda()
    paths = lb.littlebit_from_dense(Wd, r, scale_dtype=torch.float32, oversample=16, iters=30)
    What = lb.lb_dense_reference_weight(paths, d_in, d_out, r).double()
    s = lb.lb_dual_svid(Wd, r, oversample=16, iters=30, residual=True)
    e_two = torch.linalg.norm(Wd.double() - What) / torch.linalg.norm(Wd.double())
    e_one = torch.linalg.norm(s["W_res"].double()) / torch.linalg.norm(Wd.double())
    assert float(e_two) < float(e_one) < 1.0
    x = torch.randn(4, d_in, device="cuda", dtype=torch.float32)
    y = lb.lb_linear_forward(x, paths, r)
    ref = x.double() @ What.T
    assert float(torch.linalg.norm(y.double() - ref) / torch.linalg.norm(ref)) < 1e-5


def test_dual_svid_full_size_properties():
    # Llama2-7B q_proj shape at 0.1 BPW (r = 80), default block and rounds
    d_out = d_in = 4096
    r = lb.lb_rank_for_bpw(d_in, d_out, 0.1)
    W = synth.dense_weight(d_out, d_in, 2 * r, 0.05, cfg=73)
    Wd = torch.from_numpy(W).cuda().double()
    s = lb.lb_dual_svid(torch.from_numpy(W).cuda(), r, iters=30, residual=True)
    torch.cuda.synchronize()
    for p, Wp in ((0, Wd), (1, s["W_res"].double())):
        Ul, Vl, sig = s["U"][p].double(), s["V"][p].double(), s["sigma"][p].double()
        assert bool(torch.all(sig[:-1] >= sig[1:])) and bool(torch.all(sig > 0))
        Ur, Vr = Ul / sig.sqrt(), Vl / sig.sqrt()
        eye = torch.eye(r, device="cuda", dtype=torch.float64)
        assert float((Ur.T @ Ur - eye).abs().max()) < 1e-5
        assert float((Vr.T @ Vr - eye).abs().max()) < 1e-5
        # singular triplets: W v_k = sigma_k u_k and W^T u_k = sigma_k v_k
        res1 = torch.linalg.norm(Wp @ Vr - Ur * sig, dim=0) / sig[0]
        res2 = torch.linalg.norm(Wp.T @ Ur - Vr * sig, dim=0) / sig[0]
        assert float(res1.max()) < 1e-4 and float(res2.max()) < 1e-4, (p, float(res1.max()), float(res2.max()))
        # sign convention: each left vector's entry of largest magnitude is positive
        idx = Ul.abs().argmax(dim=0)
        assert bool(torch.all(Ul[idx, torch.arange(r, device="cuda")] > 0))
        # rank-1 factors: h and l_u are the top singular pair of |U'| (power-iteration fixed point)
        M = Ul.abs()
        h = s["h"][p].double()
        lu_dir = M.T @ h
        hh = M @ (lu_dir / torch.linalg.norm(lu_dir))
        assert float(torch.linalg.norm(hh / torch.linalg.norm(hh) - h / torch.linalg.norm(h))) < 1e-5
        assert float(h.sum()) >= 0 and float(s["g"][p].double().sum()) >= 0
    # W_res = W - diag(h) sign(U') diag(l) sign(V')^T diag(g) of path 0
    su = torch.where(s["U"][0] < 0, -1.0, 1.0).double()
    sv = torch.where(s["V"][0] < 0, -1.0, 1.0).double()
    What = (s["h"][0].double()[:, None] * su * s["l"][0].double()) @ (sv.T * s["g"][0].double()[None, :])
    assert float((Wd - What - s["W_res"].double()).abs().max()) <= 1e-5 * float(Wd.abs().max())
