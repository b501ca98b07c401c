"""GPU parity: causal prompt attention with row statistics (antkv_prefill_attn; paper Sec. 2.1 and the first step
of Alg. 1) against the CPU oracle, and its hand-over to the Anchor Score pass."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2506_19505_amd as antkv
from gpu_util import check_index_sets, dev
from workloads import CONFIGS, anchor_count, make_qkv

pytestmark = pytest.mark.gpu

# fp16 probabilities in the value product (2^-11 relative each, averaged over a row) and the fp16 output rounding
OUT_TOL = 2e-3


def _check(oracle, seed, B, Hq, Hkv, N, Nq, scale, q_gain=1.0):
    q, k, v = make_qkv(seed, B, Hq, Hkv, N, Nq, 128)
    q = (q.astype(np.float32) * q_gain).astype(np.float16)
    geom = antkv.Geometry(B, Hq, Hkv, 8)
    out, rm, rs = antkv.prefill_attn(geom, dev(q), dev(k), dev(v), scale)
    torch.cuda.synchronize()
    want, wm, wl = oracle.prefill_attn(q, k, v, scale)
    got = out.cpu().numpy().astype(np.float64)
    err = np.linalg.norm(got - want, axis=-1) / np.maximum(np.linalg.norm(want, axis=-1), 1e-30)
    assert err.max() <= OUT_TOL, f"relative L2 {err.max():.3e}"
    np.testing.assert_allclose(rm.cpu().numpy(), wm, rtol=2e-6, atol=2e-6)
    np.testing.assert_allclose(rs.cpu().numpy(), wl, rtol=1e-4)
    print(f"N={N} Nq={Nq} G={Hq // Hkv}: out rel-L2 max {err.max():.2e}")
    return q, k, v, rm, rs


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(1, 8, 2, 300, 300), (2, 4, 4, 1000, 137), (1, 4, 1, 257, 257),
                                           (1, 4, 2, 64, 64), (1, 2, 2, 1, 1), (1, 8, 2, 2100, 33),
                                           (2, 8, 4, 95, 95)])
def test_prefill_attn_small(oracle, B, Hq, Hkv, N, Nq):
    _check(oracle, 61, B, Hq, Hkv, N, Nq, 1.0 / np.sqrt(128))


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(1, 4, 4, 33, 33), (1, 4, 1, 127, 127), (2, 4, 2, 129, 65), (1, 8, 8, 600, 600),
                                           (3, 8, 2, 161, 161), (1, 2, 1, 391, 390), (1, 4, 1, 1025, 700)])
def test_prefill_attn_tile_edges(oracle, B, Hq, Hkv, N, Nq):
    """Every number of key tiles modulo the loop's four, waves of one workgroup that end at different tiles, windows that
    start inside a tile."""
    _check(oracle, 64, B, Hq, Hkv, N, Nq, 1.0 / np.sqrt(128))


@pytest.mark.parametrize("Hq,Hkv", [(4, 1), (2, 2)])
def test_prefill_attn_later_rows_stay_unseen(oracle, Hq, Hkv):
    """Rows of K and V behind a query's 32-key tile take no part in its result, whatever they hold."""
    N, seen, scale = 700, 320, 1.0 / np.sqrt(128)
    q, k, v = make_qkv(65, 1, Hq, Hkv, N, N, 128)
    k[:, :, seen:], v[:, :, seen:] = np.nan, np.inf
    out, rm, rs = antkv.prefill_attn(antkv.Geometry(1, Hq, Hkv, 8), dev(q), dev(k), dev(v), scale)
    want, wm, wl = oracle.prefill_attn(np.ascontiguousarray(q[:, :, :seen]), np.ascontiguousarray(k[:, :, :seen]),
                                       np.ascontiguousarray(v[:, :, :seen]), scale)
    got = out.cpu().numpy().astype(np.float64)[:, :, :seen]
    assert (np.linalg.norm(got - want, axis=-1) <= OUT_TOL * np.linalg.norm(want, axis=-1)).all()
    np.testing.assert_allclose(rm.cpu().numpy()[:, :, :seen], wm, rtol=2e-6, atol=2e-6)
    np.testing.assert_allclose(rs.cpu().numpy()[:, :, :seen], wl, rtol=1e-4)


def test_prefill_attn_wide_score_range(oracle):
    """Scores spread over a few hundred log2 units: the softmax reference has to move many times per row."""
    _check(oracle, 62, 1, 4, 2, 700, 700, 1.0 / np.sqrt(128), q_gain=12.0)


def test_prefill_attn_feeds_anchor_select(oracle):
    """Alg. 1: the attention pass hands its row statistics to the Anchor Score pass."""
    B, Hq, Hkv, N = 1, 8, 2, 1536
    scale = 1.0 / np.sqrt(128)
    q, k, v, rm, rs = _check(oracle, 63, B, Hq, Hkv, N, N, scale)
    kk = anchor_count(N)
    geom = antkv.Geometry(B, Hq, Hkv, 8)
    idx_k, idx_v, ans_k, ans_v = antkv.anchor_select(geom, dev(q), dev(k), scale, kk, row_max=rm, row_sum=rs)
    ok, ov = oracle.anchor_score(q, k, scale)
    np.testing.assert_allclose(ans_v.cpu().numpy(), ov, rtol=1e-4, atol=1e-9)
    np.testing.assert_allclose(ans_k.cpu().numpy(), ok, rtol=1e-4, atol=1e-9)
    for got, score in ((idx_k, ok), (idx_v, ov)):
        want, margin = oracle.topk(score, kk, want_margin=True)
        check_index_sets(got.cpu().numpy(), want, margin)


def test_prefill_attn_full_prefill_sampled_rows(oracle):
    """Config 3 at full size (N = Nq = 32768, 32 heads): sampled query rows against the oracle's definition,
    computed row by row."""
    w = CONFIGS["cfg3"]
    q, k, v = make_qkv(w.seed, w.B, w.Hq, w.Hkv, w.N, w.N, w.D)
    geom = antkv.Geometry(w.B, w.Hq, w.Hkv, w.d_sub)
    out, rm, rs = antkv.prefill_attn(geom, dev(q), dev(k), dev(v), w.scale)
    torch.cuda.synchronize()
    rng = np.random.default_rng(5)
    G = w.Hq // w.Hkv
    rows = [(0, 0, 0), (0, w.Hq - 1, w.N - 1), (0, 3, 31), (0, 5, 32), (0, 7, 63), (0, 9, 64)]
    rows += [(0, int(rng.integers(w.Hq)), int(rng.integers(w.N))) for _ in range(40)]
    got_all, rm_all, rs_all = out.cpu().numpy(), rm.cpu().numpy(), rs.cpu().numpy()
    worst = 0.0
    for b, h, i in rows:
        # one row through the oracle: the query alone (Nq = 1) over the keys it sees
        want, wm, wl = oracle.prefill_attn(q[b:b + 1, h:h + 1, i:i + 1], k[b:b + 1, h // G:h // G + 1, :i + 1],
                                           v[b:b + 1, h // G:h // G + 1, :i + 1], w.scale)
        got = got_all[b, h, i].astype(np.float64)
        err = np.linalg.norm(got - want[0, 0, 0]) / np.linalg.norm(want[0, 0, 0])
        worst = max(worst, err)
        assert err <= OUT_TOL, f"row {(b, h, i)}: relative L2 {err:.3e}"
        assert abs(rm_all[b, h, i] - wm[0, 0, 0]) <= 2e-6 * (1 + abs(wm[0, 0, 0]))
        assert abs(rs_all[b, h, i] - wl[0, 0, 0]) <= 1e-4 * wl[0, 0, 0]
    print(f"cfg3 sampled rows: out rel-L2 max {worst:.2e}")


def test_prefill_attn_rejects_bad_arguments():
    lib = antkv.load_library()
    g = antkv.Geometry(1, 4, 2, 8).c()
    x = torch.zeros(1, 4, 8, 128, dtype=torch.float16, device="cuda")
    kv = torch.zeros(1, 2, 8, 128, dtype=torch.float16, device="cuda")
    st = torch.zeros(1, 4, 8, dtype=torch.float32, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    call = lambda **o: lib.antkv_prefill_attn(
        ctypes.byref(g), o.get("q", p(x)), p(kv), p(kv), o.get("N", 8), o.get("Nq", 8), o.get("scale", 0.1), p(x),
        o.get("rm", p(st)), p(st), None)
    assert call(Nq=9) != 0
    assert call(N=0, Nq=0) != 0
    assert call(q=None) != 0
    assert call(rm=None) != 0
    assert call(scale=0.0) != 0
    assert call(q=ctypes.c_void_p(x.data_ptr() + 2)) != 0
    torch.cuda.synchronize()


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(47, 8, 8, 70, 70), (48, 8, 8, 70, 70), (95, 16, 4, 33, 33), (96, 16, 4, 33, 33), (1, 16, 8, 289, 130),
                                           (96, 8, 4, 129, 97), (1, 4, 1, 1, 1)])
def test_prefill_either_workgroup_size(B, Hq, Hkv, N, Nq):
    """Workgroups of four waves up to 383 of eight, of eight from there; groups of 1, 2 and 4, ragged tiles, queries behind a
    cached prefix; against float64.  Bounds: fp16 weights and output, 2^-11 each, 1e-4 for the rest; statistics as fp32 gives them."""
    gen = torch.Generator(device="cuda").manual_seed(N + B)
    rnd = lambda *s: torch.randn(s, dtype=torch.float16, device="cuda", generator=gen)
    q, k, v, scale = rnd(B, Hq, Nq, 128), rnd(B, Hkv, N, 128), rnd(B, Hkv, N, 128), 128 ** -0.5
    out, row_max, row_sum = antkv.prefill_attn(antkv.Geometry(B, Hq, Hkv, 8), q, k, v, scale)
    kx, vx = (t.double().repeat_interleave(Hq // Hkv, dim=1) for t in (k, v))
    s = scale * (q.double() @ kx.transpose(2, 3).contiguous())
    s = s.masked_fill(torch.arange(N, device="cuda")[None, :] > torch.arange(N - Nq, N, device="cuda")[:, None], -float("inf"))
    m = s.amax(-1)
    e = torch.exp(s - m[..., None])
    want = (e @ vx) / e.sum(-1, keepdim=True)
    err = ((out.double() - want).norm(dim=-1) / want.norm(dim=-1)).max().item()
    print(f"B{B} {Hq}/{Hkv} {Nq} of {N}: {err:.2e}")
    assert err <= 2.0 ** -10 + 1e-4
    assert (row_max.double() - m).abs().max().item() <= 1e-5 and ((row_sum.double() / e.sum(-1)) - 1).abs().max().item() <= 1e-4
