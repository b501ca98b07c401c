"""GPU parity: Anchor Score (paper Eq. (4)) + selection against the CPU oracle."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2506_19505_amd as antkv
from gpu_util import check_index_sets, dev
from workloads import CONFIGS, anchor_count, make_qkv

pytestmark = pytest.mark.gpu


def _run(oracle, seed, B, Hq, Hkv, N, Nq, k, scale=None, check_scores=True):
    q, kk, _ = make_qkv(seed, B, Hq, Hkv, N, Nq, 128, want_v=False)
    scale = scale or 1.0 / np.sqrt(128)
    geom = antkv.Geometry(B, Hq, Hkv, 8)
    idx_k, idx_v, ans_k, ans_v = antkv.anchor_select(geom, dev(q), dev(kk), scale, k)
    torch.cuda.synchronize()
    ok, ov = oracle.anchor_score(q, kk, scale)
    gk, gv = ans_k.cpu().numpy().astype(np.float64), ans_v.cpu().numpy().astype(np.float64)
    if check_scores:
        # informative tolerance on the scores themselves; the gate is the index sets below
        np.testing.assert_allclose(gv, ov, rtol=2e-5, atol=1e-9)
        np.testing.assert_allclose(gk, ok, rtol=2e-5, atol=1e-9)
    np.testing.assert_allclose(gv.sum(-1), Nq * (Hq // Hkv), rtol=1e-5)      # rows of A sum to one
    soft = 0
    for got, score in ((idx_k, ok), (idx_v, ov)):
        want, margin = oracle.topk(score, k, want_margin=True)
        soft += check_index_sets(got.cpu().numpy(), want, margin)
    rel = max(np.abs(gk - ok).max() / np.abs(ok).max(), np.abs(gv - ov).max() / np.abs(ov).max())
    print(f"N={N} Nq={Nq}: score max-rel-err {rel:.2e}, near-tie index disagreements {soft}")


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(1, 4, 1, 96, 96), (2, 8, 2, 777, 777), (1, 4, 2, 1000, 37),
                                           (1, 2, 2, 300, 1), (2, 4, 4, 65, 64), (1, 4, 1, 5000, 32)])
def test_anchor_select_small(oracle, B, Hq, Hkv, N, Nq):
    _run(oracle, 21, B, Hq, Hkv, N, Nq, anchor_count(N))


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(4, 16, 16, 4200, 300), (8, 16, 8, 4096, 257), (16, 16, 4, 4353, 289)])
def test_anchor_select_wide_key_blocks(oracle, B, Hq, Hkv, N, Nq):
    """Enough (head, key block) pairs for the column reduction with 64 keys per wave; ragged keys, ragged queries and a
    diagonal that starts inside a key block, for one, two and four heads per KV head."""
    _run(oracle, 27, B, Hq, Hkv, N, Nq, 40)


@pytest.mark.parametrize("Nq", [32, 33, 65, 97, 129, 161])
@pytest.mark.parametrize("Hq", [2, 4])
def test_anchor_select_step_counts(oracle, Hq, Nq):
    """Every remainder of the column reduction's (head, query tile) steps by four, from one step on."""
    _run(oracle, 29, 1, Hq, 2, 410, Nq, 17)


@pytest.mark.parametrize("Nq", [257, 289, 321, 353])
def test_anchor_select_step_counts_wide_key_blocks(oracle, Nq):
    _run(oracle, 30, 4, 16, 16, 4100, Nq, 40)


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(1, 4, 1, 1024, 31), (1, 4, 2, 1025, 32), (2, 2, 2, 2081, 33), (1, 8, 2, 9217, 64)])
def test_anchor_select_key_ranges(oracle, B, Hq, Hkv, N, Nq):
    """Phase 1 of a query window split over keys: one range, a last range of a few keys, queries inside the last ranges."""
    _run(oracle, 28, B, Hq, Hkv, N, Nq, anchor_count(N))


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(1, 1, 1, 7, 1), (1, 4, 1, 31, 31), (2, 4, 2, 33, 32), (1, 4, 2, 1000, 20), (1, 2, 1, 4099, 64),
                                           (1, 1, 1, 12345, 128), (2, 1, 1, 260, 96), (5, 24, 24, 129, 7), (1, 32, 8, 24611, 32)])
def test_anchor_select_windows(oracle, B, Hq, Hkv, N, Nq):
    """Every step count of the window kernels (heads of the group x query tiles, 1 to 4): fewer tiles than waves, ragged keys and
    queries, a diagonal over several key tiles, and ranges of several rounds of the waves."""
    _run(oracle, 31, B, Hq, Hkv, N, Nq, anchor_count(N))


def test_anchor_select_k_edges(oracle):
    _run(oracle, 22, 1, 4, 1, 200, 200, 0)
    _run(oracle, 22, 1, 4, 1, 200, 200, 200)


def test_anchor_select_with_supplied_row_stats(oracle):
    """The extended-attention path of Sec. 3.3: row max / row sum come from outside."""
    B, Hq, Hkv, N, Nq, k = 1, 8, 2, 640, 640, 7
    q, kk, _ = make_qkv(23, B, Hq, Hkv, N, Nq, 128, want_v=False)
    scale = 0.1
    ok, ov, st = oracle.anchor_score(q, kk, scale, want_stats=True)
    geom = antkv.Geometry(B, Hq, Hkv, 8)
    rm, rs = dev(st["row_max"].astype(np.float32)), dev(st["row_sum"].astype(np.float32))
    idx_k, idx_v, ans_k, ans_v = antkv.anchor_select(geom, dev(q), dev(kk), scale, k, row_max=rm, row_sum=rs)
    np.testing.assert_allclose(ans_v.cpu().numpy(), ov, rtol=3e-5, atol=1e-9)
    np.testing.assert_allclose(ans_k.cpu().numpy(), ok, rtol=3e-5, atol=1e-9)


def test_anchor_select_tiny_decode_config(oracle):
    """Config 0: 32 query / 8 KV heads, 4096-token prompt scored against itself, 41 anchors."""
    w = CONFIGS["cfg0"]
    _run(oracle, w.seed, w.B, w.Hq, w.Hkv, w.N, w.Nq_select, w.k)


def test_anchor_select_mid_prefill(oracle):
    _run(oracle, 24, 1, 8, 2, 8192, 8192, anchor_count(8192))


def test_anchor_select_long_context_window(oracle):
    """32-query observation window over a 131072-token context (the long-context decode workload)."""
    _run(oracle, 25, 1, 8, 2, 131072, 32, anchor_count(131072))


def test_anchor_select_full_prefill_invariants(oracle):
    """Config 3 at full size (Nq = N = 32768, 32 heads).  All heads: what holds at any size (rows of A sum to one,
    AnS(K) within its bound, ascending unique index sets that pick the largest scores).  One KV head with its four
    query heads: every score and both index sets against the oracle (the oracle needs ~10-20 s for one head)."""
    w = CONFIGS["cfg3"]
    q, kk, _ = make_qkv(w.seed, w.B, w.Hq, w.Hkv, w.N, w.N, w.D, want_v=False)
    geom = antkv.Geometry(w.B, w.Hq, w.Hkv, w.d_sub)
    idx_k, idx_v, ans_k, ans_v = antkv.anchor_select(geom, dev(q), dev(kk), w.scale, w.k)
    gk, gv = ans_k.cpu().numpy().astype(np.float64), ans_v.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(gv.sum(-1), w.N * w.G, rtol=1e-5)
    qn = np.linalg.norm(q.astype(np.float64), axis=-1).reshape(w.B, w.Hkv, -1).sum(-1)
    assert (gk >= 0).all() and (gk <= 0.25 * qn[..., None]).all()
    for idx, sc in ((idx_k.cpu().numpy(), ans_k.cpu().numpy()), (idx_v.cpu().numpy(), ans_v.cpu().numpy())):
        for b in range(w.B):
            for g in range(w.Hkv):
                sel = idx[b, g]
                assert np.all(np.diff(sel) > 0) and sel.min() >= 0 and sel.max() < w.N
                rest = np.delete(sc[b, g], sel)
                assert sc[b, g][sel].min() >= rest.max()
    g = 5                                                      # a KV head in the middle: non-zero head offsets
    print("oracle on one KV head of cfg3 ...", flush=True)
    ok, ov = oracle.anchor_score(q[:, g * w.G:(g + 1) * w.G], kk[:, g:g + 1], w.scale)
    np.testing.assert_allclose(gv[:, g], ov[:, 0], rtol=3e-5, atol=1e-9)
    np.testing.assert_allclose(gk[:, g], ok[:, 0], rtol=3e-5, atol=1e-9)
    soft = 0
    for got, score in ((idx_k, ok), (idx_v, ov)):
        want, margin = oracle.topk(score, w.k, want_margin=True)
        soft += check_index_sets(got.cpu().numpy()[:, g:g + 1], want, margin)
    print(f"cfg3, KV head {g}: scores within 3e-5, near-tie index disagreements {soft}")


def _scores64(q, k, scale):
    """Anchor Scores of K and V in float64: [B, Hkv, N] each."""
    (B, Hq, Nq, _), (_, Hkv, N, _) = q.shape, k.shape
    s = scale * (q.double() @ k.double().repeat_interleave(Hq // Hkv, dim=1).transpose(2, 3).contiguous())
    a = s.masked_fill(torch.arange(N, device="cuda")[None, :] > torch.arange(N - Nq, N, device="cuda")[:, None], -float("inf")).softmax(-1)
    per_head = (a * (1 - a) * q.double().norm(dim=-1)[..., None]).sum(2), a.sum(2)
    return [x.view(B, Hkv, -1, N).sum(2) for x in per_head]


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(1, 16, 8, 1030, 1030), (1, 16, 8, 1100, 1100), (1, 8, 4, 1500, 1500), (1, 32, 8, 900, 900)])
def test_row_statistics_of_every_call(B, Hq, Hkv, N, Nq):
    """Workgroups whose waves differ in length, several in a row: a wave that is ahead must not write the third key tile while another
    reads the first (that made one call in two wrong by 1e-3).  Bound: the 3e-5 that scores are held to."""
    gen = torch.Generator(device="cuda").manual_seed(N)
    q, k = (torch.randn((B, h, n, 128), dtype=torch.float16, device="cuda", generator=gen) for h, n in ((Hq, Nq), (Hkv, N)))
    want = _scores64(q, k, 128 ** -0.5)
    for _ in range(8):
        _, _, *got = antkv.anchor_select(antkv.Geometry(B, Hq, Hkv, 8), q, k, 128 ** -0.5, 4)
        for a, b in zip(got, want):
            assert ((a.double() - b).abs() / b).max().item() <= 3e-5


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(1, 4, 1, 257, 257), (1, 4, 1, 500, 500), (1, 8, 2, 1201, 1201), (1, 16, 8, 1031, 1031), (3, 8, 8, 1025, 1025),
                                           (2, 16, 8, 700, 650), (1, 32, 8, 2100, 2100), (1, 4, 1, 1000, 255)])
def test_column_sums_in_parts(B, Hq, Hkv, N, Nq):
    """Key blocks whose steps are dealt to two, four and eight workgroups, parts without a step among them, against one workgroup per
    block, which a workspace without room for the parts' sums leaves.  The parts' sums are fp64: the fp32 scores differ by their
    last rounding at most."""
    gen = torch.Generator(device="cuda").manual_seed(N + Hq)
    rnd = lambda *s: torch.randn(s, dtype=torch.float16, device="cuda", generator=gen)
    q, k, lib = rnd(B, Hq, Nq, 128), rnd(B, Hkv, N, 128), antkv.load_library()
    g = antkv.Geometry(B, Hq, Hkv, 8).c()
    need = lib.antkv_anchor_select_workspace(ctypes.byref(g), N, Nq, 0)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    res, want = [], _scores64(q, k, 128 ** -0.5)
    for cut in (0, 256):
        ws = torch.full((need // 4,), float("nan"), device="cuda")
        for _ in range(3):                                     # (on what the call before left, too)
            ans = [torch.full((B, Hkv, N), float("nan"), device="cuda") for _ in range(2)]
            rc = lib.antkv_anchor_select(ctypes.byref(g), p(q), p(k), N, Nq, 128 ** -0.5, 0, None, None, p(ans[0]), p(ans[1]), None, None,
                                         p(ws), need - cut, None)
            if cut and rc == 3:                                # (phase 1's partials are larger than the parts' sums)
                return
            assert rc == 0
            for a, b in zip(ans, want):
                assert ((a.double() - b).abs() / b).max().item() <= 3e-5
        res.append(ans)
    for a, b in zip(*res):
        assert ((a - b).abs() <= 2.0 ** -23 * b.abs()).all()


def test_column_sums_in_parts_on_any_workspace():
    """Pairs of small integers, as index lists and counters leave them, where the arrival counters lie: the result is that of a
    workspace of zeros, bit for bit (the parts are added up in their order)."""
    B, Hq, Hkv, N = 1, 8, 2, 1201
    gen = torch.Generator(device="cuda").manual_seed(2)
    q, k = (torch.randn((B, h, N, 128), dtype=torch.float16, device="cuda", generator=gen) for h in (Hq, Hkv))
    lib, g = antkv.load_library(), antkv.Geometry(B, Hq, Hkv, 8).c()
    need = lib.antkv_anchor_select_workspace(ctypes.byref(g), N, N, 0)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    ws, word = torch.zeros((need // 8,), dtype=torch.int64, device="cuda"), torch.arange(need // 8, device="cuda") % 16
    ans, want = ([torch.empty((B, Hkv, N), device="cuda") for _ in range(2)] for _ in range(2))
    call = lambda out: lib.antkv_anchor_select(ctypes.byref(g), p(q), p(k), N, N, 128 ** -0.5, 0, None, None, p(out[0]), p(out[1]), None, None,
                                               p(ws), need, None)
    assert call(want) == 0
    wrong = torch.zeros((), dtype=torch.int64, device="cuda")
    for high in range(0, 4096, 16):
        ws.copy_((high + word) << 32 | 1 + word % 3)
        assert call(ans) == 0
        wrong += sum((a != b).sum() for a, b in zip(ans, want))
    assert wrong.item() == 0


@pytest.mark.parametrize("B,Hq,Hkv,N,Nq", [(23, 8, 8, 300, 32), (24, 32, 8, 33, 32), (28, 32, 8, 300, 32), (48, 16, 8, 257, 33), (400, 4, 1, 150, 7),
                                           (100, 8, 8, 1031, 128)])
def test_window_of_many_pairs(B, Hq, Hkv, N, Nq):
    """A window's Anchor Score on either side of the number of pairs from which a wave has two key tiles, and with one workgroup per
    pair; ragged keys and queries, the diagonal inside the last tiles.  Bound: the 3e-5 that scores are held to."""
    gen = torch.Generator(device="cuda").manual_seed(N)
    q, k = (torch.randn((B, h, n, 128), dtype=torch.float16, device="cuda", generator=gen) for h, n in ((Hq, Nq), (Hkv, N)))
    _, _, *got = antkv.anchor_select(antkv.Geometry(B, Hq, Hkv, 8), q, k, 128 ** -0.5, 4)
    for a, b in zip(got, _scores64(q, k, 128 ** -0.5)):
        assert ((a.double() - b).abs() / b).max().item() <= 3e-5
