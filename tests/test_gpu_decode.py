"""GPU parity: decode attention over VQ codes + FP16 anchors, and the decode-time Anchor Score + re-selection."""
import numpy as np
import pytest
import torch

import paper_2506_19505_amd as antkv
from gpu_util import ATTN_TOL, attn_tol_for_range, check_index_sets, dev, rel_l2_rows, table_range
from workloads import (CONFIGS, anchor_count, make_codebooks, make_decode_query, make_qkv, normal_fp16,
                       random_anchor_sets, random_codes)

pytestmark = pytest.mark.gpu


def _cache_from_kv(oracle, seed, B, Hq, Hkv, N, d, k_k, k_v, anchors="score"):
    """A full synthetic cache built the way the method builds it, all on the CPU side (oracle + generator)."""
    qwin, k, v = make_qkv(seed, B, Hq, Hkv, N, min(N, 32), 128)
    cbk, cbv = make_codebooks(seed, k, d, 256, "k", max_sample=2048), make_codebooks(seed, v, d, 256, "v", max_sample=2048)
    ck, cv = oracle.encode(k, cbk).astype(np.uint8), oracle.encode(v, cbv).astype(np.uint8)
    if anchors == "score":
        ak, av = oracle.anchor_score(qwin, k, 1 / np.sqrt(128))
        ik, iv = oracle.topk(ak, k_k), oracle.topk(av, k_v)
    else:
        ik, iv = random_anchor_sets(seed, "k", B, Hkv, N, k_k), random_anchor_sets(seed, "v", B, Hkv, N, k_v)
    rk = np.take_along_axis(k, ik[..., None].astype(np.int64), axis=2) if k_k else np.zeros((B, Hkv, 0, 128), np.float16)
    rv = np.take_along_axis(v, iv[..., None].astype(np.int64), axis=2) if k_v else np.zeros((B, Hkv, 0, 128), np.float16)
    q = make_decode_query(seed, B, Hq, 128)
    return dict(q=q, ck=ck, cv=cv, cbk=cbk, cbv=cbv, ik=ik.astype(np.int32), rk=rk, iv=iv.astype(np.int32), rv=rv)


def _run_decode(oracle, c, geom, scale, N=None, want_ans=False, k_resel=0):
    t = {n: dev(a) for n, a in c.items()}
    res = antkv.decode_attn(geom, t["q"], scale, t["ck"], t["cv"], t["cbk"], t["cbv"],
                            t["ik"] if c["ik"].shape[-1] else None, t["rk"] if c["ik"].shape[-1] else None,
                            t["iv"] if c["iv"].shape[-1] else None, t["rv"] if c["iv"].shape[-1] else None,
                            N=N, want_ans=want_ans, k_resel=k_resel)
    torch.cuda.synchronize()
    n = c["ck"].shape[2] if N is None else N
    want = oracle.decode_attn(c["q"], c["ck"][:, :, :n], c["cv"][:, :, :n], c["cbk"], c["cbv"], c["ik"], c["rk"],
                              c["iv"], c["rv"], scale, want_ans=want_ans or k_resel > 0)
    return res, want


def _check_out(got, want, what):
    err = rel_l2_rows(got.cpu().numpy(), want)
    print(f"{what}: rel-L2 max {err.max():.2e} mean {err.mean():.2e}")
    assert err.max() <= ATTN_TOL, f"{what}: relative L2 {err.max():.3e} > {ATTN_TOL}"


@pytest.mark.parametrize("d", [4, 8, 16])
@pytest.mark.parametrize("B,Hq,Hkv,N", [(2, 8, 2, 3000), (1, 4, 1, 1237)])
def test_decode_small(oracle, d, B, Hq, Hkv, N):
    k = anchor_count(N)
    c = _cache_from_kv(oracle, 31 + d, B, Hq, Hkv, N, d, k, k)
    got, want = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), 1 / np.sqrt(128))
    _check_out(got, want, f"decode d={d} N={N}")


@pytest.mark.parametrize("B,Hkv,N", [(3, 8, 11300), (3, 1, 90000), (43, 3, 2100), (257, 1, 70)])
def test_decode_pair_counts(oracle, B, Hkv, N):
    """Numbers of (sequence, KV head) pairs that do not divide the 256 workgroups of a launch, and more pairs than that."""
    c = _cache_from_kv(oracle, 36, B, Hkv, Hkv, N, 8, 5, 5, anchors="random")
    got, want = _run_decode(oracle, c, antkv.Geometry(B, Hkv, Hkv, 8), 1 / np.sqrt(128))
    _check_out(got, want, f"decode B={B} Hkv={Hkv} N={N}")


@pytest.mark.parametrize("G", [1, 2])
def test_decode_other_group_sizes(oracle, G):
    B, Hkv, N, d = 1, 2, 700, 8
    c = _cache_from_kv(oracle, 40 + G, B, Hkv * G, Hkv, N, d, 9, 5)
    got, want = _run_decode(oracle, c, antkv.Geometry(B, Hkv * G, Hkv, d), 0.1)
    _check_out(got, want, f"decode G={G}")


@pytest.mark.parametrize("k_k,k_v", [(0, 0), (0, 13), (13, 0), (64, 64), (500, 500)])
def test_decode_anchor_edge_cases(oracle, k_k, k_v):
    """No anchors, one-sided anchors, anchors == all tokens (then codes are ignored)."""
    B, Hq, Hkv, N, d = 1, 4, 1, 500, 8
    c = _cache_from_kv(oracle, 50, B, Hq, Hkv, N, d, k_k, k_v, anchors="random")
    got, want = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), 1 / np.sqrt(128))
    _check_out(got, want, f"decode k_k={k_k} k_v={k_v}")


@pytest.mark.parametrize("B,Hkv,N,k_k,k_v", [(8, 8, 6000, 2000, 1900),    # several anchor tiles per wave, lists held in LDS
                                             (2, 2, 9000, 3500, 3100),    # lists too long for LDS: searched in global memory
                                             (8, 8, 5000, 3300, 40)])     # one long list, one short
def test_decode_long_anchor_lists(oracle, B, Hkv, N, k_k, k_v):
    """Anchor lists that are long for the number of workgroups, with a large overlap between the K and the V list."""
    d, Hq = 8, 4 * Hkv
    c = _cache_from_kv(oracle, 70 + B, B, Hq, Hkv, N, d, k_k, k_v, anchors="random")
    got, want = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), 1 / np.sqrt(128))
    _check_out(got, want, f"decode B={B} N={N} k_k={k_k} k_v={k_v}")


@pytest.mark.parametrize("d", [4, 8, 16])
@pytest.mark.parametrize("gain", [2, 4, 8, 16])
def test_decode_query_gain(oracle, d, gain):
    """Queries 2 .. 16 times larger than the synthetic recipe's (sharper softmax, larger table entries).  The 2e-3
    tolerance holds while the largest table entry stays inside the range that the 15-bit table quantum serves
    (about 14 / 20 / 29 log2-units for d_sub 4 / 8 / 16); beyond it the bound grows with the entry magnitude."""
    B, Hq, Hkv, N = 2, 8, 2, 3000
    k = anchor_count(N)
    c = _cache_from_kv(oracle, 31 + d, B, Hq, Hkv, N, d, k, k)
    c["q"] = (c["q"].astype(np.float32) * gain).astype(np.float16)
    scale = 1 / np.sqrt(128)
    got, want = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), scale)
    err = rel_l2_rows(got.cpu().numpy(), want)
    R = table_range(c["q"], c["cbk"], scale, Hq // Hkv)
    tol = attn_tol_for_range(R, 128 // d, 16256).reshape(err.shape)
    print(f"decode d={d} query gain {gain}: rel-L2 max {err.max():.2e}; table range {R.min():.1f} .. {R.max():.1f}, "
          f"tolerance {tol.min():.1e} .. {tol.max():.1e}")
    assert (err <= tol).all(), f"relative L2 {err.max():.3e}"


@pytest.mark.parametrize("d", [8, 16])
@pytest.mark.parametrize("gain", [1, 4, 16, 64])
def test_decode_wide_table(oracle, d, gain):
    """ANTKV_DECODE_WIDE_TABLE: with the residual entries in the table the plain 2e-3 tolerance holds whatever the query
    magnitude is (here up to 64 times the recipe's), anchors, one-sided lists and a ragged tail included."""
    B, Hq, Hkv, N = 2, 8, 2, 3000 + 37
    k = anchor_count(N)
    c = _cache_from_kv(oracle, 31 + d, B, Hq, Hkv, N, d, k, k // 2)
    c["q"] = (c["q"].astype(np.float32) * gain).astype(np.float16)
    was = antkv.set_decode_options(antkv.DECODE_WIDE_TABLE)
    try:
        got, want = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), 1 / np.sqrt(128))
    finally:
        antkv.set_decode_options(was)
    _check_out(got, want, f"wide table d={d} query gain {gain}")


def _residuals(scale, a, x):
    """Residual entries of the wide table, in its units, for entries c1 * a * x of a table whose largest entry is c1 * a * 16256:
    the kernel's own fp32 steps."""
    f = np.float32
    c1 = f(f(scale) * f(1.4426950408889634))
    val = (f(a) * x.astype(f)) * c1
    r = np.abs(f(a) * f(16256) * c1)
    inv, quantum = f(16256) / r, r / f(16256)
    rest = (val.astype(np.float64) - np.rint(val * inv).astype(np.float64) * np.float64(quantum)).astype(f)
    return np.rint(rest * (inv * f(32512)))


@pytest.mark.parametrize("d", [8, 16])
@pytest.mark.parametrize("scale,a", [(0.004019, 1.0), (0.013349, 1.171875), (0.03955, -1.1328125)])     # R_h 94, 367, 1051
def test_decode_wide_table_residuals_at_half_a_quantum(oracle, d, scale, a):
    """Entries half a quantum above a multiple of it: their residuals reach -16256 units and, with the rounding of the quantum and
    of its reciprocal, a few units more.  Tokens with such entries compete with tokens half a quantum below them, whose V rows
    are -1/2 times theirs: a residual that is off by one quantum shifts the weights by 0.4 % (R_h = 94) to 4.5 % (1051) and the
    output by about three times that."""
    B, Hq, Hkv, M, C = 1, 4, 1, 128 // d, 256
    x = np.arange(16000, 16016) + 0.5
    res = _residuals(scale, a, x)
    x = x[res < -16256]
    assert x.size == 16 and _residuals(scale, a, x - 0.5).min() > -16256
    n = x.size
    hi = np.floor(np.concatenate([x, x - 0.5]) / 8) * 8                       # fp16 holds multiples of 8 and the rest beside them
    cbk = np.zeros((Hkv, M, C, d), np.float16)
    cbk[0, 0, 1:2 * n + 1, 0], cbk[0, 0, 1:2 * n + 1, 1] = hi, np.concatenate([x, x - 0.5]) - hi
    cbk[0, 0, 255, 0] = 16256                                                # sets the range; no token has it
    cbv = normal_fp16(41, "v", (Hkv, M, C, d))
    cbv[:, :, 2] = -0.5 * cbv[:, :, 1]
    N = 64 * n
    ck, cv = np.zeros((B, Hkv, N, M), np.uint8), np.zeros((B, Hkv, N, M), np.uint8)
    ck[..., 0] = 1 + np.arange(N) % (2 * n)
    cv[:] = np.where(np.arange(N) % (2 * n) < n, 1, 2)[None, None, :, None]
    q = np.zeros((B, Hq, 128), np.float16)
    q[0, :, :2] = np.array([a, -a, 1.3125, -1.3125])[:, None]
    none = np.zeros((B, Hkv, 0), np.int32), np.zeros((B, Hkv, 0, 128), np.float16)
    c = dict(q=q, ck=ck, cv=cv, cbk=cbk, cbv=cbv, ik=none[0], rk=none[1], iv=none[0], rv=none[1])
    prev = antkv.set_decode_options(antkv.DECODE_WIDE_TABLE)
    try:
        got, want = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), scale)
    finally:
        antkv.set_decode_options(prev)
    _check_out(got, want, f"wide table, d={d}, R_h {abs(a) * 16256 * scale * 1.4427:.0f}")


def test_decode_tiny_contexts(oracle):
    B, Hq, Hkv, d = 2, 4, 1, 8
    for N in (1, 2, 63, 64, 65):
        c = _cache_from_kv(oracle, 60 + N, B, Hq, Hkv, max(N, 1), d, min(N, 1), min(N, 1), anchors="random")
        got, want = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), 0.2)
        _check_out(got, want, f"decode N={N}")
    # N = 0 inside a larger code tensor: output is defined as zeros
    c = _cache_from_kv(oracle, 61, B, Hq, Hkv, 8, d, 0, 0)
    t = {n: dev(a) for n, a in c.items()}
    out = antkv.decode_attn(antkv.Geometry(B, Hq, Hkv, d), t["q"], 0.2, t["ck"], t["cv"], t["cbk"], t["cbv"],
                            None, None, None, None, N=0)
    assert torch.count_nonzero(out).item() == 0


def test_decode_respects_N_below_capacity(oracle):
    B, Hq, Hkv, d, cap, N = 1, 4, 1, 8, 900, 611
    c = _cache_from_kv(oracle, 62, B, Hq, Hkv, cap, d, 0, 0)
    c["ik"] = np.array([[[3, 600]]], np.int32)
    c["rk"] = normal_fp16(62, "rows_k", (1, 1, 2, 128))
    got, want = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), 0.1, N=N)
    _check_out(got, want, "decode N < N_cap")


def test_decode_identity_codebook_equals_plain_attention(oracle):
    """Lossless VQ (centroid c = token c's sub-vector): the result must be textbook attention on FP16 K, V."""
    B, Hq, Hkv, N, d = 1, 4, 1, 256, 8
    _, k, v = make_qkv(63, B, Hq, Hkv, N, 1, 128)
    cbk = np.ascontiguousarray(k[0].reshape(Hkv, N, 16, d).transpose(0, 2, 1, 3))
    cbv = np.ascontiguousarray(v[0].reshape(Hkv, N, 16, d).transpose(0, 2, 1, 3))
    codes = np.ascontiguousarray(np.broadcast_to(np.arange(N, dtype=np.uint8)[None, None, :, None], (B, Hkv, N, 16)))
    q = make_decode_query(63, B, Hq, 128)
    out = antkv.decode_attn(antkv.Geometry(B, Hq, Hkv, d), dev(q), 1 / np.sqrt(128), dev(codes), dev(codes),
                            dev(cbk), dev(cbv), None, None, None, None)
    qt = torch.from_numpy(q.astype(np.float64))[:, :, None]
    kt = torch.from_numpy(k.astype(np.float64)).repeat_interleave(Hq // Hkv, 1)
    vt = torch.from_numpy(v.astype(np.float64)).repeat_interleave(Hq // Hkv, 1)
    ref = torch.nn.functional.scaled_dot_product_attention(qt, kt, vt)[:, :, 0].numpy()
    _check_out(out, ref, "identity codebook")


def test_decode_tiny_config(oracle):
    """Config 0 end to end on the GPU: encode -> anchor select -> gather -> decode, checked stage by stage."""
    w = CONFIGS["cfg0"]
    qwin, k, v = make_qkv(w.seed, w.B, w.Hq, w.Hkv, w.N, w.Nq_select, w.D)
    cbk, cbv = make_codebooks(w.seed, k, w.d_sub, 256, "k"), make_codebooks(w.seed, v, w.d_sub, 256, "v")
    q = make_decode_query(w.seed, w.B, w.Hq, w.D)
    geom = antkv.Geometry(w.B, w.Hq, w.Hkv, w.d_sub)
    kd, vd = dev(k), dev(v)
    ck, cv = antkv.encode(geom, kd, dev(cbk)), antkv.encode(geom, vd, dev(cbv))
    ik, iv, _, _ = antkv.anchor_select(geom, dev(qwin), kd, w.scale, w.k)
    rk, rv = antkv.gather_rows(geom, kd, ik), antkv.gather_rows(geom, vd, iv)
    out = antkv.decode_attn(geom, dev(q), w.scale, ck, cv, dev(cbk), dev(cbv), ik, rk, iv, rv)
    torch.cuda.synchronize()
    # gather is a copy: exact
    assert np.array_equal(rk.cpu().numpy(), np.take_along_axis(k, ik.cpu().numpy()[..., None].astype(np.int64), axis=2))
    # the oracle consumes the GPU's own codes / anchors here; each stage has its own parity test
    want = oracle.decode_attn(q, ck.cpu().numpy(), cv.cpu().numpy(), cbk, cbv, ik.cpu().numpy(), rk.cpu().numpy(),
                              iv.cpu().numpy(), rv.cpu().numpy(), w.scale)
    _check_out(out, want, "cfg0 pipeline")


def test_decode_headline_config_on_library_built_cache(oracle):
    """Config 2 at full size on the cache the benchmark times: seeded K/V -> the library's encode -> Anchor Score over a
    32-query window -> top-1 % -> gather -> decode (real codes, real anchor positions and rows).  The oracle consumes
    the GPU's own codes and anchors here; each stage has its own parity test."""
    w = CONFIGS["cfg2"]
    qwin, k, v = make_qkv(w.seed, w.B, w.Hq, w.Hkv, w.N, min(w.Nq_select, 32), w.D)
    cbk, cbv = make_codebooks(w.seed, k, w.d_sub, w.C, "k"), make_codebooks(w.seed, v, w.d_sub, w.C, "v")
    q = make_decode_query(w.seed, w.B, w.Hq, w.D)
    geom = antkv.Geometry(w.B, w.Hq, w.Hkv, w.d_sub)
    kd, vd = dev(k), dev(v)
    del k, v
    ck, cv = antkv.encode(geom, kd, dev(cbk)), antkv.encode(geom, vd, dev(cbv))
    ik, iv, _, _ = antkv.anchor_select(geom, dev(qwin), kd, w.scale, w.k, want_scores=False)
    rk, rv = antkv.gather_rows(geom, kd, ik), antkv.gather_rows(geom, vd, iv)
    del kd, vd
    out = antkv.decode_attn(geom, dev(q), w.scale, ck, cv, dev(cbk), dev(cbv), ik, rk, iv, rv)
    torch.cuda.synchronize()
    ikn, ivn = ik.cpu().numpy(), iv.cpu().numpy()
    assert (np.diff(ikn, axis=-1) > 0).all() and (np.diff(ivn, axis=-1) > 0).all(), "anchor lists are sorted and distinct"
    want = oracle.decode_attn(q, ck.cpu().numpy(), cv.cpu().numpy(), cbk, cbv, ikn, rk.cpu().numpy(), ivn, rv.cpu().numpy(), w.scale)
    _check_out(out, want, "cfg2 on the library-built cache")


@pytest.mark.parametrize("name", ["cfg1", "cfg2", "cfg4"])
def test_decode_full_size_cache(oracle, name):
    """Decode at the real cache shapes (cache-shaped random codes, anchors concentrated at head and tail)."""
    w = CONFIGS[name]
    _, ks, vs = make_qkv(w.seed, 1, w.Hq, w.Hkv, 2048, 1, w.D)
    cbk, cbv = make_codebooks(w.seed, ks, w.d_sub, 256, "k"), make_codebooks(w.seed, vs, w.d_sub, 256, "v")
    c = dict(q=make_decode_query(w.seed, w.B, w.Hq, w.D),
             ck=random_codes(w.seed, "k", w.B, w.Hkv, w.N, w.M), cv=random_codes(w.seed, "v", w.B, w.Hkv, w.N, w.M),
             cbk=cbk, cbv=cbv,
             ik=random_anchor_sets(w.seed, "k", w.B, w.Hkv, w.N, w.k), iv=random_anchor_sets(w.seed, "v", w.B, w.Hkv, w.N, w.k),
             rk=normal_fp16(w.seed, "rows_k", (w.B, w.Hkv, w.k, w.D)), rv=normal_fp16(w.seed, "rows_v", (w.B, w.Hkv, w.k, w.D)))
    got, want = _run_decode(oracle, c, antkv.Geometry(w.B, w.Hq, w.Hkv, w.d_sub), w.scale)
    _check_out(got, want, f"{name} decode")


@pytest.mark.parametrize("d,N", [(8, 2500), (16, 4100), (4, 900)])
def test_decode_time_anchor_score_and_reselection(oracle, d, N):
    B, Hq, Hkv = 2, 8, 2
    k = anchor_count(N)
    c = _cache_from_kv(oracle, 70 + d, B, Hq, Hkv, N, d, k, k)
    (out, ans_k, ans_v, rk, rv), (want, ex) = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), 1 / np.sqrt(128),
                                                          k_resel=k)
    _check_out(out, want, f"decode+AnS d={d}")
    gk, gv = ans_k.cpu().numpy().astype(np.float64), ans_v.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(gv, ex["ans_v"], rtol=2e-5, atol=1e-12)
    np.testing.assert_allclose(gk, ex["ans_k"], rtol=2e-5, atol=1e-12)
    np.testing.assert_allclose(gv.sum(-1), Hq // Hkv, rtol=1e-5)
    soft = 0
    for got, score in ((rk, ex["ans_k"]), (rv, ex["ans_v"])):
        wi, margin = oracle.topk(score, k, want_margin=True)
        soft += check_index_sets(got.cpu().numpy(), wi, margin, "re-selection")
    print(f"re-selection near-tie disagreements: {soft}")


@pytest.mark.parametrize("d,C", [(8, 256), (32, 4096)])
@pytest.mark.parametrize("Hkv,N", [(2, 16384), (2, 16385), (2, 16388), (2, 32768), (2, 32772), (32, 16388)])
def test_reselection_is_the_top_k_of_the_scores(oracle, d, C, Hkv, N):
    """Both sides of the sizes at which the selection goes from one launch to counted scores: the sets are those of the scores
    that the call returns, exactly."""
    geom = antkv.Geometry(1, 4 * Hkv, Hkv, d, n_centroids=C)
    gen = torch.Generator(device="cuda").manual_seed(N)
    normal = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    codes = torch.randint(0, 256, (1, Hkv, N, geom.code_bytes), dtype=torch.uint8, device="cuda", generator=gen)
    cb = normal(Hkv, 128 // d, C, d)
    idx = torch.arange(0, N, 97, dtype=torch.int32, device="cuda").expand(1, Hkv, -1).contiguous()
    rows = normal(1, Hkv, idx.shape[-1], 128)
    _, ans_k, ans_v, rk, rv = antkv.decode_attn(geom, normal(1, 4 * Hkv, 128), 1 / np.sqrt(128), codes, codes, cb, cb, idx, rows,
                                                idx, rows, N=N, k_resel=N // 100)
    for got, score in ((rk, ans_k), (rv, ans_v)):
        assert np.array_equal(got.cpu().numpy(), oracle.topk(score.cpu().numpy(), N // 100))


@pytest.mark.parametrize("k_v", [0, 13])
def test_decode_time_anchor_score_without_key_anchors(oracle, k_v):
    """Scores and re-selection on a cache whose K list is empty (null list pointers): nothing of that list may be read."""
    B, Hq, Hkv, N, d = 1, 4, 1, 700, 8
    c = _cache_from_kv(oracle, 55, B, Hq, Hkv, N, d, 0, k_v, anchors="random")
    k_resel = 9
    (out, ans_k, ans_v, rk, rv), (want, ex) = _run_decode(oracle, c, antkv.Geometry(B, Hq, Hkv, d), 1 / np.sqrt(128),
                                                          k_resel=k_resel)
    _check_out(out, want, f"decode+AnS without K anchors, k_v={k_v}")
    np.testing.assert_allclose(ans_v.cpu().numpy().astype(np.float64), ex["ans_v"], rtol=2e-5, atol=1e-12)
    np.testing.assert_allclose(ans_k.cpu().numpy().astype(np.float64), ex["ans_k"], rtol=2e-5, atol=1e-12)
    for got, score in ((rk, ex["ans_k"]), (rv, ex["ans_v"])):
        wi, margin = oracle.topk(score, k_resel, want_margin=True)
        check_index_sets(got.cpu().numpy(), wi, margin, "re-selection")


@pytest.mark.parametrize("d", [4, 8, 16])
@pytest.mark.parametrize("G", [1, 2, 4])
def test_decode_time_anchor_score_of_an_infinite_key(oracle, d, G):
    """An anchored key, or centroid, with an infinity that every head scores -inf weighs nothing: both its scores are 0 and the other
    tokens' are those beside a key so far off that its weight is 0 in float64.  Heads that the group does not have add nothing."""
    B, Hkv, N, k, at = 1, 2, 900, 9, 4
    c = _cache_from_kv(oracle, 60 + G, B, G * Hkv, Hkv, N, d, k, 5)
    c["q"][..., 0] = 1 + np.abs(c["q"][..., 0])
    geom = antkv.Geometry(B, G * Hkv, Hkv, d)
    c["rk"][:, :, at, 0] = -60000
    _, (_, want) = _run_decode(oracle, c, geom, 1 / np.sqrt(128), want_ans=True)
    assert (np.take_along_axis(want["ans_v"], c["ik"].astype(np.int64), axis=2)[:, :, at] == 0).all()
    t = {n: dev(a) for n, a in c.items()}
    t["rk"][:, :, at, 0] = -float("inf")
    out, ans_k, ans_v, *_ = antkv.decode_attn(geom, t["q"], 1 / np.sqrt(128), t["ck"], t["cv"], t["cbk"], t["cbv"], t["ik"], t["rk"], t["iv"],
                                              t["rv"], want_ans=True)
    assert torch.isfinite(out).all()
    np.testing.assert_allclose(ans_v.cpu().numpy(), want["ans_v"], rtol=3e-5, atol=1e-12)
    np.testing.assert_allclose(ans_k.cpu().numpy(), want["ans_k"], rtol=3e-5, atol=1e-12)
    c["cbk"][:, 0, c["ck"][0, 0, 5, 0], 0] = -60000            # (the codes' table: the attention itself has none for such a centroid)
    _, (_, want) = _run_decode(oracle, c, geom, 1 / np.sqrt(128), want_ans=True)
    t["cbk"] = dev(np.where(c["cbk"] == -60000, np.float16(-np.inf), c["cbk"]))
    _, ans_k, ans_v, *_ = antkv.decode_attn(geom, t["q"], 1 / np.sqrt(128), t["ck"], t["cv"], t["cbk"], t["cbv"], t["ik"], t["rk"], t["iv"],
                                            t["rv"], want_ans=True)
    np.testing.assert_allclose(ans_v.cpu().numpy(), want["ans_v"], rtol=3e-5, atol=1e-12)
    np.testing.assert_allclose(ans_k.cpu().numpy(), want["ans_k"], rtol=3e-5, atol=1e-12)


def test_extreme_context_reselection(oracle):
    """Config 4: 840000-token context at 0.5 bit, decode step plus anchor re-selection of 8400 tokens."""
    w = CONFIGS["cfg4"]
    _, ks, vs = make_qkv(w.seed, 1, w.Hq, w.Hkv, 2048, 1, w.D)
    cbk, cbv = make_codebooks(w.seed, ks, w.d_sub, 256, "k"), make_codebooks(w.seed, vs, w.d_sub, 256, "v")
    c = dict(q=make_decode_query(w.seed, w.B, w.Hq, w.D),
             ck=random_codes(w.seed, "k", w.B, w.Hkv, w.N, w.M), cv=random_codes(w.seed, "v", w.B, w.Hkv, w.N, w.M),
             cbk=cbk, cbv=cbv,
             ik=random_anchor_sets(w.seed, "k", w.B, w.Hkv, w.N, w.k), iv=random_anchor_sets(w.seed, "v", w.B, w.Hkv, w.N, w.k),
             rk=normal_fp16(w.seed, "rows_k", (w.B, w.Hkv, w.k, w.D)), rv=normal_fp16(w.seed, "rows_v", (w.B, w.Hkv, w.k, w.D)))
    (out, ans_k, ans_v, rk, rv), (want, ex) = _run_decode(oracle, c, antkv.Geometry(w.B, w.Hq, w.Hkv, w.d_sub),
                                                          w.scale, k_resel=w.k)
    _check_out(out, want, "cfg4 decode")
    soft = 0
    for got, score in ((rk, ex["ans_k"]), (rv, ex["ans_v"])):
        wi, margin = oracle.topk(score, w.k, want_margin=True)
        soft += check_index_sets(got.cpu().numpy(), wi, margin, "cfg4 re-selection")
    print(f"cfg4 re-selection near-tie disagreements: {soft}")


def test_decode_workspace_reuse_across_shapes(oracle):
    """One workspace serves calls of different context lengths in turn (the number of workgroups per (b, g), and with
    it the arrival count the in-kernel merge waits for, changes from call to call)."""
    B, Hq, Hkv, d = 1, 8, 2, 8
    geom = antkv.Geometry(B, Hq, Hkv, d)
    scale = 1 / np.sqrt(128)
    N_big = 9000
    c = _cache_from_kv(oracle, 77, B, Hq, Hkv, N_big, d, 40, 40, anchors="random")
    t = {n: dev(a) for n, a in c.items()}
    ws = antkv.DecodeWorkspace(geom, N_big, 40, 40, 0, t["q"].device)
    ws.buf.fill_(0x5A)                                    # arbitrary content: nothing may rely on zeros
    for rep, n in enumerate((9000, 700, 9000, 130, 4200, 4200)):
        keep_k, keep_v = c["ik"] < n, c["iv"] < n          # anchors inside the shorter context (lists are ascending)
        kk = int(keep_k.sum(-1).min()); kv = int(keep_v.sum(-1).min())
        ik, iv = c["ik"][..., :kk], c["iv"][..., :kv]
        rk, rv = c["rk"][:, :, :kk], c["rv"][:, :, :kv]
        got = antkv.decode_attn(geom, t["q"], scale, t["ck"], t["cv"], t["cbk"], t["cbv"],
                                dev(ik) if kk else None, dev(rk) if kk else None, dev(iv) if kv else None,
                                dev(rv) if kv else None, N=n, workspace=ws)
        torch.cuda.synchronize()
        want = oracle.decode_attn(c["q"], c["ck"][:, :, :n], c["cv"][:, :, :n], c["cbk"], c["cbv"], ik, rk, iv, rv, scale)
        _check_out(got, want, f"reused workspace, call {rep}, N={n}")


def test_decode_repeated_on_one_workspace(oracle):
    """The same step 200 times back to back on one workspace, no host synchronisation in between: every launch's last
    workgroup must merge this launch's partials (arrival words carry the launch tag; partials are written and read at
    device scope).  A stale or half-written partial would show as a large deviation; the run-to-run differences that
    remain come from the order in which waves pull tiles (fp32 sums in another order) and stay at rounding level."""
    B, Hq, Hkv, N, d = 4, 32, 8, 20000, 8
    k = anchor_count(N)
    c = _cache_from_kv(oracle, 77, B, Hq, Hkv, N, d, k, k, anchors="random")
    t = {n: dev(a) for n, a in c.items()}
    geom = antkv.Geometry(B, Hq, Hkv, d)
    ws = antkv.DecodeWorkspace(geom, N, k, k, 0, "cuda")
    outs = torch.empty((200, B, Hq, 128), dtype=torch.float16, device="cuda")
    for i in range(200):
        antkv.decode_attn(geom, t["q"], 0.1, t["ck"], t["cv"], t["cbk"], t["cbv"], t["ik"], t["rk"], t["iv"], t["rv"],
                          out=outs[i], workspace=ws)
    torch.cuda.synchronize()
    got = outs.cpu().numpy().astype(np.float64)
    want = oracle.decode_attn(c["q"], c["ck"], c["cv"], c["cbk"], c["cbv"], c["ik"], c["rk"], c["iv"], c["rv"], 0.1)
    err = np.linalg.norm(got - want[None], axis=-1) / np.linalg.norm(want, axis=-1)[None]
    spread = np.linalg.norm(got - got[:1], axis=-1) / np.linalg.norm(want, axis=-1)[None]
    print(f"200 launches: rel-L2 to the oracle max {err.max():.2e}; launch-to-launch spread max {spread.max():.2e}, "
          f"bit-identical launches {(np.abs(got - got[:1]).reshape(200, -1).max(axis=1) == 0).sum()} of 200")
    assert err.max() <= ATTN_TOL
    assert spread.max() <= 1e-3          # one fp16 unit in the last place of the largest channels


@pytest.mark.parametrize("d,C,B,N", [(8, 256, 2, 1237), (16, 256, 1, 4100), (32, 4096, 2, 1500), (16, 4096, 4, 700)])
def test_decode_on_any_workspace(d, C, B, N):
    """Pairs of small integers, as index lists and counters leave them, where the arrival words lie: no workgroup takes them for arrivals
    and merges parts that are not stored yet.  Sums in a fixed order, so the result is that of a workspace of zeros, bit for bit."""
    Hq, Hkv, k, M = 8, 4, 20, 128 // d
    gen = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    codes = [torch.randint(0, 256, (B, Hkv, N, M if C == 256 else 3 * M // 2), dtype=torch.uint8, device="cuda", generator=gen) for _ in range(2)]
    idx = [torch.rand((B, Hkv, N), device="cuda", generator=gen).argsort(dim=-1)[..., :k].sort(dim=-1).values.int() for _ in range(2)]
    geom = antkv.Geometry(B, Hq, Hkv, d, n_centroids=C)
    args = (geom, rnd(B, Hq, 128), 128 ** -0.5, *codes, rnd(Hkv, M, C, d), rnd(Hkv, M, C, d), idx[0], rnd(B, Hkv, k, 128), idx[1], rnd(B, Hkv, k, 128))
    ws = antkv.DecodeWorkspace(geom, N, k, k, 0, "cuda")
    words = ws.buf[:ws.buf.numel() // 8 * 8].view(torch.int64)
    low = torch.arange(words.numel(), device="cuda")
    old = antkv.set_decode_options(antkv.DECODE_FIXED_ORDER)
    try:
        words.zero_()
        want, wrong = antkv.decode_attn(*args, workspace=ws), torch.zeros((), dtype=torch.int64, device="cuda")
        for high in range(0, 8192, 4):
            words.copy_((high + low % 4) << 32 | 1 + low % 3)
            wrong += (antkv.decode_attn(*args, workspace=ws) != want).sum()
    finally:
        antkv.set_decode_options(old)
    assert wrong.item() == 0


def test_decode_graph_replay(oracle):
    """The decode step captured into a HIP graph and replayed: every replay must equal the eager result for the inputs
    of that moment (the launch tag of the arrival words is frozen in the captured launch)."""
    B, Hq, Hkv, d, N = 2, 8, 2, 8, 5000
    geom = antkv.Geometry(B, Hq, Hkv, d)
    scale = 1 / np.sqrt(128)
    c = _cache_from_kv(oracle, 91, B, Hq, Hkv, N, d, 50, 50, anchors="random")
    t = {n: dev(a) for n, a in c.items()}
    ws = antkv.DecodeWorkspace(geom, N, 50, 50, 0, t["q"].device)
    out = torch.empty((B, Hq, 128), dtype=torch.float16, device=t["q"].device)
    q_live = t["q"].clone()

    def step():
        antkv.decode_attn(geom, q_live, scale, t["ck"], t["cv"], t["cbk"], t["cbv"], t["ik"], t["rk"], t["iv"], t["rv"],
                          out=out, workspace=ws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()                                            # warm-up outside the capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(4):
        q_np = make_decode_query(500 + rep, B, Hq, 128)
        q_live.copy_(dev(q_np))
        graph.replay()
        torch.cuda.synchronize()
        got_graph = out.clone()
        step()                                            # eager launch between the replays, same workspace
        torch.cuda.synchronize()
        # (tiles are handed to waves dynamically, so two runs may differ in the last bits of the fp32 sums)
        diff = rel_l2_rows(got_graph.cpu().numpy(), out.cpu().numpy().astype(np.float64))
        assert diff.max() <= 1e-3, f"replay {rep} differs from the eager result: {diff.max():.2e}"
        want = oracle.decode_attn(q_np, c["ck"], c["cv"], c["cbk"], c["cbv"], c["ik"], c["rk"], c["iv"], c["rv"], scale)
        _check_out(got_graph, want, f"graph replay {rep}")


def test_decode_random_shapes(oracle):
    """Twenty seeded random geometries: batch, heads, group size, sub-vector width, context length around tile and
    split boundaries, anchor counts (including 0, a single one and lists that share tokens), spare capacity."""
    rng = np.random.default_rng(2024)
    lengths = [1, 2, 63, 64, 65, 127, 129, 1023, 1024, 1025, 2047, 2049, 3000, 4097, 6000]
    _, ks, vs = make_qkv(77, 1, 4, 4, 1024, 1, 128)
    books = {d: (make_codebooks(77, ks, d, 256, "k", max_sample=1024), make_codebooks(77, vs, d, 256, "v", max_sample=1024))
             for d in (4, 8, 16)}
    for case in range(20):
        B, Hkv, G = int(rng.integers(1, 4)), int(rng.integers(1, 4)), int(rng.choice([1, 2, 4]))
        d = int(rng.choice([4, 8, 16]))
        N = int(rng.choice(lengths))
        N_cap = N + int(rng.choice([0, 0, 1, 37]))
        k_k = int(rng.choice([0, 1, min(N, 5), min(N, max(1, N // 50))]))
        k_v = int(rng.choice([0, 1, min(N, 9), min(N, max(1, N // 70))]))
        Hq, M = Hkv * G, 128 // d
        seed = 500 + case
        c = dict(q=make_decode_query(seed, B, Hq, 128),
                 ck=random_codes(seed, "k", B, Hkv, N_cap, M), cv=random_codes(seed, "v", B, Hkv, N_cap, M),
                 cbk=books[d][0][np.arange(Hkv) % 4], cbv=books[d][1][np.arange(Hkv) % 4],
                 ik=random_anchor_sets(seed, "k", B, Hkv, N, k_k), iv=random_anchor_sets(seed, "v", B, Hkv, N, k_v),
                 rk=normal_fp16(seed, "rows_k", (B, Hkv, k_k, 128)), rv=normal_fp16(seed, "rows_v", (B, Hkv, k_v, 128)))
        if k_k and k_v:                                        # let the two lists share their first entries
            n_common = min(k_k, k_v, 3)
            for b in range(B):
                for g in range(Hkv):
                    merged = np.union1d(c["iv"][b, g][n_common:], c["ik"][b, g][:n_common])
                    if merged.size >= k_v:
                        c["iv"][b, g] = np.sort(merged)[:k_v]
        geom = antkv.Geometry(B, Hq, Hkv, d)
        res, want = _run_decode(oracle, c, geom, 1 / np.sqrt(128), N=N)
        _check_out(res, want, f"case {case}: B{B} Hkv{Hkv} G{G} d{d} N{N}/{N_cap} anchors {k_k}/{k_v}")


def _step_in_fixed_order(d, N):
    """A decode step whose ranges hold at most one tile per wave: nothing in it is handed out dynamically."""
    B, Hq, Hkv, M, k = 1, 8, 2, 128 // d, 70
    geom = antkv.Geometry(B, Hq, Hkv, d)
    codes = [dev(random_codes(9, w, B, Hkv, N, M)) for w in "kv"]
    books = [dev(normal_fp16(9, w, (Hkv, M, 256, d))) for w in "kv"]
    idx = [dev(random_anchor_sets(9, w, B, Hkv, N, k).astype(np.int32)) for w in "kv"]
    rows = [dev(normal_fp16(9, "rows_" + w, (B, Hkv, k, 128))) for w in "kv"]
    q = dev(normal_fp16(9, "q_decode", (B, Hq, 128)))
    return antkv.decode_attn(geom, q, 1 / np.sqrt(128), *codes, *books, idx[0], rows[0], idx[1], rows[1]).cpu().numpy()


# 3 and 20 ranges: sums over the waves, over eight slots at a time and over the slots that are left
@pytest.mark.parametrize("d,N,bits", [(4, 2500, "77a12fd33050ce04"), (8, 2500, "7f583cc3e891b0e0"), (16, 2500, "6f110897e67013e2"),
                                      (4, 20000, "180519fc40281f89"), (8, 20000, "6d93124f18e111dc"), (16, 20000, "b60fb7e787f6cc4c")])
def test_decode_rounding_is_pinned(d, N, bits):
    """The assignment of tiles to waves (each wave rounds its fp16 weights against a reference of its own), the rounding of the
    table entries and the order of the fp32 sums are part of the result: a short step repeats itself bit for bit, from one
    version of the library to the next.  `bits` is the digest of the output."""
    import hashlib

    assert hashlib.sha256(_step_in_fixed_order(d, N).tobytes()).hexdigest()[:16] == bits
