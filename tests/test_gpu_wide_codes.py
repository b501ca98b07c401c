"""GPU parity for the 12-bit codebooks (paper Sec. 4: 4096 centroids with 32-channel sub-vectors, "0.375 bit", and with
16-channel sub-vectors, "0.75 bit"): encode, decode attention, append and decode-time Anchor Score against the CPU
oracle, which is generic in the codebook size."""
import numpy as np
import pytest
import torch

import paper_2506_19505_amd as antkv
from gpu_util import check_codes, dev, pack12, unpack12
from workloads import make_codebooks, make_qkv

pytestmark = pytest.mark.gpu

C = 4096


class Books(tuple):
    """(K codebook, V codebook) + the format: d = sub-vector width, M = codes per token, nbytes = 3 M / 2."""
    def __new__(cls, k, v, d):
        self = super().__new__(cls, (k, v))
        self.d, self.M, self.nbytes = d, 128 // d, 128 // d * 3 // 2
        return self


@pytest.fixture(scope="module", params=[32, 16], ids=["d32", "d16"])
def books(request):
    """K and V codebooks [2 KV heads][M][4096][d] picked from 6000 synthetic rows."""
    d = request.param
    _, k, v = make_qkv(81, 1, 2, 2, 6000, 1, 128)
    return Books(make_codebooks(81, k, d, C, "k", max_sample=6000), make_codebooks(81, v, d, C, "v", max_sample=6000), d)


def test_pack_unpack_roundtrip():
    rng = np.random.default_rng(0)
    c = rng.integers(0, 4096, size=(3, 5, 4))
    assert np.array_equal(unpack12(pack12(c)), c) and pack12(c).shape == (3, 5, 6)
    assert pack12(np.array([[0x123, 0x456, 0x789, 0xABC]])).tolist() == [[0x23, 0x61, 0x45, 0x89, 0xC7, 0xAB]]
    c8 = rng.integers(0, 4096, size=(2, 7, 8))
    assert np.array_equal(unpack12(pack12(c8)), c8) and pack12(c8).shape == (2, 7, 12)
    assert np.array_equal(pack12(c8)[..., :6], pack12(c8[..., :4])) and np.array_equal(pack12(c8)[..., 6:], pack12(c8[..., 4:]))


@pytest.mark.parametrize("B,n", [(1, 700), (2, 70), (1, 257)])
def test_encode12_matches_oracle(oracle, books, B, n):
    _, x, _ = make_qkv(82 + n, B, 2, 2, n, 1, 128, want_v=False)
    geom = antkv.Geometry(B, 2, 2, books.d, n_centroids=C)
    codes = antkv.encode(geom, dev(x), dev(books[0]))
    torch.cuda.synchronize()
    assert codes.shape == (B, 2, n, books.nbytes)
    got = unpack12(codes.cpu().numpy())
    want, margin = oracle.encode(x, books[0], want_margin=True)
    soft = check_codes(got, want, margin)
    print(f"n={n}: near-tie disagreements {soft} of {want.size}")


def test_encode12_duplicate_centroids_and_offsets(oracle, books):
    """Exact ties go to the lower index; token_offset / N_cap place the rows."""
    cb = books[0].copy()
    cb[:, :, 4000:4096] = cb[:, :, 100:196]                   # 96 exact duplicates far apart
    cb[:, :, 33] = cb[:, :, 32]                                 # and one inside a tile
    _, x, _ = make_qkv(83, 1, 2, 2, 300, 1, 128, want_v=False)
    geom = antkv.Geometry(1, 2, 2, books.d, n_centroids=C)
    buf = torch.full((1, 2, 400, books.nbytes), 0xEE, dtype=torch.uint8, device="cuda")
    antkv.encode(geom, dev(x), dev(cb), codes=buf, token_offset=50)
    got_all = buf.cpu().numpy()
    assert (got_all[:, :, :50] == 0xEE).all() and (got_all[:, :, 350:] == 0xEE).all()
    got = unpack12(got_all[:, :, 50:350])
    want, margin = oracle.encode(x, cb, want_margin=True)
    check_codes(got, want, margin)
    assert not np.isin(got, np.arange(4000, 4096)).any() and not (got == 33).any()


@pytest.mark.parametrize("B,n", [(1, 1), (1, 31), (2, 513), (2, 17003), (2, 33001), (3, 44007)])
def test_encode12_work_splits(oracle, books, B, n):
    """From one token (all waves of a workgroup on one group) to several groups per wave and rounds of workgroups; rows at
    the ends and a sample between against the oracle, ties between far tiles, neighbours and half-waves included."""
    cb = books[0].copy()
    cb[:, :, 2048 + 7:2048 + 2047] = cb[:, :, 7:2047]           # most centroids twice
    cb[:, :, 4] = cb[:, :, 0]                                   # rows 0 and 4 of a tile belong to different half-waves
    x = np.random.default_rng(n).standard_normal((B, 2, n, 128)).astype(np.float16)
    x[:, :, :2, :books.d] = cb[:, 0, 4][None, :, None]
    geom = antkv.Geometry(B, 2, 2, books.d, n_centroids=C)
    got = unpack12(antkv.encode(geom, dev(x), dev(cb)).cpu().numpy())
    rows = np.unique(np.concatenate([np.arange(min(n, 70)), np.arange(max(0, n - 70), n),
                                     np.random.default_rng(n + 1).integers(0, n, 300)]))
    want, margin = oracle.encode(np.ascontiguousarray(x[:, :, rows]), cb, want_margin=True)
    check_codes(got[:, :, rows], want, margin)
    assert (got[:, :, :2, 0] != 4).all() and not np.isin(got, np.arange(2048 + 7, 2048 + 2047)).any()


def test_encode12_more_tokens_than_one_launch_takes(books):
    """The tokens of one head beyond what the grid's second axis (65536 chunks of 1536 or 2048 tokens) holds: rows at the ends and
    at every seam get the codes that a call on them alone gives."""
    n, off = 65536 * (1536 if books.d == 32 else 2048) + 77, 3
    geom = antkv.Geometry(1, 1, 1, books.d, n_centroids=C)
    cb = dev(books[0][:1])
    x = torch.empty((1, 1, n, 128), dtype=torch.float16, device="cuda")
    block = torch.randn((1 << 20, 128), dtype=torch.float16, device="cuda", generator=torch.Generator(device="cuda").manual_seed(4))
    for t in range(0, n, 1 << 20):                             # rows repeat, turned by one more channel each time
        x[0, 0, t:t + (1 << 20)] = block[:min(1 << 20, n - t)].roll(t >> 20, dims=1)
    codes = torch.full((1, 1, n + off + 5, books.nbytes), 0xEE, dtype=torch.uint8, device="cuda")
    antkv.encode(geom, x, cb, codes, off)
    assert (codes[:, :, :off] == 0xEE).all() and (codes[:, :, n + off:] == 0xEE).all()
    for at in (0, 1 << 26, n - 40000, n):
        lo, hi = max(0, at - 3000), min(n, at + 3000)
        part = antkv.encode(geom, x[:, :, lo:hi].contiguous(), cb)
        assert torch.equal(codes[:, :, off + lo:off + hi], part), (lo, hi)


def _decode_case(oracle, books, seed, B, Hq, Hkv, N, k_k, k_v, N_cap=None, scale=None, range_tolerance=False, tolerance=2e-3):
    from workloads import make_decode_query, normal_fp16
    rng = np.random.default_rng(seed)
    scale = scale or 1.0 / np.sqrt(128)
    N_cap = N_cap or N
    cbk, cbv = books[0][:Hkv], books[1][:Hkv]
    ck = rng.integers(0, C, (B, Hkv, N_cap, books.M)).astype(np.int32)
    cv = rng.integers(0, C, (B, Hkv, N_cap, books.M)).astype(np.int32)
    pick = lambda k: np.stack([[np.sort(rng.choice(N, k, replace=False)) for _ in range(Hkv)]
                               for _ in range(B)]).astype(np.int32).reshape(B, Hkv, k)
    ik, iv = pick(k_k), pick(k_v)
    if k_k and k_v:                                            # make some tokens anchored in both lists
        n_common = min(k_k, k_v) // 3
        for b in range(B):
            for g in range(Hkv):
                both = np.union1d(iv[b, g][n_common:], ik[b, g][:n_common])
                extra = np.setdiff1d(np.arange(N), both)[:k_v - both.size]
                iv[b, g] = np.sort(np.concatenate([both, extra]))[:k_v]
    rk = normal_fp16(seed, "rows_k", (B, Hkv, k_k, 128))
    rv = normal_fp16(seed, "rows_v", (B, Hkv, k_v, 128))
    q = make_decode_query(seed, B, Hq, 128)
    geom = antkv.Geometry(B, Hq, Hkv, books.d, n_centroids=C)
    out = antkv.decode_attn(geom, dev(q), scale, dev(pack12(ck)), dev(pack12(cv)), dev(cbk), dev(cbv),
                            dev(ik) if k_k else None, dev(rk) if k_k else None,
                            dev(iv) if k_v else None, dev(rv) if k_v else None, N=N)
    torch.cuda.synchronize()
    want = oracle.decode_attn(q, ck[:, :, :N], cv[:, :, :N], cbk, cbv, ik, rk, iv, rv, scale)
    got = out.cpu().numpy().astype(np.float64)
    err = np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)
    tol = np.full(err.shape, tolerance)
    if range_tolerance:
        from gpu_util import attn_tol_for_range, table_range
        R = table_range(q, cbk, scale, Hq // Hkv)
        tol = attn_tol_for_range(R, books.M, 32767)
        print(f"table range {R.min():.1f} .. {R.max():.1f}, tolerance {tol.min():.1e} .. {tol.max():.1e}")
    assert (err <= tol).all(), f"relative L2 {err.max():.3e}"
    print(f"B={B} Hq={Hq} Hkv={Hkv} N={N} anchors {k_k}/{k_v}: rel-L2 max {err.max():.2e}")


@pytest.mark.parametrize("B,Hq,Hkv,N,k_k,k_v", [(2, 8, 2, 3000, 30, 30), (1, 2, 2, 1237, 0, 0), (1, 4, 2, 700, 12, 0),
                                                (1, 4, 1, 900, 0, 9), (1, 8, 2, 70000, 700, 700), (1, 4, 2, 65569, 650, 700), (1, 2, 2, 65537, 700, 3),
                                                (1, 4, 1, 65599, 0, 90)])
def test_decode12_matches_oracle(oracle, books, B, Hq, Hkv, N, k_k, k_v):
    """Short contexts are scored row by row; two KV heads of more than 65536 tokens go through the table and the gathering stream, also
    with a last range that is not full and with tokens in both lists."""
    _decode_case(oracle, books, 90 + N, B, Hq, Hkv, N, k_k, k_v)


@pytest.mark.parametrize("gain", [2, 4, 8, 16])
def test_decode12_query_gain(oracle, books, gain):
    """Sharper softmax / larger table entries (the scale argument multiplies every score).  A short context has no table: row by row,
    the bound of test_decode12_short_ranges holds at any gain.  Through the table (a longer one), 2e-3 holds while the largest entry
    stays inside the range that the 16-bit quantum serves (about 82 / 58 log2-units for d_sub 32 / 16); beyond it the bound grows
    with the entry magnitude."""
    _decode_case(oracle, books, 94, 2, 8, 2, 3000, 30, 30, scale=gain / np.sqrt(128), tolerance=2.0 ** -10 + 1e-4)
    _decode_case(oracle, books, 94, 1, 8, 2, 65569, 300, 310, scale=gain / np.sqrt(128), range_tolerance=True)


def test_decode12_tiny_contexts_and_capacity(oracle, books):
    for N in (1, 63, 64, 65):
        _decode_case(oracle, books, 95, 1, 4, 2, N, min(N, 2), min(N, 3))
    _decode_case(oracle, books, 96, 1, 4, 2, 500, 5, 5, N_cap=800)
    _decode_case(oracle, books, 97, 1, 4, 2, 300, 300, 300)      # every token anchored in both lists


def _least(ws):
    """The same workspace without room for the weights that adding the values up by code needs.  (One that has no such room is
    refused when it is cut short: a call with this workspace shows that the whole one is used by code.)"""
    ws.buf = ws.buf[:ws.buf.numel() - 256]
    return ws


def _switch(geom):
    """The smallest context whose values are added up by code (one or two heads per KV head: its workspace holds four bytes per
    token and KV head that the gathering kernel does not need)."""
    size = lambda n: antkv.DecodeWorkspace(geom, n, 0, 0, 0, "meta").nbytes
    by_code = lambda n: size(n) - size(64) > 4 * geom.B * geom.Hkv * n
    n = next(n for n in range(1024, 1 << 20, 64) if by_code(n))
    return next(m for m in range(n - 63, n + 1) if by_code(m))


# (ranges of the second kernel: sequences x KV heads x M / 2 workgroups share the chip, the last two shapes in two rounds)
@pytest.mark.parametrize("d,B,Hq,Hkv,N,k_k,k_v", [(32, 16, 8, 8, 14335, 30, 30), (32, 16, 8, 8, 14337, 150, 140), (32, 8, 16, 8, 28673, 0, 290),
                                                  (32, 32, 16, 4, 14400, 145, 0), (16, 8, 8, 8, 8191, 20, 20), (16, 8, 32, 8, 8257, 83, 90),
                                                  (16, 8, 16, 8, 8192, 0, 0), (16, 16, 8, 2, 16449, 700, 1100),
                                                  (32, 24, 8, 8, 16001, 161, 30), (16, 12, 16, 8, 13001, 131, 140)])
def test_decode12_values_by_code(oracle, books, d, B, Hq, Hkv, N, k_k, k_v):
    """Contexts whose values are added up by code, among them ranges of a tile more, less and not quite: against the oracle, and
    against the gathering stream that a smaller workspace leaves (2e-3 is the bound of either against the oracle, so 4e-3)."""
    if d != books.d:
        pytest.skip("the other format's case")
    from workloads import make_decode_query, normal_fp16, random_anchor_sets
    rng = np.random.default_rng(N)
    rep = (Hkv + 1) // 2
    cbk, cbv = np.tile(books[0], (rep, 1, 1, 1))[:Hkv], np.tile(books[1], (rep, 1, 1, 1))[:Hkv]
    ck, cv = (rng.integers(0, C, (B, Hkv, N, books.M), dtype=np.int32) for _ in range(2))
    cv[:, 0] = 5                                               # every token of a head on one sum
    ik, iv = random_anchor_sets(N, "k", B, Hkv, N, k_k), random_anchor_sets(N, "v", B, Hkv, N, k_v)
    rk, rv = normal_fp16(N, "rows_k", (B, Hkv, k_k, 128)), normal_fp16(N, "rows_v", (B, Hkv, k_v, 128))
    q = make_decode_query(N, B, Hq, 128)
    scale = 1.0 / np.sqrt(128)
    geom = antkv.Geometry(B, Hq, Hkv, d, n_centroids=C)
    args = (geom, dev(q), scale, dev(pack12(ck)), dev(pack12(cv)), dev(cbk), dev(cbv), dev(ik) if k_k else None, dev(rk) if k_k else None,
            dev(iv) if k_v else None, dev(rv) if k_v else None)
    by_code = antkv.DecodeWorkspace(geom, N, k_k, k_v, 0, "cuda")
    got = antkv.decode_attn(*args, workspace=by_code)
    assert torch.equal(got, antkv.decode_attn(*args, workspace=by_code))          # integer sums: the same bits again
    got = got.cpu().numpy().astype(np.float64)
    want = oracle.decode_attn(q, ck, cv, cbk, cbv, ik, rk, iv, rv, scale)
    err = np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert err.max() <= 2e-3, err.max()
    gather = antkv.decode_attn(*args, workspace=_least(antkv.DecodeWorkspace(geom, N, k_k, k_v, 0, "cuda"))).cpu().numpy().astype(np.float64)
    assert (np.linalg.norm(got - gather, axis=-1) / np.linalg.norm(want, axis=-1)).max() <= 4e-3
    print(f"d{d} B={B} {Hq}/{Hkv} N={N} anchors {k_k}/{k_v}: rel-L2 max {err.max():.2e}")


def test_decode12_values_by_code_sections_and_unused_centroids(books):
    """Ranges longer than the 1792 tiles whose factors fit LDS, few tokens behind the last whole one; centroids that no token uses
    hold infinities and change nothing.  Against the gathering stream (bound as above)."""
    B, Hkv, N, k = 8, 8, 1792 * 64 * (2 if books.d == 32 else 1) + 70, 1200
    gen = torch.Generator(device="cuda").manual_seed(6)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    codes = torch.randint(0, C - 1, (2, 1, 1, N, books.M), device="cuda", generator=gen)      # code 4095 is not used
    packed = torch.empty((2, B, Hkv, N, books.nbytes), dtype=torch.uint8, device="cuda")
    for m in range(0, books.M, 2):
        w = codes[..., m] | codes[..., m + 1] << 12
        for i in range(3):
            packed[..., 3 * m // 2 + i] = (w >> 8 * i & 255).to(torch.uint8)
    cbk, cbv = (dev(b[:1]).expand(Hkv, -1, -1, -1).contiguous() for b in books)
    cbv[:, :, C - 1] = float("inf")
    geom = antkv.Geometry(B, Hkv, Hkv, books.d, n_centroids=C)
    idx = torch.randint(0, N // k, (B, Hkv, k), device="cuda", generator=gen) + torch.arange(k, device="cuda") * (N // k)
    args = (geom, rnd(B, Hkv, 128), 128 ** -0.5, packed[0], packed[1], cbk, cbv, idx.int(), rnd(B, Hkv, k, 128), idx.int(), rnd(B, Hkv, k, 128))
    got = antkv.decode_attn(*args).double()
    want = antkv.decode_attn(*args, workspace=_least(antkv.DecodeWorkspace(geom, N, k, k, 0, "cuda"))).double()
    assert torch.isfinite(got).all()
    err = ((got - want).norm(dim=-1) / want.norm(dim=-1)).max().item()
    print(f"N={N}: {err:.2e}")
    assert err <= 4e-3


def _pack12_dev(codes):
    """pack12 on the GPU: [..., M] codes -> [..., 3M/2] bytes."""
    out = torch.empty((*codes.shape[:-1], codes.shape[-1] * 3 // 2), dtype=torch.uint8, device="cuda")
    for m in range(0, codes.shape[-1], 2):
        w = codes[..., m] | codes[..., m + 1] << 12
        for i in range(3):
            out[..., 3 * m // 2 + i] = (w >> 8 * i & 255).to(torch.uint8)
    return out


def _effective(codes, cb, idx, rows):
    """float64 [Hkv, N, 128] of one sequence: the centroids of the codes, the FP16 rows in the anchored places."""
    Hkv, N, M = codes.shape
    out = torch.empty((Hkv, N, 128), dtype=torch.float64, device="cuda")
    for m in range(M):
        d = 128 // M
        for g in range(Hkv):
            out[g, :, m * d:(m + 1) * d] = cb[g, m].double()[codes[g, :, m]]
    if idx is not None:
        for g in range(Hkv):
            out[g, idx[g].long()] = rows[g].double()
    return out


def _decode_exact(q, scale, codes_k, codes_v, cb_k, cb_v, idx_k, rows_k, idx_v, rows_v):
    """Decode attention of unpacked codes in float64: (output [B, Hq, 128], softmax weights [B, Hq, N])."""
    outs, ps = [], []
    for b in range(q.shape[0]):
        k = _effective(codes_k[b], cb_k, None if idx_k is None else idx_k[b], None if rows_k is None else rows_k[b])
        s = scale * (q[b].double().view(k.shape[0], -1, 128) @ k.transpose(1, 2).contiguous())
        del k
        p = torch.softmax(s, dim=-1)
        v = _effective(codes_v[b], cb_v, None if idx_v is None else idx_v[b], None if rows_v is None else rows_v[b])
        outs.append((p @ v).view(-1, 128))
        ps.append(p.view(-1, p.shape[-1]))
    return torch.stack(outs), torch.stack(ps)


def _by_code_shape(books):
    """(B, Hkv, N) at which the values are added up by code, one range per KV head."""
    return (16, 8, 14400) if books.d == 32 else (8, 8, 8257)


@pytest.mark.parametrize("by_code", [True, False])
def test_decode12_scores_of_v_anchors(books, by_code):
    """Where a table does not hold every head, a V-anchored token outside the K list is scored by fp32 products and not through the
    16-bit table, whichever way the values are added up.  The V centroids are zero and every V row has one channel, so that a
    channel of the output is one token's softmax weight, and a centroid that no token uses makes the table coarse: its rounding alone
    would move a weight by 8e-4 rms.  Bound: the output's rounding 2^-11, gathering also the fp16 weight's; 1e-4 for the rest."""
    if books.d == 32:
        pytest.skip("the table holds every head")
    B, Hkv, N = _by_code_shape(books)
    Hq, k_k, k_v, M, d = 4 * Hkv, 90, 128, books.M, books.d
    gen = torch.Generator(device="cuda").manual_seed(11)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    codes_k, codes_v = (torch.randint(0, C - 1, (B, Hkv, N, M), device="cuda", generator=gen) for _ in range(2))
    cb_k = rnd(Hkv, M, C, d) * 0.5
    cb_k[:, :, C - 1] = 45 * rnd(Hkv, M, d).sign()
    cb_v = torch.zeros((Hkv, M, C, d), dtype=torch.float16, device="cuda")
    order = torch.rand((B, Hkv, N), device="cuda", generator=gen).argsort(dim=-1)
    idx_v = order[..., :k_v].sort(dim=-1).values.int().contiguous()
    idx_k = order[..., k_v - 30:k_v - 30 + k_k].sort(dim=-1).values.int().contiguous()      # 30 tokens in both lists
    rows_k = rnd(B, Hkv, k_k, 128) * 0.5
    rows_v = (1024 * torch.eye(128, dtype=torch.float16, device="cuda")).expand(B, Hkv, k_v, 128).contiguous()
    q, scale = rnd(B, Hq, 128), 128 ** -0.5
    geom = antkv.Geometry(B, Hq, Hkv, d, n_centroids=C)
    ws = antkv.DecodeWorkspace(geom, N, k_k, k_v, 0, "cuda")
    got = antkv.decode_attn(geom, q, scale, _pack12_dev(codes_k), _pack12_dev(codes_v), cb_k, cb_v, idx_k, rows_k, idx_v, rows_v,
                            workspace=ws if by_code else _least(ws)).double()
    _, p = _decode_exact(q, scale, codes_k, codes_v, cb_k, cb_v, idx_k, rows_k, idx_v, rows_v)
    want = 1024 * p.gather(-1, idx_v.long().repeat_interleave(Hq // Hkv, dim=1))
    err = ((got - want) / want).abs()
    print(f"d{d} by code {by_code}: largest {err.max().item():.2e}, rms {err.pow(2).mean().sqrt().item():.2e}")
    assert err.max().item() <= (1 if by_code else 2) * 2.0 ** -11 + 1e-4


@pytest.mark.parametrize("gap", [24.5, 28.25, 30.5, 31.5])
@pytest.mark.parametrize("large", ["code", "anchor"])
def test_decode12_small_weights_beside_a_large_one(books, large, gap):
    """One token whose value is zero outweighs every other one by 2^gap: what is left of the output is the sum of the small weights,
    all equal and rounded alike.  Added up by code, a weight is a number of units of at most 17/16 2^-31 of the streamed sum, what
    is left of one being counted for the right part of a tile's 64 tokens: a tile's sum is off by less than a unit.  An FP16 row's
    token is not part of that sum.  Besides: 2^-11 for the output, half a unit of the smallest fp16 weights (2^-36 of the
    large one) in a wave that has the large token, 2e-4 for table, exponentials and fp32 sums."""
    B, Hkv, N = _by_code_shape(books)
    M, d = books.M, books.d
    codes_k = torch.zeros((B, Hkv, N, M), dtype=torch.int64, device="cuda")
    codes_v = torch.ones_like(codes_k)
    cb_k = torch.zeros((Hkv, M, C, d), dtype=torch.float16, device="cuda")
    cb_v = torch.zeros_like(cb_k)
    cb_k[:, 0, 1, 0] = gap
    cb_v[:, :, 1] = 30000
    at = 777
    codes_v[:, :, at] = 0
    idx_k = rows_k = None
    if large == "code":
        codes_k[:, :, at, 0] = 1
    else:
        idx_k = torch.full((B, Hkv, 1), at, dtype=torch.int32, device="cuda")
        rows_k = torch.zeros((B, Hkv, 1, 128), dtype=torch.float16, device="cuda")
        rows_k[..., 0] = gap
    q = torch.zeros((B, Hkv, 128), dtype=torch.float16, device="cuda")
    q[..., 0] = 1
    geom = antkv.Geometry(B, Hkv, Hkv, d, n_centroids=C)
    ck, cv = _pack12_dev(codes_k), _pack12_dev(codes_v)
    want = 30000 * (N - 1) / (2.0 ** gap + N - 1)
    for by_code in (True, False):
        ws = antkv.DecodeWorkspace(geom, N, 1 if idx_k is not None else 0, 0, 0, "cuda")
        got = antkv.decode_attn(geom, q, float(np.log(2)), ck, cv, cb_k, cb_v, idx_k, rows_k, None, None,
                                workspace=ws if by_code else _least(ws)).double()
        bound = 2.0 ** -11 + 2e-4
        if large == "code":
            bound += 2.0 ** (gap - 37) + (17 / 16 * 2.0 ** (gap - 31) / 64 if by_code else 0)
        err = ((got - want) / want).abs().max().item()
        print(f"d{d} {large} 2^{gap}, by code {by_code}: {err:.2e}, bound {bound:.2e}")
        assert err <= bound


@pytest.mark.parametrize("B,Hkv", [(8, 8), (3, 2), (12, 8)])
def test_decode12_either_side_of_the_switch(books, B, Hkv):
    """The first context that is added up by code and the last that is not, against float64; the workspace of the latter is refused when
    it is cut short, that of the former is not."""
    geom = antkv.Geometry(B, Hkv, Hkv, books.d, n_centroids=C)
    n, k = _switch(geom), 40
    gen = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    codes_k, codes_v = (torch.randint(0, C, (B, Hkv, n, books.M), device="cuda", generator=gen) for _ in range(2))
    cb_k, cb_v = rnd(Hkv, books.M, C, books.d), rnd(Hkv, books.M, C, books.d)
    q, rows_k, rows_v = rnd(B, Hkv, 128), rnd(B, Hkv, k, 128), rnd(B, Hkv, k, 128)
    for N in (n - 1, n):
        idx_k, idx_v = (torch.rand((B, Hkv, N), device="cuda", generator=gen).argsort(dim=-1)[..., :k].sort(dim=-1).values.int() for _ in range(2))
        args = (geom, q, 128 ** -0.5, _pack12_dev(codes_k[:, :, :N]), _pack12_dev(codes_v[:, :, :N]), cb_k, cb_v, idx_k, rows_k, idx_v, rows_v)
        want, _ = _decode_exact(q, 128 ** -0.5, codes_k[:, :, :N], codes_v[:, :, :N], cb_k, cb_v, idx_k, rows_k, idx_v, rows_v)
        got = antkv.decode_attn(*args).double()
        assert ((got - want).norm(dim=-1) / want.norm(dim=-1)).max().item() <= 2e-3
        least = _least(antkv.DecodeWorkspace(geom, N, k, k, 0, "cuda"))
        if N == n:
            antkv.decode_attn(*args, workspace=least)
        else:
            with pytest.raises(antkv.AntkvError):
                antkv.decode_attn(*args, workspace=least)


# Edges of a tile (32 tokens), of the waves (8 tiles), of the split (128 tokens a range, 32 ranges), groups of 1, 2 and 4, all
# or no tokens anchored, lists that are cut to the ranges; the longest ranges that are gathered row by row (8 heads: 32 x 3072 and 32 x 1792 tokens) and one more.
@pytest.mark.parametrize("B,Hq,Hkv,N,k_k,k_v", [(1, 4, 1, 1, 1, 0), (3, 2, 2, 31, 0, 31), (1, 8, 2, 33, 33, 33), (2, 4, 2, 127, 1, 1),
                                                (1, 8, 8, 129, 5, 7), (300, 1, 1, 257, 3, 9), (1, 4, 2, 4095, 700, 1300), (1, 16, 4, 4097, 41, 41),
                                                (5, 32, 8, 3001, 62, 62), (1, 32, 8, -1, 300, 310), (1, 32, 8, -2, 310, 300),
                                                (1, 8, 2, 9000, 2048, 2049), (2, 4, 2, 20001, 20001, 0), (1, 2, 2, 30000, 2049, 29000)])
def test_decode12_short_ranges(books, B, Hq, Hkv, N, k_k, k_v):
    """Row by row, against float64.  Bound: a weight's rounding to fp16 and the output's, 2^-11 each; 1e-4 for the rest (through
    the table, one token past the longest, the bound that its other tests have)."""
    longest = 32 * (3072 if books.d == 32 else 1792)
    by_table = N == -2
    N = longest - 1 - N if N < 0 else N
    gen = torch.Generator(device="cuda").manual_seed(N + B)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    codes_k, codes_v = (torch.randint(0, C, (B, Hkv, N, books.M), device="cuda", generator=gen) for _ in range(2))
    cb_k, cb_v = rnd(Hkv, books.M, C, books.d), rnd(Hkv, books.M, C, books.d)
    pick = lambda k: torch.rand((B, Hkv, N), device="cuda", generator=gen).argsort(dim=-1)[..., :k].sort(dim=-1).values.int().contiguous()
    q, rows_k, rows_v, idx_k, idx_v = rnd(B, Hq, 128), rnd(B, Hkv, k_k, 128), rnd(B, Hkv, k_v, 128), pick(k_k), pick(k_v)
    room = torch.nn.functional.pad
    got = antkv.decode_attn(antkv.Geometry(B, Hq, Hkv, books.d, n_centroids=C), q, 128 ** -0.5, room(_pack12_dev(codes_k), (0, 0, 0, 3), value=255),
                            room(_pack12_dev(codes_v), (0, 0, 0, 3), value=255), cb_k, cb_v, idx_k if k_k else None,
                            rows_k if k_k else None, idx_v if k_v else None, rows_v if k_v else None, N=N).double()
    want, _ = _decode_exact(q, 128 ** -0.5, codes_k, codes_v, cb_k, cb_v, idx_k, rows_k, idx_v, rows_v)
    err = ((got - want).norm(dim=-1) / want.norm(dim=-1)).max().item()
    print(f"d{books.d} N{N}: {err:.2e}")
    assert err <= (2e-3 if by_table else 2.0 ** -10 + 1e-4)


@pytest.mark.parametrize("gain", [1, 4, 16])
@pytest.mark.parametrize("G", [1, 2, 4])
def test_decode12_values_by_code_query_gain(books, gain, G):
    """Sharp softmaxes by code: references that rise late in a wave's walk, ranges far below the sequence's reference, tokens and FP16
    rows with most of the weight.  Bound: as in test_decode12_query_gain, 2e-3 inside the table's range and growing with it beyond.
    Several ranges of the second kernel per KV head, the last one ragged."""
    from gpu_util import attn_tol_for_range, table_range
    B, Hkv, N, k, M = 4, 2, 260077 if books.d == 32 else 100077, 200, books.M
    gen = torch.Generator(device="cuda").manual_seed(10 * gain + G)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    codes_k, codes_v = (torch.randint(0, C, (B, Hkv, N, M), device="cuda", generator=gen) for _ in range(2))
    cb_k, cb_v = dev(books[0][:Hkv]), dev(books[1][:Hkv])
    order = torch.rand((B, Hkv, N), device="cuda", generator=gen).argsort(dim=-1)
    idx_k, idx_v = order[..., :k].sort(dim=-1).values.int().contiguous(), order[..., k - 50:2 * k - 50].sort(dim=-1).values.int().contiguous()
    q, rows_k, rows_v, scale = rnd(B, G * Hkv, 128), rnd(B, Hkv, k, 128), rnd(B, Hkv, k, 128), gain * 128 ** -0.5
    geom = antkv.Geometry(B, G * Hkv, Hkv, books.d, n_centroids=C)
    args = (geom, q, scale, _pack12_dev(codes_k), _pack12_dev(codes_v), cb_k, cb_v, idx_k, rows_k, idx_v, rows_v)
    got = antkv.decode_attn(*args)
    gather = antkv.decode_attn(*args, workspace=_least(antkv.DecodeWorkspace(geom, N, k, k, 0, "cuda")))
    want, _ = _decode_exact(q, scale, codes_k, codes_v, cb_k, cb_v, idx_k, rows_k, idx_v, rows_v)
    tol = attn_tol_for_range(table_range(q.cpu().numpy(), books[0][:Hkv], scale, G), M, 32767)
    err, err_g = (((x.double() - want).norm(dim=-1) / want.norm(dim=-1)).cpu().numpy() for x in (got, gather))
    print(f"d{books.d} G={G} gain {gain}: {err.max():.2e}, gathering {err_g.max():.2e}, bound {tol.min():.1e} .. {tol.max():.1e}")
    assert (err <= tol).all() and (err_g <= tol).all()


def test_decode12_values_by_code_every_token_anchored(books):
    """Every token has an FP16 K row, and some or all an FP16 V row: all the stream's weights are zero."""
    B, Hkv, N = _by_code_shape(books)
    gen = torch.Generator(device="cuda").manual_seed(13)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    codes_k, codes_v = (torch.randint(0, C, (B, Hkv, N, books.M), device="cuda", generator=gen) for _ in range(2))
    cb_k, cb_v = rnd(Hkv, books.M, C, books.d), rnd(Hkv, books.M, C, books.d)
    q, rows_k = rnd(B, Hkv, 128), rnd(B, Hkv, N, 128)
    every = torch.arange(N, dtype=torch.int32, device="cuda")
    idx_k = every.expand(B, Hkv, N).contiguous()
    geom = antkv.Geometry(B, Hkv, Hkv, books.d, n_centroids=C)
    for idx in (every[::7], every):
        idx_v = idx.expand(B, Hkv, -1).contiguous()
        rows_v = rnd(B, Hkv, idx_v.shape[-1], 128)
        got = antkv.decode_attn(geom, q, 128 ** -0.5, _pack12_dev(codes_k), _pack12_dev(codes_v), cb_k, cb_v, idx_k, rows_k, idx_v, rows_v,
                                workspace=antkv.DecodeWorkspace(geom, N, N, idx_v.shape[-1], 0, "cuda")).double()
        want, _ = _decode_exact(q, 128 ** -0.5, codes_k, codes_v, cb_k, cb_v, idx_k, rows_k, idx_v, rows_v)
        assert ((got - want).norm(dim=-1) / want.norm(dim=-1)).max().item() <= 2e-3


def test_encode12_then_decode12(oracle, books):
    """Codes produced by the library's own encode feed its decode; the oracle decodes the oracle's codes."""
    from workloads import make_decode_query
    B, Hq, Hkv, N = 1, 8, 2, 2000
    _, k, v = make_qkv(98, B, Hq, Hkv, N, 1, 128)
    geom = antkv.Geometry(B, Hq, Hkv, books.d, n_centroids=C)
    cbk, cbv = dev(books[0]), dev(books[1])
    ck, cv = antkv.encode(geom, dev(k), cbk), antkv.encode(geom, dev(v), cbv)
    q = make_decode_query(98, B, Hq, 128)
    scale = 1.0 / np.sqrt(128)
    out = antkv.decode_attn(geom, dev(q), scale, ck, cv, cbk, cbv, None, None, None, None)
    none = np.zeros((B, Hkv, 0), np.int32)
    rows = np.zeros((B, Hkv, 0, 128), np.float16)
    want = oracle.decode_attn(q, unpack12(ck.cpu().numpy()), unpack12(cv.cpu().numpy()), books[0], books[1], none, rows,
                              none, rows, scale)
    err = np.linalg.norm(out.cpu().numpy().astype(np.float64) - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert err.max() <= 2e-3


def test_wide_geometry_rejections(books):
    import ctypes
    lib = antkv.load_library()
    bad = antkv.Geometry(1, 4, 2, 8, n_centroids=C).c()          # 4096 centroids need d_sub 32 or 16
    assert lib.antkv_decode_attn_workspace(ctypes.byref(bad), 100, 0, 0, 0) == 0
    ok = antkv.Geometry(1, 4, 2, books.d, n_centroids=C).c()
    assert lib.antkv_decode_attn_workspace(ctypes.byref(ok), 100, 0, 0, 0) > 0
    assert lib.antkv_decode_attn_workspace(ctypes.byref(ok), 100, 0, 0, 5) > lib.antkv_decode_attn_workspace(
        ctypes.byref(ok), 100, 0, 0, 0)
    assert lib.antkv_kmeans_step_workspace(ctypes.byref(ok)) >= 2 * 128 * 4096 * 4        # fp32 sums of two KV heads


@pytest.mark.parametrize("W", [8, 0])
def test_append12_then_decode12(oracle, books, W):
    """Decode loop on 12-bit codes: append with an FP16 window, then attention, step by step against the oracle."""
    from gpu_util import NEAR_TIE
    from workloads import make_decode_query
    B, Hq, Hkv, N0, k_a = 1, 4, 2, 200, 5
    T = 2 * W + 3 if W else 4
    scale = 1 / np.sqrt(128)
    _, k_all, v_all = make_qkv(99 + W, B, Hq, Hkv, N0 + T, 1, 128)
    cbk, cbv = books
    N_cap = N0 + T
    codes_k = np.zeros((B, Hkv, N_cap, books.M), np.int32)
    codes_v = np.zeros((B, Hkv, N_cap, books.M), np.int32)
    codes_k[:, :, :N0] = oracle.encode(k_all[:, :, :N0], cbk)
    codes_v[:, :, :N0] = oracle.encode(v_all[:, :, :N0], cbv)
    anchors = np.arange(3, 3 + 11 * k_a, 11)
    idx = np.broadcast_to(np.concatenate([anchors, np.arange(N0 - W, N0)]), (B, Hkv, k_a + W)).astype(np.int32).copy()
    idx_k, idx_v = idx.copy(), idx.copy()
    rows_k = np.take_along_axis(k_all, idx[..., None].astype(np.int64), axis=2).copy()
    rows_v = np.take_along_axis(v_all, idx[..., None].astype(np.int64), axis=2).copy()
    geom = antkv.Geometry(B, Hq, Hkv, books.d, n_centroids=C)
    g = dict(ck=dev(pack12(codes_k)), cv=dev(pack12(codes_v)), cbk=dev(cbk), cbv=dev(cbv),
             ik=dev(idx_k), rk=dev(rows_k), iv=dev(idx_v), rv=dev(rows_v))
    N = N0
    for t in range(T):
        kn, vn = k_all[:, :, N0 + t], v_all[:, :, N0 + t]
        N_new, mk, mv = oracle.append_token(kn, vn, N, W, cbk, cbv, codes_k, codes_v, idx_k, rows_k, idx_v, rows_v,
                                            want_margin=True)
        N_gpu = antkv.append_token(geom, dev(kn), dev(vn), N, W, g["cbk"], g["cbv"], g["ck"], g["cv"], g["ik"], g["rk"],
                                   g["iv"], g["rv"])
        torch.cuda.synchronize()
        assert N_gpu == N_new
        pos = N - W
        for name, got_c, want_c, margin in (("K", g["ck"], codes_k, mk), ("V", g["cv"], codes_v, mv)):
            got = unpack12(got_c[:, :, pos].cpu().numpy())
            bad = got != want_c[:, :, pos]
            assert not (bad & (margin >= NEAR_TIE)).any(), f"step {t}: {name} codes of position {pos} differ"
            got_c[:, :, pos] = dev(pack12(want_c[:, :, pos]))
        assert (g["ik"].cpu().numpy() == idx_k).all() and (g["rk"].cpu().numpy() == rows_k).all(), f"step {t}"
        assert (g["iv"].cpu().numpy() == idx_v).all() and (g["rv"].cpu().numpy() == rows_v).all(), f"step {t}"
        N = N_new
        q = make_decode_query(950 + t, B, Hq, 128)
        out = antkv.decode_attn(geom, dev(q), scale, g["ck"], g["cv"], g["cbk"], g["cbv"], g["ik"], g["rk"], g["iv"],
                                g["rv"], N=N)
        want = oracle.decode_attn(q, codes_k[:, :, :N], codes_v[:, :, :N], cbk, cbv, idx_k, rows_k, idx_v, rows_v, scale)
        err = np.linalg.norm(out.cpu().numpy().astype(np.float64) - want, axis=-1) / np.linalg.norm(want, axis=-1)
        assert err.max() <= 2e-3, f"step {t}: decode relative L2 {err.max():.3e}"
    print(f"W={W}: {T} appends + decodes on 12-bit codes ok")


@pytest.mark.parametrize("B,Hq,Hkv,N,k_k,k_v", [(1, 8, 2, 2500, 25, 25), (2, 4, 2, 900, 0, 7), (1, 2, 2, 1300, 13, 0),
                                                (1, 8, 2, 70000, 700, 700)])
def test_decode12_anchor_score_and_reselection(oracle, books, B, Hq, Hkv, N, k_k, k_v):
    """Decode-time Anchor Score over 12-bit codes (one walk per one or two heads, the shares add up) + re-selection."""
    from gpu_util import check_index_sets
    from workloads import make_decode_query, normal_fp16, random_anchor_sets
    rng = np.random.default_rng(N)
    scale = 1.0 / np.sqrt(128)
    cbk, cbv = books[0][:Hkv], books[1][:Hkv]
    ck = rng.integers(0, C, (B, Hkv, N, books.M)).astype(np.int32)
    cv = rng.integers(0, C, (B, Hkv, N, books.M)).astype(np.int32)
    ik, iv = random_anchor_sets(N, "k", B, Hkv, N, k_k), random_anchor_sets(N, "v", B, Hkv, N, k_v)
    rk, rv = normal_fp16(N, "rows_k", (B, Hkv, k_k, 128)), normal_fp16(N, "rows_v", (B, Hkv, k_v, 128))
    q = make_decode_query(N, B, Hq, 128)
    k_resel = max(1, N // 100)
    geom = antkv.Geometry(B, Hq, Hkv, books.d, n_centroids=C)
    out, ans_k, ans_v, rsk, rsv = antkv.decode_attn(
        geom, dev(q), scale, dev(pack12(ck)), dev(pack12(cv)), dev(cbk), dev(cbv), dev(ik) if k_k else None,
        dev(rk) if k_k else None, dev(iv) if k_v else None, dev(rv) if k_v else None, k_resel=k_resel)
    torch.cuda.synchronize()
    want, ex = oracle.decode_attn(q, ck, cv, cbk, cbv, ik, rk, iv, rv, scale, want_ans=True)
    err = np.linalg.norm(out.cpu().numpy().astype(np.float64) - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert err.max() <= 2e-3
    np.testing.assert_allclose(ans_v.cpu().numpy(), ex["ans_v"], rtol=3e-5, atol=1e-12)
    np.testing.assert_allclose(ans_k.cpu().numpy(), ex["ans_k"], rtol=3e-5, atol=1e-12)
    soft = 0
    for got, score in ((rsk, ex["ans_k"]), (rsv, ex["ans_v"])):
        w_idx, margin = oracle.topk(score, k_resel, want_margin=True)
        soft += check_index_sets(got.cpu().numpy(), w_idx, margin)
    print(f"N={N} G={Hq // Hkv}: scores within 3e-5, near-tie index disagreements {soft}")


def test_decode12_extreme_context_reselection(oracle, books):
    """The 840000-token shape (1 sequence, 32 query heads on 8 KV heads, 8400 anchors per head) on 12-bit codes: the
    decode step, the decode-time Anchor Score and the re-selection of 8400 tokens, all against the oracle."""
    from gpu_util import check_index_sets
    from workloads import CONFIGS, make_decode_query, normal_fp16, random_anchor_sets
    w = CONFIGS["cfg4"]
    B, Hq, Hkv, N, k = w.B, w.Hq, w.Hkv, w.N, w.k
    rng = np.random.default_rng(840000 + books.d)
    heads = np.arange(Hkv) % books[0].shape[0]                 # the fixture's two heads, repeated over the eight KV heads
    cbk, cbv = np.ascontiguousarray(books[0][heads]), np.ascontiguousarray(books[1][heads])
    ck = rng.integers(0, C, (B, Hkv, N, books.M)).astype(np.int32)
    cv = rng.integers(0, C, (B, Hkv, N, books.M)).astype(np.int32)
    ik, iv = random_anchor_sets(w.seed, "k", B, Hkv, N, k), random_anchor_sets(w.seed, "v", B, Hkv, N, k)
    rk, rv = normal_fp16(w.seed, "rows_k", (B, Hkv, k, 128)), normal_fp16(w.seed, "rows_v", (B, Hkv, k, 128))
    q = make_decode_query(w.seed, B, Hq, 128)
    geom = antkv.Geometry(B, Hq, Hkv, books.d, n_centroids=C)
    out, ans_k, ans_v, rsk, rsv = antkv.decode_attn(geom, dev(q), w.scale, dev(pack12(ck)), dev(pack12(cv)), dev(cbk), dev(cbv),
                                                    dev(ik), dev(rk), dev(iv), dev(rv), k_resel=k)
    torch.cuda.synchronize()
    want, ex = oracle.decode_attn(q, ck, cv, cbk, cbv, ik, rk, iv, rv, w.scale, want_ans=True)
    err = np.linalg.norm(out.cpu().numpy().astype(np.float64) - want, axis=-1) / np.linalg.norm(want, axis=-1)
    assert err.max() <= 2e-3, f"relative L2 {err.max():.3e}"
    np.testing.assert_allclose(ans_v.cpu().numpy(), ex["ans_v"], rtol=3e-5, atol=1e-12)
    np.testing.assert_allclose(ans_k.cpu().numpy(), ex["ans_k"], rtol=3e-5, atol=1e-12)
    soft = 0
    for got, score in ((rsk, ex["ans_k"]), (rsv, ex["ans_v"])):
        w_idx, margin = oracle.topk(score, k, want_margin=True)
        soft += check_index_sets(got.cpu().numpy(), w_idx, margin)
    print(f"d{books.d}m4096 N={N}: decode rel-L2 max {err.max():.2e}, near-tie index disagreements {soft}")


@pytest.mark.parametrize("B,n", [(2, 2500), (1, 70)])
def test_kmeans12_step(oracle, books, B, n):
    """One weighted k-means iteration on a 4096-centroid codebook: assignment by the code rule, update compared on the
    assignment the GPU used (most centroids get no token here and must keep their value)."""
    _, x, _ = make_qkv(101 + n, B, 2, 2, n, 1, 128, want_v=False)
    w = np.random.default_rng(n).gamma(0.5, 1.0, size=(B, 2, n)).astype(np.float32)
    w[:, :, ::7] = 0.0                                         # some tokens carry no weight at all
    cb = books[0]
    geom = antkv.Geometry(B, 2, 2, books.d, n_centroids=C)
    new, codes, wsum, obj = antkv.kmeans_step(geom, dev(x), dev(w), dev(cb))
    torch.cuda.synchronize()
    assert codes.shape == (B, 2, n, books.nbytes) and wsum.shape == (2, books.M, C)
    codes_h = unpack12(codes.cpu().numpy())
    want_codes, margin = oracle.encode(x, cb, want_margin=True)
    soft = check_codes(codes_h, want_codes, margin)
    want, want_w, want_obj = oracle.kmeans_update(x, w, codes_h, cb)
    np.testing.assert_allclose(wsum.cpu().numpy(), want_w, rtol=2e-5, atol=1e-30)
    np.testing.assert_allclose(obj.cpu().numpy(), want_obj, rtol=2e-5)
    got = new.cpu().numpy()
    empty = want_w == 0
    assert np.array_equal(got[empty], cb[empty]), "a centroid without assigned weight must keep its value"
    tol = np.abs(want) * 2.0 ** -10 + 2.0 ** -24 + 1e-5 * np.abs(want)
    assert (np.abs(got.astype(np.float64) - want) <= tol).all()
    print(f"d{books.d} n={n}: near-tie codes {soft}, centroids without weight {int(empty.sum())} of {empty.size}")


@pytest.mark.parametrize("B,n,distinct", [(3, 13001, 2), (1, 32769, 40), (5, 4099, 4099)])
def test_kmeans12_update_crowded(oracle, books, B, n, distinct):
    """More tokens of one range of centroids than a sorted chunk holds, runs over many windows, chunks that end inside a
    sequence.  Sums of up to 32 products per window, 256 windows and 5 chunks in fp32: within 300 * 2^-24 of the sum of
    magnitudes.  The weights are such a sum too, so a mean is within twice that, and its division rounds once more."""
    _, rows, _ = make_qkv(107, B, 2, 2, distinct, 1, 128, want_v=False)
    x = rows[:, :, np.random.default_rng(n).integers(0, distinct, n)]
    w = np.random.default_rng(n + 1).gamma(0.5, 1.0, size=(B, 2, n)).astype(np.float32)
    cb = books[0]
    new, codes, wsum, obj = antkv.kmeans_step(antkv.Geometry(B, 2, 2, books.d, n_centroids=C), dev(x), dev(w), dev(cb))
    codes_h = unpack12(codes.cpu().numpy())
    want, want_w, want_obj = oracle.kmeans_update(x, w, codes_h, cb)
    mag, _, _ = oracle.kmeans_update(np.abs(x), w, codes_h, np.abs(cb))
    np.testing.assert_allclose(wsum.cpu().numpy(), want_w, rtol=2e-5, atol=1e-30)
    np.testing.assert_allclose(obj.cpu().numpy(), want_obj, rtol=2e-5)
    got = new.cpu().numpy()
    assert np.array_equal(got[want_w == 0], cb[want_w == 0])
    assert (np.abs(got.astype(np.float64) - want) <= np.abs(want) * 2.0 ** -10 + 2.0 ** -24 + 601 * 2.0 ** -24 * mag).all()


def test_kmeans12_iterations_descend(oracle, books):
    _, x, _ = make_qkv(103, 2, 2, 2, 6000, 1, 128, want_v=False)
    w = np.random.default_rng(3).gamma(0.5, 1.0, size=(2, 2, 6000)).astype(np.float32)
    geom = antkv.Geometry(2, 2, 2, books.d, n_centroids=C)
    xd, wd, cur = dev(x), dev(w), dev(books[1])                # start from the V codebook: a poor fit for these K rows
    hist = []
    for _ in range(4):
        cur, _, _, obj = antkv.kmeans_step(geom, xd, wd, cur)
        hist.append(obj.cpu().numpy().sum())
    assert all(b <= a * (1 + 1e-4) for a, b in zip(hist, hist[1:])), hist
    assert hist[-1] < 0.9 * hist[0], hist


@pytest.mark.parametrize("B,Hq,Hkv,N", [(1, 4, 1, 1), (2, 2, 2, 45), (1, 8, 2, 3007), (1, 8, 8, 20001)])
def test_decode12_short_ranges_unused_codes_of_anchors(books, B, Hq, Hkv, N):
    """The newest tokens are in the V list and their codes, which nothing has written, name a centroid with infinities that no other
    token uses: they are ignored, also behind the last token of a tile that is not full.  Bound as in test_decode12_short_ranges."""
    gen = torch.Generator(device="cuda").manual_seed(N)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    W = min(N, 32)
    codes_k, codes_v = (torch.randint(0, C - 1, (B, Hkv, N, books.M), device="cuda", generator=gen) for _ in range(2))
    codes_k[:, :, N - W:] = codes_v[:, :, N - W:] = C - 1
    cb_k, cb_v = rnd(Hkv, books.M, C, books.d), rnd(Hkv, books.M, C, books.d)
    cb_v[:, :, C - 1] = float("inf")
    idx = torch.arange(N - W, N, dtype=torch.int32, device="cuda").expand(B, Hkv, W).contiguous()
    q, rows_k, rows_v = rnd(B, Hq, 128), rnd(B, Hkv, W, 128), rnd(B, Hkv, W, 128)
    got = antkv.decode_attn(antkv.Geometry(B, Hq, Hkv, books.d, n_centroids=C), q, 128 ** -0.5, _pack12_dev(codes_k), _pack12_dev(codes_v),
                            cb_k, cb_v, idx, rows_k, idx, rows_v).double()
    assert torch.isfinite(got).all()
    want, _ = _decode_exact(q, 128 ** -0.5, codes_k, codes_v, cb_k, cb_v, idx, rows_k, idx, rows_v)
    assert ((got - want).norm(dim=-1) / want.norm(dim=-1)).max().item() <= 2.0 ** -10 + 1e-4


@pytest.mark.parametrize("N", [32, 1000])
@pytest.mark.parametrize("gap", [24.5, 26.1, 28.25, 30.5])
def test_decode12_short_ranges_small_weights(books, N, gap):
    """One token whose value is zero outweighs every other one by 2^gap (test_decode12_small_weights_beside_a_large_one): 2^-11 for the
    output, half a unit of the smallest fp16 weights (2^-36 of the large one), 2e-4 for exponentials and fp32 sums."""
    B, Hkv, M, at = 1, 2, books.M, 7
    codes_k = torch.zeros((B, Hkv, N, M), dtype=torch.int64, device="cuda")
    codes_v = torch.ones_like(codes_k)
    cb_k = torch.zeros((Hkv, M, C, books.d), dtype=torch.float16, device="cuda")
    cb_v = torch.zeros_like(cb_k)
    cb_k[:, 0, 1, 0] = gap
    cb_v[:, :, 1] = 30000
    codes_k[:, :, at, 0], codes_v[:, :, at] = 1, 0
    q = torch.zeros((B, Hkv, 128), dtype=torch.float16, device="cuda")
    q[..., 0] = 1
    real = float(cb_k[0, 0, 1, 0])
    got = antkv.decode_attn(antkv.Geometry(B, Hkv, Hkv, books.d, n_centroids=C), q, float(np.log(2)), _pack12_dev(codes_k),
                            _pack12_dev(codes_v), cb_k, cb_v, None, None, None, None).double()
    want = 30000 * (N - 1) / (2.0 ** real + N - 1)
    err = ((got - want) / want).abs().max().item()
    print(f"d{books.d} N={N} 2^{gap}: {err:.2e}")
    assert err <= 2.0 ** -11 + 2e-4 + 2.0 ** (gap - 37)


def test_decode12_short_ranges_replayed(books):
    """A captured step, replayed: the arrival words still hold the launch's own tag from the replay before."""
    B, Hq, Hkv, N, k = 1, 8, 2, 1500, 20
    gen = torch.Generator(device="cuda").manual_seed(21)
    rnd = lambda *shape: torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen)
    codes = [_pack12_dev(torch.randint(0, C, (B, Hkv, N, books.M), device="cuda", generator=gen)) for _ in range(2)]
    cb = [rnd(Hkv, books.M, C, books.d) for _ in range(2)]
    idx = [torch.rand((B, Hkv, N), device="cuda", generator=gen).argsort(dim=-1)[..., :k].sort(dim=-1).values.int().contiguous() for _ in range(2)]
    q, rows = rnd(B, Hq, 128), [rnd(B, Hkv, k, 128) for _ in range(2)]
    geom, out = antkv.Geometry(B, Hq, Hkv, books.d, n_centroids=C), torch.empty((B, Hq, 128), dtype=torch.float16, device="cuda")
    ws = antkv.DecodeWorkspace(geom, N, k, k, 0, "cuda")
    step = lambda o: antkv.decode_attn(geom, q, 128 ** -0.5, *codes, *cb, idx[0], rows[0], idx[1], rows[1], out=o, workspace=ws)
    step(out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(out)
    for _ in range(6):
        q.copy_(rnd(B, Hq, 128))
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, step(torch.empty_like(out)))
