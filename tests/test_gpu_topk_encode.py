"""GPU parity: top-k selection and VQ encode against the CPU oracle (bit-exact bar)."""
import numpy as np
import pytest
import torch

import paper_2506_19505_amd as antkv
from gpu_util import check_codes, check_index_sets, dev
from workloads import CONFIGS, make_codebooks, make_qkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,N,k", [(3, 1, 1), (2, 100, 7), (4, 8192, 82), (3, 8193, 100), (2, 50000, 500),
                                      (2, 300, 300), (1, 840000, 8400), (16, 131072, 1311)])
def test_topk_matches_oracle(oracle, rows, N, k):
    rng = np.random.default_rng(N + k)
    s = rng.lognormal(0.0, 2.0, size=(rows, N)).astype(np.float32)
    if rows > 1:
        s[1] = np.round(s[1] * 4) / 4                      # plenty of exact ties at the threshold
    got = antkv.topk(dev(s), k).cpu().numpy()
    want = oracle.topk(s, k)                               # fp32 values are exact in fp64: no tolerance at all
    assert np.array_equal(got, want)


def test_topk_degenerate_rows(oracle):
    s = np.zeros((3, 5000), np.float32)
    s[1] = -1.5
    s[2, ::7] = np.float32(2.0)
    got = antkv.topk(dev(s), 40).cpu().numpy()
    assert np.array_equal(got[0], np.arange(40)) and np.array_equal(got[1], np.arange(40))
    assert np.array_equal(got[2], np.arange(0, 280, 7))
    # negative and mixed-sign scores order correctly
    t = np.random.default_rng(0).standard_normal((2, 3000)).astype(np.float32)
    assert np.array_equal(antkv.topk(dev(t), 33).cpu().numpy(), oracle.topk(t, 33))
    assert antkv.topk(dev(t), 0).shape == (2, 0)
    assert np.array_equal(antkv.topk(dev(t), 3000).cpu().numpy(), np.tile(np.arange(3000), (2, 1)))


def test_topk_scores_crowded_into_one_bin(oracle):
    """All scores of a row share their top 11 key bits, so the candidate list of the k-th key's bin overflows its
    buffer (N/8 + 4096 entries) and the selection falls back to walking the row; with and without ties."""
    rng = np.random.default_rng(3)
    N = 100000
    s = (1.0 + 0.18 * rng.random((3, N))).astype(np.float32)
    s[1] = np.round(s[1] * 64) / 64                        # a dozen distinct values: long runs of ties
    s[2] = -s[2]
    for k in (1, 1000, 99999):
        assert np.array_equal(antkv.topk(dev(s), k).cpu().numpy(), oracle.topk(s, k))


@pytest.mark.parametrize("N", [2047, 2048, 2049, 8192, 8195, 32767, 32768, 32769, 40963])
def test_topk_row_sizes(oracle, N):
    """Both sides of the sizes at which another kernel takes a row, rows that are not 16-byte aligned, and rows whose scores
    crowd into one bin of the first histogram with long runs of ties, of either sign."""
    rng = np.random.default_rng(N)
    s = np.exp(3.0 * rng.standard_normal((4, N))).astype(np.float32)
    s[1] = 1.0 + 0.2 * rng.random(N)
    s[2] = np.round(s[1] * 64) / 64
    s[3] = -s[2]
    for k in (1, N // 100, N - 1, N):
        assert np.array_equal(antkv.topk(dev(s), k).cpu().numpy(), oracle.topk(s, k))


def test_topk_negative_nans_in_a_short_last_slice():
    """NaNs with the sign bit and a full payload have the lowest keys of all, the bin that unused registers of the last
    slice fall into as well: one score in that slice, and a candidate list that holds the NaNs but not 8191 entries more."""
    N, n_nan = 32768 + 8192 + 1, 2000
    rng = np.random.default_rng(5)
    s = rng.random((2, N)).astype(np.float32)
    nan = np.sort(rng.permutation(N - 1)[:n_nan])
    s.view(np.uint32)[:, nan] = 0xffffe000 + (np.arange(n_nan) % 7).astype(np.uint32)
    bits = s.view(np.uint32)
    key = np.where(bits >> 31 == 1, ~bits, bits | 0x80000000)
    for k in (N - n_nan + 1, N - 1000, N):
        want = np.sort(np.argsort(0xffffffff - key.astype(np.int64), axis=1, kind="stable")[:, :k], axis=1)
        assert np.array_equal(antkv.topk(dev(s), k).cpu().numpy(), want)


@pytest.mark.parametrize("N", [1000, 2048, 8191, 32767, 32768, 40960, 40961, 49156, 73728])
def test_topk_lowest_key_at_the_threshold(N):
    """NaNs 0xffffffff have the lowest key of all, 0, which the registers past a row's end hold as well: the threshold is that
    key, in one launch per row and in many, with whole and partial last slices, rows aligned to 16 bytes and not."""
    rng = np.random.default_rng(N)
    n_nan = N // 5
    s = rng.random((3, N)).astype(np.float32)
    bits = s.view(np.uint32)
    for r, at in enumerate((rng.permutation(N)[:n_nan], np.arange(n_nan), np.arange(N - n_nan, N))):
        bits[r, at] = 0xffffffff
    key = np.where(bits == 0xffffffff, 0, bits | 0x80000000).astype(np.int64)
    for k in (N - n_nan, N - n_nan + 1, N - n_nan // 2, N):
        want = np.sort(np.argsort(-key, axis=1, kind="stable")[:, :k], axis=1)
        assert np.array_equal(antkv.topk(dev(s), k).cpu().numpy(), want)


@pytest.mark.parametrize("N", [32772, 40960, 65536, 73729])
def test_topk_ties_across_slices(oracle, N):
    """Ties at the threshold that run over threads, waves and slices, rows that are 16-byte aligned and rows that are not."""
    rng = np.random.default_rng(N)
    s = np.exp(rng.standard_normal((4, N))).astype(np.float32)
    s[0, ::2] = 1.0                                            # every thread has some
    s[1, 8000:24800] = 1.0                                     # a run over two slice ends
    s[2] = 1.0
    s[3, rng.permutation(N)[:50]] = 1.0
    for k in (1, N // 100, N // 3, N // 2, N - 1):
        assert np.array_equal(antkv.topk(dev(s), k).cpu().numpy(), oracle.topk(s, k))


@pytest.mark.parametrize("N", [33000, 65543])
@pytest.mark.parametrize("k", [1, 327, 4125, 20000, -1, 0])
def test_topk_listed_crowded_and_walked(oracle, N, k):
    """Long rows of every kind in one call: few keys in the threshold's bin, a crowded bin, ties in 22 bits for more keys than the
    list holds (zeros, as exponentials that underflow leave them), all scores equal; k from one to all of them."""
    k = k if k > 0 else N + k                                  # N - 1 and N
    rng = np.random.default_rng(N + k)
    rows = np.empty((6, N), np.float32)
    rows[0] = np.exp(2 * rng.standard_normal(N)) / N
    rows[1] = 5 + 0.2 * rng.standard_normal(N)
    rows[2] = 0
    rows[2, rng.choice(N, N // 300, replace=False)] = rng.random(N // 300)
    rows[3] = -1.5
    rows[4] = np.round(rng.standard_normal(N) * 50) / 50
    rows[5] = 1 + rng.integers(0, 3, N) * np.float32(2.0 ** -23)
    got = antkv.topk(dev(rows), k).cpu().numpy()
    assert np.array_equal(got, oracle.topk(rows, k))


@pytest.mark.parametrize("rows,N", [(2, 33000), (7, 40963), (16, 73728)])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_topk_either_side_of_the_list_rule(oracle, rows, N, more):
    """k at 3000 + rows N / 1280, up to which a row's list holds every key from the threshold's bin up, beyond that the bin's alone:
    heavy tails, a crowded bin, a bin that fits the list only by itself, ties in 22 bits, at aligned and other row lengths."""
    k = 3000 + rows * N // 1280 + more
    rng = np.random.default_rng(N + more)
    s = np.exp(2 * rng.standard_normal((rows, N))).astype(np.float32)
    s[0, rng.permutation(N)[:N // 9]] += 1e6                   # k and the bin together are more than the list
    s[1] = 5 + 0.2 * rng.standard_normal(N)
    if rows > 2:
        s[2] = np.round(s[2], 1)
        s[3] = 0
        s[4, :N // 8] = 3.0
        s[5] = -s[5]
    assert np.array_equal(antkv.topk(dev(s), k).cpu().numpy(), oracle.topk(s, k))


@pytest.mark.parametrize("k", [9, 1000, 300000])
def test_topk_more_than_2048_slices(k):
    """Rows of more than 2048 x 8192 scores, whose slices are counted in windows of 2048: selected scores and ties at the threshold on
    both sides of slice 2048 and in the short last slice, in a row whose list holds them and in one that is walked."""
    edge, N = 2048 * 8192, 2049 * 8192 + 5
    gen = torch.Generator(device="cuda").manual_seed(k)
    s = torch.rand((3, N), dtype=torch.float32, device="cuda", generator=gen)
    s[0] = torch.exp(6 * s[0])
    s[1] = 0.5
    s[2] = torch.where(s[2] < 0.4, s[2], torch.full_like(s[2], 0.5))
    for at in (0, 5, edge - 2, edge - 1, edge, edge + 1, edge + 8191, edge + 8192, N - 1):
        s[:, at] = 1000.0 + (at % 3)
    got = antkv.topk(s, k)
    want = torch.sort(s, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
    assert torch.equal(got.long(), want)


@pytest.mark.parametrize("N", [33000, 65543])
@pytest.mark.parametrize("k", [20, 4125, 20000, 32999])
def test_topk_workspace_of_a_smaller_k(oracle, N, k):
    """A workspace sized for k = 1 serves any k."""
    s = np.exp(np.random.default_rng(N + k).standard_normal((3, N))).astype(np.float32)
    s[1] = np.round(s[1], 2)
    s[2] = 0.25
    lib = antkv.load_library()
    ws = torch.full((lib.antkv_topk_workspace(3, N, 1) + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    idx = torch.full((3, k), -1, dtype=torch.int32, device="cuda")
    x = dev(s)
    assert lib.antkv_topk(x.data_ptr(), 3, N, k, idx.data_ptr(), ws.data_ptr(), ws.numel() - 4096, None) == 0
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), oracle.topk(s, k))
    assert bool((ws[-4096:] == 0x5a).all())


@pytest.mark.parametrize("d", [4, 8, 16])
@pytest.mark.parametrize("B,Hq,Hkv,n", [(2, 4, 2, 333), (1, 8, 8, 70)])
def test_encode_matches_oracle(oracle, d, B, Hq, Hkv, n):
    _, k, v = make_qkv(11 + d, B, Hq, Hkv, n, 1, 128)
    geom = antkv.Geometry(B, Hq, Hkv, d)
    soft = 0
    for which, x in (("k", k), ("v", v)):
        cb = make_codebooks(11 + d, x, d, 256, which)
        want, margin = oracle.encode(x, cb, want_margin=True)
        got = antkv.encode(geom, dev(x), dev(cb)).cpu().numpy()
        soft += check_codes(got, want, margin, f"codes_{which} d={d}")
    print(f"near-tie disagreements: {soft}")


@pytest.mark.parametrize("d", [4, 8, 16])
def test_encode_large_magnitudes(oracle, d):
    """Keys and centroids some 40 times the synthetic recipe's (outlier channels reach several hundred): half the squared
    norm of a centroid's sub-vector exceeds the fp16 range, which the scaled norm terms must survive; and the append
    path (fp32 norms) must agree with antkv_encode on the same rows."""
    B, Hq, Hkv, n = 1, 4, 2, 300
    _, k, _ = make_qkv(17 + d, B, Hq, Hkv, n, 1, 128)
    unit = (make_codebooks(17 + d, k, d, 256, "k").astype(np.float64) ** 2).sum(-1).max()
    k = (k.astype(np.float32) * np.sqrt(1.5e6 / unit)).astype(np.float16)      # largest sub-vector norm^2 about 1.5e6
    cb = make_codebooks(17 + d, k, d, 256, "k")
    norms = (cb.astype(np.float64) ** 2).sum(-1)
    assert norms.max() / 2 > 65504 and norms.max() < 2.09e6, f"largest sub-vector norm^2 {norms.max():.3g}"
    want, margin = oracle.encode(k, cb, want_margin=True)
    got = antkv.encode(antkv.Geometry(B, Hq, Hkv, d), dev(k), dev(cb)).cpu().numpy()
    soft = check_codes(got, want, margin, f"large-magnitude codes d={d}")
    print(f"d={d}: largest ||c||^2 {norms.max():.3g}, near-tie disagreements {soft}")


@pytest.mark.parametrize("d", [4, 8, 16])
@pytest.mark.parametrize("over", ["first tile", "leading quads", "scattered", "all but the last", "infinite and NaN"])
def test_encode_never_chooses_oversize_centroids(d, over):
    """Centroids beyond ||c||^2 = 2.09e6 (and ones that are not finite) are never chosen, not even by a token that equals one: the
    codes are the nearest among the others, wherever in the tiles and quads of the arg-max the oversize ones sit."""
    B, Hkv, n, M, C = 1, 2, 200, 128 // d, 256
    rng = np.random.default_rng(d)
    bad = {"first tile": np.arange(32), "leading quads": np.r_[0:4, 40:44, 68:76], "scattered": rng.permutation(C)[:60],
           "all but the last": np.arange(C - 1), "infinite and NaN": np.r_[0, 5, 33, 255]}[over]
    cb = rng.standard_normal((Hkv, M, C, d)).astype(np.float16)
    x = rng.standard_normal((B, Hkv, n, 128)).astype(np.float16)
    size = np.sqrt(rng.uniform(2.1e6, 4e6, bad.size) / d)[:, None]           # ||c||^2 = 2.1e6 .. 4e6
    cb[:, :, bad] = (size * rng.choice([-1.0, 1.0], (bad.size, d))).astype(np.float16)
    x[..., :50, :] = cb[:, :, bad[np.arange(50) % bad.size]].transpose(0, 2, 1, 3).reshape(Hkv, 50, 128)
    if over == "infinite and NaN":
        cb[:, :, bad[0]], cb[:, :, bad[1]], cb[:, :, bad[2]], cb[:, :, bad[3], 0] = np.inf, np.nan, -np.inf, np.nan
    good = np.setdiff1d(np.arange(C), bad)
    got = antkv.encode(antkv.Geometry(B, Hkv, Hkv, d), dev(x), dev(cb)).cpu().numpy()
    assert np.isin(got, good).all()
    c = cb[:, :, good].astype(np.float64)
    xs = x.astype(np.float64).reshape(B, Hkv, n, M, d)
    score = np.einsum("bgnmd,gmcd->bgnmc", xs, c) - 0.5 * (c ** 2).sum(-1)[None, :, None]
    mine = np.take_along_axis(score, np.searchsorted(good, got.astype(np.int64))[..., None], -1)[..., 0]
    # d products of |x_i c_i| <= |x| |c| and the norm, summed in fp32
    slack = (d + 4) * 2.0 ** -24 * (np.linalg.norm(xs, axis=-1) * np.sqrt((c ** 2).sum(-1).max()) + 0.5 * (c ** 2).sum(-1).max())
    assert (mine >= score.max(-1) - 2 * slack).all()
    assert (got == good[score.argmax(-1)])[..., 50:, :].mean() > 0.999


def test_encode_duplicate_centroids_and_offsets(oracle):
    # fewer sample tokens than centroids -> duplicated centroids: the lower index must win exactly
    B, Hq, Hkv, n, d = 1, 2, 1, 100, 8
    _, k, _ = make_qkv(5, B, Hq, Hkv, n, 1, 128)
    cb = make_codebooks(5, k, d, 256, "k")
    assert len({c.tobytes() for c in cb[0, 0]}) < 256
    want, margin = oracle.encode(k, cb, want_margin=True)
    geom = antkv.Geometry(B, Hq, Hkv, d)
    # write into the middle of a larger code tensor, from a strided (non-contiguous) source
    wide = torch.zeros((B, Hkv, n, 256), dtype=torch.float16, device="cuda")
    wide[..., :128] = dev(k)
    codes = torch.full((B, Hkv, n + 50, 16), 255, dtype=torch.uint8, device="cuda")
    antkv.encode(geom, wide[..., :128], dev(cb), codes=codes, token_offset=20)
    got = codes.cpu().numpy()
    check_codes(got[:, :, 20:20 + n], want, margin)
    assert (got[:, :, :20] == 255).all() and (got[:, :, 20 + n:] == 255).all()


@pytest.mark.parametrize("d", [4, 8, 16])
@pytest.mark.parametrize("B,n", [(1, 1), (1, 33), (3, 31), (1, 4097), (2, 9001)])
def test_encode_work_splits_and_ties(oracle, d, B, n):
    """From one block of 32 tokens to several blocks per wave; centroids repeated in the same quad of a tile, in the other
    half-wave's rows, in other quads and in other tiles: the lower index has to win exactly."""
    M = 128 // d
    rng = np.random.default_rng(100 * d + n)
    cb = rng.standard_normal((2, M, 256, d)).astype(np.float16)
    for lo, hi in ((0, 1), (2, 6), (9, 17), (20, 28), (40, 44), (50, 250), (70, 102), (130, 255)):
        cb[:, :, hi] = cb[:, :, lo]
    x = rng.standard_normal((B, 2, n, 128)).astype(np.float16)
    dup = [0, 2, 9, 20, 40, 50, 70, 130]
    for t in range(min(n, 32)):                                  # tokens that sit on a repeated centroid
        x[:, :, t] = cb[:, :, dup[t % 8]].reshape(1, 2, 128)
    want, margin = oracle.encode(x, cb, want_margin=True)
    got = antkv.encode(antkv.Geometry(B, 2, 2, d), dev(x), dev(cb)).cpu().numpy()
    check_codes(got, want, margin)
    assert not np.isin(got, [1, 6, 17, 28, 44, 250, 102, 255]).any()


@pytest.mark.parametrize("d,n", [(4, 24448), (4, 24513), (8, 48960), (8, 49025)])
def test_encode_workgroups_per_cu(oracle, d, n):
    """Two KV heads at the token counts (382 and 384, 765 and 767 units of 64) around which the launch goes from two to three
    workgroups per CU: every unit is encoded once, in its place."""
    rng = np.random.default_rng(n)
    cb = rng.standard_normal((2, 128 // d, 256, d)).astype(np.float16)
    x = rng.standard_normal((1, 2, n, 128)).astype(np.float16)
    codes = torch.full((1, 2, n + 9, 128 // d), 0xEE, dtype=torch.uint8, device="cuda")
    codes = antkv.encode(antkv.Geometry(1, 2, 2, d), dev(x), dev(cb), codes, 5).cpu().numpy()
    assert (codes[:, :, :5] == 0xEE).all() and (codes[:, :, n + 5:] == 0xEE).all()
    want, margin = oracle.encode(x, cb, want_margin=True)
    check_codes(codes[:, :, 5:n + 5], want, margin)


def test_encode_full_prefill_shape(oracle):
    """32768 new tokens x 8 KV heads, 1-bit VQ: the encode workload at its real size."""
    w = CONFIGS["cfg3"]
    _, k, v = make_qkv(w.seed, w.B, w.Hq, w.Hkv, w.N, 1, w.D)
    geom = antkv.Geometry(w.B, w.Hq, w.Hkv, w.d_sub)
    for which, x in (("k", k), ("v", v)):
        cb = make_codebooks(w.seed, x, w.d_sub, 256, which, max_sample=4096)
        got = antkv.encode(geom, dev(x), dev(cb)).cpu().numpy()
        want, margin = oracle.encode(x, cb, want_margin=True)
        soft = check_codes(got, want, margin, f"cfg3 codes_{which}")
        print(f"cfg3 {which}: {soft} near-tie disagreements of {got.size}")
