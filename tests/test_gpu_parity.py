"""Parity of the HIP path (through the C ABI) with the fp64 CPU oracle.

Tolerances for N(0,1) inputs: O max-abs 2e-2, mean-abs 2e-3; LSE max-abs 1e-2.
"""
import math

import numpy as np
import pytest

from paper_2510_14719_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "the gpu tests need a GPU"
    from tests import gpu_util
    from paper_2510_14719_amd import binding
    binding.load_library()   # fails loudly if the extension was not built
    return gpu_util


def _full(G, oracle, B, H, N, d, dtype, causal, seed, scale=None, peaky=False, what=""):
    q, k, v = I.make_qkv(B, H, N, d, dtype, seed, peaky=peaky)
    scale = 1.0 / math.sqrt(d) if scale is None else scale
    print("case %s B%d H%d N%d d%d dtype%d causal%d seed%d" % (what, B, H, N, d, dtype, causal, seed), flush=True)
    o_ref, l_ref = oracle.attn_ref(q, k, v, dtype, scale, causal)
    o, l = G.run_gpu(q, k, v, dtype, scale, causal)
    G.check(o, l, o_ref, l_ref, what or "full")


# ------------------------------------------------------------ element-by-element, oracle-sized
@pytest.mark.parametrize("dtype", [I.FP16, I.BF16])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [1, 31, 64, 129, 256, 577, 1000])
def test_small_shapes_full_compare(G, oracle, N, d, causal, dtype):
    _full(G, oracle, 2, 3, N, d, dtype, causal, seed=50 + N)


@pytest.mark.parametrize("causal,dtype", [(False, I.FP16), (True, I.BF16)])
def test_more_tiles_than_resident_workgroups(G, oracle, causal, dtype):
    # 650 query tiles at d = 128: a persistent launch walks up to three rounds of its tile schedule,
    # the last one partial, each workgroup switching head and query tile between rounds
    _full(G, oracle, 5, 26, 1100, 128, dtype, causal, seed=77, what="multi-round")


def test_config_c1(G, oracle):
    w = I.WORKLOADS["c1"]
    _full(G, oracle, w.B, w.H, w.N, w.d, w.dtype, w.causal, w.seed, what="c1")


@pytest.mark.parametrize("causal", [False, True])
def test_many_tiles_ragged_tail(G, oracle, causal):
    # several query tiles, many K/V tiles, and a tail that is not a multiple of any tile size
    _full(G, oracle, 1, 2, 2309, 128, I.FP16, causal, seed=77, what="ragged")
    _full(G, oracle, 1, 2, 1531, 64, I.BF16, causal, seed=78, what="ragged")


# ------------------------------------------------------------ the benchmark configurations, sampled rows
def _sampled(G, oracle, name, n_rows):
    w = I.WORKLOADS[name]
    print("config %s: B%d H%d N%d d%d dtype%d causal%d peaky%d" % (name, w.B, w.H, w.N, w.d, w.dtype, w.causal, w.peaky), flush=True)
    q, k, v = I.make_workload(w)
    always = [(0, 0, 0), (w.B - 1, w.H - 1, w.N - 1), (0, 0, w.N // 2), (w.B - 1, 0, 1)]
    rows = I.sample_rows(w.B, w.H, w.N, n_rows, seed=w.seed + 7, always=always)
    o_ref, l_ref = oracle.attn_ref_rows(q, k, v, w.dtype, rows, w.scale, w.causal)
    o, l = G.run_gpu(q, k, v, w.dtype, w.scale, w.causal)
    assert np.isfinite(o).all() and np.isfinite(l).all()
    idx = np.asarray(rows)
    G.check(o[idx[:, 0], idx[:, 1], idx[:, 2]], l[idx[:, 0], idx[:, 1], idx[:, 2]], o_ref, l_ref, name)
    return q, k, v, o, l


@pytest.mark.parametrize("name", ["c2", "c2_causal", "c3", "c4", "c5"])
def test_benchmark_configs_sampled_rows(G, oracle, name):
    _sampled(G, oracle, name, 192)


# ------------------------------------------------------------ the full-size configurations, whole heads
@pytest.mark.parametrize("name", ["c2", "c2_causal", "c3", "c4", "c5"])
def test_whole_heads_of_the_large_configs(G, oracle, name):
    """Full size, the launch configuration ``bench.py`` times: every element of O and LSE was written (the buffers
    start out as NaN), and the first and the last (batch, head) agree with the oracle element by element."""
    w = I.WORKLOADS[name]
    print("config %s whole heads: B%d H%d N%d d%d dtype%d causal%d peaky%d" % (name, w.B, w.H, w.N, w.d, w.dtype, w.causal, w.peaky), flush=True)
    q, k, v = I.make_workload(w)
    o, l = G.run_gpu(q, k, v, w.dtype, w.scale, w.causal)
    assert np.isfinite(o).all() and np.isfinite(l).all(), "an element of O or LSE was never written"
    for (b, h) in [(0, 0), (w.B - 1, w.H - 1)]:
        sl = (slice(b, b + 1), slice(h, h + 1))
        o_ref, l_ref = oracle.attn_ref(np.ascontiguousarray(q[sl]), np.ascontiguousarray(k[sl]), np.ascontiguousarray(v[sl]),
                                       w.dtype, w.scale, w.causal)
        G.check(o[sl], l[sl], o_ref, l_ref, "%s head (%d,%d)" % (name, b, h))


# ------------------------------------------------------------ the forms for few and for many tiles
# Few heads, 128-row tiles whose keys two wave groups share (group B sees keys 32 ... 63 of every 64, none at all up
# to N = 32 and in the first rows of a causal head); many heads, 256-row tiles: each form by name, whatever a plain call would take.  Lengths around the 32-key shares, the 64-key tiles
# and the 128- and 256-row tiles; keys with a few dominant rows, so that the two groups end with different references.
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,lengths,rows", [(2, (1, 32, 33, 64, 65, 96, 97, 127, 129, 161, 2049), 128), (300, (33, 97, 129, 257), 256), (300, (33, 129, 545), 128)])
def test_few_and_many_tiles(G, oracle, H, lengths, rows, d, causal):
    for N in lengths:
        dtype = I.BF16 if N % 3 == 0 else I.FP16
        q, k, v = I.make_qkv(1, H, N, d, dtype, 2000 + N + d, peaky=True)
        print("case few/many tiles H%d N%d d%d causal%d dtype%d rows%d" % (H, N, d, causal, dtype, rows), flush=True)
        o, l = G.run_gpu(q, k, v, dtype, 1.0 / math.sqrt(d), causal, rows=rows)
        for h in (0, H - 1):
            sl = (slice(0, 1), slice(h, h + 1))
            o_ref, l_ref = oracle.attn_ref(np.ascontiguousarray(q[sl]), np.ascontiguousarray(k[sl]), np.ascontiguousarray(v[sl]),
                                           dtype, 1.0 / math.sqrt(d), causal)
            # rows that one key dominates carry the rounding of |O| up to ~4 (half a bf16 ulp there is 7.8e-3 ... 1.6e-2) and of P
            G.check(o[sl], l[sl], o_ref, l_ref, "H%d N%d d%d head %d" % (H, N, d, h), tol_o_max=4e-2 if dtype == I.BF16 else 2e-2)


# ------------------------------------------------------------ properties that hold at any size
def test_c4_properties(G):
    """Non-causal: permuting K and V rows together leaves O and LSE unchanged (up to rounding order)."""
    w = I.WORKLOADS["c4"]
    q, k, v = I.make_qkv(1, 2, w.N, w.d, w.dtype, w.seed)
    o1, l1 = G.run_gpu(q, k, v, w.dtype, w.scale, False)
    perm = np.random.Generator(np.random.Philox(3)).permutation(w.N)
    o2, l2 = G.run_gpu(q, np.ascontiguousarray(k[:, :, perm]), np.ascontiguousarray(v[:, :, perm]), w.dtype, w.scale, False)
    assert np.abs(o1 - o2).max() < 5e-3
    assert np.abs(l1 - l2).max() < 1e-3
    # |O| is a convex combination of V rows
    vf = G.bits_to_f64(G.to_device_bits(v), w.dtype)
    assert np.all(o1.max(axis=2) <= vf.max(axis=2) + 1e-2) and np.all(o1.min(axis=2) >= vf.min(axis=2) - 1e-2)


# ------------------------------------------------------------ degenerate and extreme inputs
@pytest.mark.parametrize("causal", [False, True])
def test_zero_q_gives_running_mean(G, oracle, causal):
    B, H, N, d = 1, 2, 300, 64
    _, k, v = I.make_qkv(B, H, N, d, I.FP16, 91)
    q = np.zeros_like(k)
    o_ref, l_ref = oracle.attn_ref(q, k, v, I.FP16, 0.125, causal)
    o, l = G.run_gpu(q, k, v, I.FP16, 0.125, causal)
    G.check(o, l, o_ref, l_ref, "zero-q", tol_lse=1e-4)


# Keys that score -inf for every query (an infinite element, or a product beyond the range of fp32) weigh nothing, wherever
# they lie: the first keys of a row, the first or second half of its first tile (the shares of the two wave groups in the
# form for few tiles), whole tiles.  Rows that see no other key have no defined result and are left out.
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,N,tile", [(2, 333, 128), (300, 300, 256)])
@pytest.mark.parametrize("dtype,low", [(I.FP16, -np.inf), (I.BF16, -3e38)])
def test_keys_that_score_minus_infinity(G, oracle, dtype, low, H, N, tile, d, causal):
    for first, last in ((0, 32), (32, 64), (0, 64), (0, 128), (64, 192)):
        q, k, v = I.make_qkv(1, H, N, d, dtype, 2100 + first + last)
        four, bad = I.to_bits(np.array([4.0, low], dtype=np.float32), dtype)
        q[..., 0] = four
        k[..., 0] = 0
        k[:, :, first:last, 0] = bad
        print("case -inf keys %d..%d H%d N%d d%d causal%d dtype%d rows%d" % (first, last, H, N, d, causal, dtype, tile), flush=True)
        o, l = G.run_gpu(q, k, v, dtype, 1.0 / math.sqrt(d), causal, rows=tile)
        rows = np.arange(last if causal and first == 0 else 0, N)
        for h in (0, H - 1):
            sl = (slice(0, 1), slice(h, h + 1))
            o_ref, l_ref = oracle.attn_ref(np.ascontiguousarray(q[sl]), np.ascontiguousarray(k[sl]), np.ascontiguousarray(v[sl]),
                                           dtype, 1.0 / math.sqrt(d), causal)
            G.check(o[sl][:, :, rows], l[sl][:, :, rows], o_ref[:, :, rows], l_ref[:, :, rows], "-inf keys %d..%d head %d" % (first, last, h))


# A NaN query spoils its own row of O and LSE, a NaN key the rows that see it; every other row is what it is without the NaN, bit for bit.
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,N,rows", [(3, 333, 128), (300, 577, 256)])
def test_nan_stays_in_its_rows(G, oracle, H, N, rows, d, causal):
    dtype = I.BF16 if d == 64 else I.FP16
    q, k, v = I.make_qkv(1, H, N, d, dtype, 2400 + N + d)
    scale, nan = 1.0 / math.sqrt(d), 0x7FC0 if dtype == I.BF16 else 0x7E00
    o0, l0 = G.run_gpu(q, k, v, dtype, scale, causal, rows=rows)
    places = [(0, 20), (0, 37), (0, N - 1), (1, 0), (H - 1, 131), (H - 1, N - 5)]
    for what in ("query", "key"):
        x = (q if what == "query" else k).copy()
        seen = np.zeros((1, H, N), dtype=bool)           # rows that meet a NaN
        for h, i in places:
            if what == "key" and (h, i) not in ((0, 37), (H - 1, N - 5)): continue
            x[0, h, i, (5 * i) % d] = nan
            if what == "query": seen[0, h, i] = True
            else: seen[0, h, i if causal else 0:] = True
        print("case NaN %s H%d N%d d%d causal%d rows%d" % (what, H, N, d, causal, rows), flush=True)
        o, l = G.run_gpu(*((x, k, v) if what == "query" else (q, x, v)), dtype, scale, causal, rows=rows)
        sl = (slice(0, 1), slice(0, 1))
        o_ref, _ = oracle.attn_ref(*(np.ascontiguousarray(y[sl]) for y in ((x, k, v) if what == "query" else (q, x, v))), dtype, scale, causal)
        assert np.array_equal(np.isnan(o_ref).all(-1), seen[sl]) and np.array_equal(np.isnan(o_ref).any(-1), seen[sl])
        assert np.array_equal(np.isnan(o).all(-1), seen) and np.array_equal(np.isnan(l), seen)
        assert np.array_equal(o[~seen], o0[~seen]) and np.array_equal(l[~seen], l0[~seen])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("H,rows", [(1, 128), (130, 256)])
def test_a_dominating_key_at_every_place_of_a_tile(G, H, rows, causal, d):
    # Query i looks at key 64 + i % 64 (its features are a scaled copy of that key's, the key rows being nearly orthogonal sign
    # patterns): the reference moves in the second tile, through whichever lane holds that key, and O is that key's row of V.
    # Bounds: the score gap is d * gain / sqrt(d) against cross terms
    # of at most gain * sqrt(d) * 5.5 / sqrt(d) (5.5 standard deviations over the 64 x 447 pairs), so the other keys weigh less than
    # 512 exp(-gain (sqrt(d) - 5.5)) < 1e-12 and O is V[key] rounded to 16 bits, which it is already: equal.
    import torch
    N, gain = 512, 16.0
    gen = torch.Generator().manual_seed(5)
    k = torch.where(torch.rand((1, H, N, d), generator=gen) < 0.5, -1.0, 1.0)
    v = torch.randn((1, H, N, d), generator=gen).to(torch.float16)
    place = 64 + torch.arange(N) % 64
    q = k[:, :, place] * gain
    q, k, v = (x.to(torch.float16).cuda() for x in (q, k, v))
    print("case dominating key H%d d%d causal%d rows%d" % (H, d, causal, rows), flush=True)
    o = torch.full_like(v, float("nan"))
    lse = torch.full((1, H, N), float("nan"), device="cuda")
    G._launch(None, G.binding.load_library().attn_fwd_by_rows, q, k, v, o, lse, (1, H, N, d), 1.0 / math.sqrt(d), causal, I.FP16, rows)
    torch.cuda.synchronize()
    seen = slice(128, N) if causal else slice(0, N)     # rows that see the key in either mask
    place = place.cuda()
    assert torch.equal(o[:, :, seen], v[:, :, place][:, :, seen])
    want = gain * math.sqrt(d)
    assert (lse[:, :, seen] - want).abs().max().item() <= 1e-5 * want


@pytest.mark.parametrize("dtype", [I.FP16, I.BF16])
def test_large_scores_exercise_rescaling(G, oracle, dtype):
    # scores with |s| up to ~60 and a maximum that keeps moving along the key axis
    B, H, N, d = 1, 2, 700, 128
    q = I.normal_bits((B, H, N, d), dtype, 92, std=2.0)
    rng = np.random.Generator(np.random.Philox(93))
    kf = rng.standard_normal((B, H, N, d), dtype=np.float32) * (0.5 + 2.5 * np.arange(N, dtype=np.float32)[None, None, :, None] / N)
    k = I.to_bits(kf, dtype)
    v = I.normal_bits((B, H, N, d), dtype, 94)
    scale = 1.0 / math.sqrt(d)
    o_ref, l_ref = oracle.attn_ref(q, k, v, dtype, scale, False)
    o, l = G.run_gpu(q, k, v, dtype, scale, False)
    # near one-hot rows: O inherits the 16-bit rounding of P and of the output, |O| up to ~4
    G.check(o, l, o_ref, l_ref, "large-scores", tol_o_max=4e-2 if dtype == I.BF16 else 2e-2, tol_lse=2e-2)


# The 256-row kernels: their steady state, more than eight key
# tiles, followed by a ragged end, with row tiles that end at different places; ends that put the epilogue's pieces in each of the
# ring's slots.  The first and the last head, and every element written.
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,dtype", [(64, I.FP16), (64, I.BF16), (128, I.FP16)])
def test_ragged_ends_with_many_heads(G, oracle, d, dtype, causal):
    for N in (577, 700, 800, 1000, 1531):
        H = 300 if N <= 700 else 70
        q, k, v = I.make_qkv(1, H, N, d, dtype, 2200 + N + d)
        print("case ragged many heads H%d N%d d%d causal%d dtype%d" % (H, N, d, causal, dtype), flush=True)
        o, l = G.run_gpu(q, k, v, dtype, 1.0 / math.sqrt(d), causal, rows=256)
        assert np.isfinite(o).all() and np.isfinite(l).all()
        for h in (0, H - 1):
            sl = (slice(0, 1), slice(h, h + 1))
            o_ref, l_ref = oracle.attn_ref(np.ascontiguousarray(q[sl]), np.ascontiguousarray(k[sl]), np.ascontiguousarray(v[sl]),
                                           dtype, 1.0 / math.sqrt(d), causal)
            G.check(o[sl], l[sl], o_ref, l_ref, "H%d N%d d%d head %d" % (H, N, d, h))


# The split form above 4 MiB of O (another way of storing it), one round and two
@pytest.mark.parametrize("d,H,N,causal", [(128, 8, 3900, False), (128, 8, 3900, True), (64, 16, 2005, False), (64, 16, 2005, True), (128, 16, 2700, True)])
def test_split_form_with_a_large_result(G, oracle, d, H, N, causal):
    q, k, v = I.make_qkv(1, H, N, d, I.FP16, 2300 + N)
    print("case split, large result H%d N%d d%d causal%d" % (H, N, d, causal), flush=True)
    o, l = G.run_gpu(q, k, v, I.FP16, 1.0 / math.sqrt(d), causal, rows=128)
    assert np.isfinite(o).all() and np.isfinite(l).all()
    sl = (slice(0, 1), slice(H - 1, H))
    o_ref, l_ref = oracle.attn_ref(np.ascontiguousarray(q[sl]), np.ascontiguousarray(k[sl]), np.ascontiguousarray(v[sl]), I.FP16, 1.0 / math.sqrt(d), causal)
    G.check(o[sl], l[sl], o_ref, l_ref, "split, large result H%d N%d d%d" % (H, N, d))


# The same growing keys as above with 256-row tiles; the first heads keep the tolerances.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_large_scores_with_many_heads(G, oracle, causal, d):
    H, N, dtype = 100, 700, I.BF16
    scale = 1.0 / math.sqrt(d)
    q = I.normal_bits((1, H, N, d), dtype, 192, std=2.0)
    rng = np.random.Generator(np.random.Philox(193))
    kf = rng.standard_normal((1, H, N, d), dtype=np.float32) * (0.5 + 2.5 * np.arange(N, dtype=np.float32)[None, None, :, None] / N)
    k = I.to_bits(kf, dtype)
    v = I.normal_bits((1, H, N, d), dtype, 194)
    print("case large scores many heads d%d causal%d" % (d, causal), flush=True)
    o, l = G.run_gpu(q, k, v, dtype, scale, causal, rows=256)
    for h in (0, H - 1):
        sl = (slice(0, 1), slice(h, h + 1))
        o_ref, l_ref = oracle.attn_ref(np.ascontiguousarray(q[sl]), np.ascontiguousarray(k[sl]), np.ascontiguousarray(v[sl]), dtype, scale, causal)
        G.check(o[sl], l[sl], o_ref, l_ref, "large-scores head %d" % h, tol_o_max=4e-2, tol_lse=2e-2)


def test_more_heads_than_a_grid_has_workgroups(G):
    # 2^23 rows of one token: a grid of that many workgroups of 512 threads would be too large.  O is V, LSE the one score.
    import torch
    H, d = 2 ** 23, 64
    print("case one token, 2^23 heads, causal", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(7)
    q, k, v = (torch.randn((1, H, 1, d), generator=gen, device="cuda", dtype=torch.float16) for _ in range(3))
    o = torch.full_like(v, float("nan"))
    lse = torch.full((1, H, 1), float("nan"), device="cuda")
    G.binding.attn_fwd(q, k, v, o, lse, 1, H, 1, d, 0.125, True)
    torch.cuda.synchronize()
    assert torch.equal(o, v)
    # (sums of 64 products of N(0,1) values in fp32, |score| < 10)
    assert (lse[0, :, 0] - (q[0, :, 0].float() * k[0, :, 0].float()).sum(-1) * 0.125).abs().max().item() < 1e-4


def test_score_shift_moves_lse_only(G):
    B, H, N, d = 1, 1, 512, 64
    scale, c = 0.125, 24.0
    rng = np.random.Generator(np.random.Philox(95))
    qf = rng.standard_normal((B, H, N, d), dtype=np.float32)
    kf = rng.standard_normal((B, H, N, d), dtype=np.float32)
    qf[..., d - 1] = 0.0
    kf[..., d - 1] = 0.0
    v = I.normal_bits((B, H, N, d), I.FP16, 96)
    o0, l0 = G.run_gpu(I.to_bits(qf, I.FP16), I.to_bits(kf, I.FP16), v, I.FP16, scale, False)
    qf[..., d - 1] = 1.0
    kf[..., d - 1] = c / scale
    o1, l1 = G.run_gpu(I.to_bits(qf, I.FP16), I.to_bits(kf, I.FP16), v, I.FP16, scale, False)
    assert np.abs(o0 - o1).max() < 2e-3
    assert np.abs(l1 - l0 - c).max() < 1e-3


def test_repeat_runs_are_bit_identical(G):
    q, k, v = I.make_qkv(2, 4, 777, 128, I.BF16, 97)
    o0, l0 = G.run_gpu(q, k, v, I.BF16, 0.09, True)
    for _ in range(5):
        o, l = G.run_gpu(q, k, v, I.BF16, 0.09, True)
        assert np.array_equal(o, o0) and np.array_equal(l, l0)


def test_non_default_stream(G, oracle):
    import torch
    q, k, v = I.make_qkv(1, 2, 200, 64, I.FP16, 98)
    o_ref, l_ref = oracle.attn_ref(q, k, v, I.FP16, 0.125, True)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        o, l = G.run_gpu(q, k, v, I.FP16, 0.125, True)
    G.check(o, l, o_ref, l_ref, "side-stream")


def test_argument_errors_on_device_pointers(G):
    import torch
    from paper_2510_14719_amd import binding
    t = torch.zeros(1 * 1 * 64 * 64 + 64, dtype=torch.float16, device="cuda")
    l = torch.zeros(64, dtype=torch.float32, device="cuda")
    o = torch.zeros_like(t)
    assert binding.attn_fwd_raw(t, t, t, o, l, 1, 1, 64, 64, 0.125, 0, None, 0) == 0
    assert binding.attn_fwd_raw(t, t, t, o, l, 1, 1, 64, 96, 0.125, 0, None, 0) == -2
    assert binding.attn_fwd_raw(t, t, t, o, l, 1, 1, 64, 64, -1.0, 0, None, 0) == -3
    assert binding.attn_fwd_raw(t[1:], t, t, o, l, 1, 1, 64, 64, 0.125, 0, None, 0) == -4
    assert binding.attn_fwd_raw(t, t, t, t, l, 1, 1, 64, 64, 0.125, 0, None, 0) == -7
    torch.cuda.synchronize()
