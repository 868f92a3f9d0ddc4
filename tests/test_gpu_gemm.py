"""Parity of the HIP matrix product (through the C ABI) with the fp64 CPU oracle.

Tolerance (derived from the arithmetic: exact 16-bit x 16-bit products, fp32 accumulation over K terms,
one final rounding to 16 bit): |C_gpu - C_ref| <= 1.01 * u * |C_ref| + 2e-6 * K, with u = 2^-11 for
fp16 and 2^-8 for bf16 (half an ulp of the output); the second term bounds the accumulated fp32
rounding for N(0,1) operands (K * 2^-24 * sum|a||b| / sqrt(K) in the typical case) with a wide margin.
"""
import numpy as np
import pytest

from paper_2510_14719_amd import inputs as I

pytestmark = pytest.mark.gpu

U = {I.FP16: 2.0 ** -11, I.BF16: 2.0 ** -8}


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available(), "the gpu tests need a GPU"
    from paper_2510_14719_amd import binding
    from oracle import gemm_ref
    binding.load_library()
    gemm_ref.build()
    return torch, binding, gemm_ref


def run_gpu(env, a, b, dtype, pad=512, config=None, finite=True, shape=None):
    torch, binding, _ = env
    M, K = a.shape
    N = b.shape[0]
    da = torch.from_numpy(a.view(np.int16)).cuda()
    db = torch.from_numpy(b.view(np.int16)).cuda()
    buf = torch.full((M * N + 2 * pad,), 0x7FFF, dtype=torch.int16, device="cuda")
    c = buf[pad:pad + M * N]
    if shape is None:
        binding.gemm_nt(da, db, c, M, N, K, dtype=dtype, config=config)
    else:                                    # the kernel by name, whatever a plain call would take
        assert binding.load_library().gemm_nt_by_shape(da.data_ptr(), db.data_ptr(), c.data_ptr(), M, N, K, torch.cuda.current_stream().cuda_stream, dtype, shape) == 0
    torch.cuda.synchronize()
    assert bool((buf[:pad] == 0x7FFF).all()) and bool((buf[pad + M * N:] == 0x7FFF).all()), "guard words overwritten"
    # (the buffer started out as NaN patterns: a finite C proves that every element was written)
    assert bool(torch.isfinite(c.view(torch.bfloat16 if dtype == I.BF16 else torch.float16)).all()) or not finite, "an element of C was never written"
    cc = c.view(torch.bfloat16 if dtype == I.BF16 else torch.float16).reshape(M, N)
    return cc


def check(c_gpu, c_ref, dtype, K, what):
    err = np.abs(c_gpu - c_ref)
    tol = 1.01 * U[dtype] * np.abs(c_ref) + 2e-6 * K
    worst = float((err / tol).max())
    print("%s: max err %.3e, worst err/tol %.3f" % (what, err.max(), worst), flush=True)
    assert np.isfinite(c_gpu).all(), what + ": non-finite C"
    assert worst <= 1.0, what


@pytest.mark.parametrize("dtype", [I.FP16, I.BF16])
@pytest.mark.parametrize("M,N,K", [(1, 1, 32), (5, 3, 64), (256, 256, 32), (256, 256, 96), (257, 255, 128), (300, 200, 160),
                                     (64, 1000, 256), (1000, 777, 512), (513, 1031, 64), (768, 512, 1024)])
def test_full_compare(env, M, N, K, dtype):
    _, _, G = env
    a, b = I.make_ab(M, N, K, dtype, seed=100 + M + N + K)
    print("case gemm M%d N%d K%d dtype%d" % (M, N, K, dtype), flush=True)
    ref = G.gemm_nt(a, b, dtype)
    c = run_gpu(env, a, b, dtype).double().cpu().numpy()
    check(c, ref, dtype, K, "full M%d N%d K%d" % (M, N, K))


@pytest.mark.parametrize("config", [1, 2, 3, 4])
@pytest.mark.parametrize("M,N,K,dtype", [(1, 1, 32, I.FP16), (257, 255, 64, I.BF16), (300, 520, 160, I.FP16), (640, 513, 1056, I.FP16),
                                           (256, 256, 2048, I.BF16)])
def test_every_kernel_configuration_in_full(env, M, N, K, dtype, config):
    # the four kernels with fixed tiles: each must handle every shape, one and two K tiles, odd and even tile
    # counts, overhanging tiles
    _, _, G = env
    a, b = I.make_ab(M, N, K, dtype, seed=600 + M + N + K)
    print("case gemm config%d M%d N%d K%d dtype%d" % (config, M, N, K, dtype), flush=True)
    ref = G.gemm_nt(a, b, dtype)
    c = run_gpu(env, a, b, dtype, config=config).double().cpu().numpy()
    check(c, ref, dtype, K, "config %d M%d N%d K%d" % (config, M, N, K))
    # the configurations add the K tiles of an entry in the same order: bit-identical results
    c1 = run_gpu(env, a, b, dtype, config=1).double().cpu().numpy()
    assert np.array_equal(c, c1)


# One to eleven 128-byte steps along K around the ring depths (4, 2, 4) of the small-tile shapes, whole and with a half-filled
# last step (K % 64 == 32), tiles that overhang by one row or column and by all but one, rows of C on and off 16-byte boundaries.
@pytest.mark.parametrize("shape,M,N,Ks", [(1, 65, 63, (32, 64, 96, 128, 192, 224, 256, 288, 320, 352, 704)), (1, 64, 128, (288, 640)),
                                          (1, 127, 136, (32, 320)), (2, 1937, 1936, (32, 64, 96, 128, 192)), (2, 1921, 2047, (160, 256)),
                                          (3, 1025, 1929, (4096,)), (3, 1793, 1793, (4000,))])
@pytest.mark.parametrize("dtype", [I.FP16, I.BF16])
def test_small_tile_shapes(env, shape, M, N, Ks, dtype):
    _, binding, G = env
    for K in Ks:
        assert binding.load_library().gemm_nt_shape(M, N, K) == shape
        a, b = I.make_ab(M, N, K, dtype, seed=1100 + M + N + K)
        print("case gemm shape%d M%d N%d K%d dtype%d" % (shape, M, N, K, dtype), flush=True)
        c = run_gpu(env, a, b, dtype, shape=shape)
        if M * N * K < 1e9:
            check(c.double().cpu().numpy(), G.gemm_nt(a, b, dtype), dtype, K, "shape %d M%d N%d K%d" % (shape, M, N, K))
        else:
            idx = np.asarray(I.sample_entries(M, N, min(4096, M * N // 2), seed=K, always=[(0, 0), (M - 1, N - 1), (0, N - 1), (M - 1, 0)]))
            check(c[idx[:, 0], idx[:, 1]].double().cpu().numpy(), G.gemm_nt_samples(a, b, dtype, idx), dtype, K,
                  "shape %d M%d N%d K%d" % (shape, M, N, K))


# The smallest tiles, each by name: 16 x 16 (512-byte stages, 16-bit operands) and 32 x 32 (256-byte stages); and what a plain call takes: 16 x 16
# up to 256 of them, else 32 x 32 up to 256, and two to a CU from 4096-byte rows on (16-bit), else 64 x 64 again.  One to six stages around the ring depth of four and more, last
# stages of every length (multiples of 64 bytes), tiles that overhang by all but one row and column; rows of C on
# and off 16-byte boundaries, nothing outside C written.
@pytest.mark.parametrize("kind", ["fp16", "bf16", "e4m3"])
@pytest.mark.parametrize("M,N,rows", [(1, 1, (64, 512, 2112)), (17, 33, tuple(range(64, 1089, 64)) + (1536, 2048, 2112, 2560, 2624, 3072, 6208)),
                                      (250, 203, (64, 448, 576, 4160)), (256, 256, (512, 1984)), (33, 8191, (64, 320, 1024)),
                                      (300, 301, tuple(range(64, 577, 64)) + (768, 832, 1024, 1088, 1280, 1344, 1536, 4032)), (512, 505, (192, 2112)),
                                      (641, 577, (64, 128, 192, 256, 512, 576, 640, 1408, 4032, 4096, 4160)), (1040, 488, (4096,))])
def test_smallest_tiles(env, kind, M, N, rows):
    torch, binding, G = env
    lib = binding.load_library()
    f8, dtype = kind == "e4m3", I.BF16 if kind == "bf16" else I.FP16
    launch, tile_of, by_shape = ((lib.gemm_nt_fp8_by_narrow_tile, lib.gemm_nt_fp8_narrow_tile, lib.gemm_nt_fp8_by_shape) if f8 else
                                 (lib.gemm_nt_by_narrow_tile, lib.gemm_nt_narrow_tile, lib.gemm_nt_by_shape))
    view = {"fp16": torch.float16, "bf16": torch.bfloat16, "e4m3": torch.float8_e4m3fn}[kind]
    out = torch.bfloat16 if kind == "bf16" else torch.float16
    for row_bytes in rows:
        K = row_bytes if f8 else row_bytes // 2
        print("case gemm smallest tiles %s M%d N%d K%d" % (kind, M, N, K), flush=True)
        gen = torch.Generator(device="cuda").manual_seed(M + N + K)
        a, b = (torch.randn((r, K), generator=gen, device="cuda").to(view) for r in (M, N))
        stream = torch.cuda.current_stream().cuda_stream
        skew = (M + K // 32) % 2                 # C on a 256-byte boundary, or one element behind it
        if f8:                                   # one order of summation in every kernel
            want = torch.empty((M, N), dtype=out, device="cuda")
            binding.gemm_nt_fp8(a, b, want, M, N, K, out_dtype=dtype, config=1)
        else:
            ref = (a.double() @ b.double().T).cpu().numpy()
        results = {}
        for tile in (32,) if f8 else (16, 32):
            buf = torch.full((M * N + 256,), 7.0, dtype=out, device="cuda")
            c = buf[128 + skew:128 + skew + M * N].view(M, N)
            c.fill_(float("nan"))
            assert launch(a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, stream, dtype, tile) == 0
            if f8:
                assert torch.equal(c, want)
            else:
                check(c.double().cpu().numpy(), ref, dtype, K, "tiles of %d, %s M%d N%d K%d" % (tile, kind, M, N, K))
            assert bool((buf[:128 + skew] == 7.0).all()) and bool((buf[128 + skew + M * N:] == 7.0).all())
            results[tile] = c
        d, e = (torch.empty((M, N), dtype=out, device="cuda") for _ in range(2))
        if f8:
            binding.gemm_nt_fp8(a, b, d, M, N, K, out_dtype=dtype)
        else:
            binding.gemm_nt(a, b, d, M, N, K)
        tile = tile_of(M, N, K)
        if tile == 0:
            assert by_shape(a.data_ptr(), b.data_ptr(), e.data_ptr(), M, N, K, stream, dtype, 1) == 0
        assert torch.equal(d, results[tile] if tile else e)


# The 256 x 256 kernel with whole lines per row, called directly: one to six 128-byte steps (ring of two and a half), with and
# without a half-filled last one, many steps; tiles that overhang by little and by nearly all.  On E4M3 it
# adds the k-steps in the order of the fixed configurations, so its results are theirs, bit for bit (16-bit operands take
# MFMAs of another shape).  A first step that is not whole is refused.
@pytest.mark.parametrize("kind", ["fp16", "bf16", "e4m3"])
@pytest.mark.parametrize("M,N", [(256, 256), (257, 511), (300, 40)])
def test_whole_line_kernel(env, kind, M, N):
    torch, binding, G = env
    lib = binding.load_library()
    launch = lib.gemm_nt_fp8_by_shape if kind == "e4m3" else lib.gemm_nt_by_shape
    f8, dtype = kind == "e4m3", I.BF16 if kind == "bf16" else I.FP16
    view = {"fp16": torch.float16, "bf16": torch.bfloat16, "e4m3": torch.float8_e4m3fn}[kind]
    out = torch.bfloat16 if kind == "bf16" else torch.float16
    for row_bytes in (128, 192, 256, 320, 384, 448, 512, 576, 640, 704, 768, 4096, 4160):
        K = row_bytes if f8 else row_bytes // 2
        print("case gemm whole lines %s M%d N%d K%d" % (kind, M, N, K), flush=True)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(M + N + K)
        a, b = (torch.randn((r, K), generator=gen, device="cuda").to(view) for r in (M, N))
        c, want = (torch.full((M, N), float("nan"), dtype=out, device="cuda") for _ in range(2))
        assert launch(a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, K, torch.cuda.current_stream().cuda_stream, dtype, 0) == 0
        if f8:
            binding.gemm_nt_fp8(a, b, want, M, N, K, out_dtype=dtype, config=1)
            assert torch.equal(c, want)
        else:
            ref = a.double().cpu() @ b.double().cpu().T
            check(c.double().cpu().numpy(), ref.numpy(), dtype, K, "whole lines %s K%d" % (kind, K))
    assert launch(a.data_ptr(), b.data_ptr(), c.data_ptr(), M, N, 64 if f8 else 32, None, dtype, 0) == -2


# Rows of C that allow 16-, 8- and 2-byte stores, and a C that is aligned to less than its rows are; tiles that overhang by one
# row and column, by most of a 32-row block and by whole waves; nothing outside C is written.
@pytest.mark.parametrize("config", [2, 4])
@pytest.mark.parametrize("M,N,skew", [(256, 264, 0), (255, 260, 0), (289, 131, 0), (97, 512, 4), (257, 256, 1), (33, 392, 8)])
def test_large_tile_stores(env, config, M, N, skew):
    torch, binding, G = env
    K, dtype = 96, I.BF16
    a, b = I.make_ab(M, N, K, dtype, seed=1300 + M + N)
    print("case gemm stores config%d M%d N%d skew%d" % (config, M, N, skew), flush=True)
    ad, bd = (torch.from_numpy(x.view(np.int16)).cuda().view(torch.bfloat16) for x in (a, b))
    buf = torch.full((M * N + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    c = buf[16 + skew:16 + skew + M * N].view(M, N)
    assert binding.gemm_nt_raw(ad, bd, c, M, N, K, None, dtype, config=config) == 0
    check(c.double().cpu().numpy(), G.gemm_nt(a, b, dtype), dtype, K, "stores config%d M%d N%d" % (config, M, N))
    assert bool((buf[:16 + skew] == 7.0).all()) and bool((buf[16 + skew + M * N:] == 7.0).all())


# The ways C leaves: whole memory lines are written through the L2 from 4 MiB on, every other tile of them past the caches from 96 MiB
# on and all above 128 MiB, anything else with ordinary stores.  The same product into a C that starts on a line and into one that does not (always ordinary) has the
# same bits, in every kernel; rows and columns overhang the tiles; nothing outside C is written.
@pytest.mark.parametrize("kind", ["bf16", "e4m3"])
@pytest.mark.parametrize("M,N,K", [(2049, 1024, 64), (2101, 3008, 512), (4099, 4160, 256), (4099, 4160, 2048), (7001, 8256, 64), (7001, 8256, 1024), (16400, 8256, 64), (16400, 8256, 1024)])
def test_ways_of_storing_c(env, kind, M, N, K):
    torch, binding, _ = env
    print("case gemm ways of storing %s M%d N%d K%d" % (kind, M, N, K), flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K)
    a, b = (torch.randn((r, K), generator=gen, device="cuda").to(torch.bfloat16 if kind == "bf16" else torch.float8_e4m3fn) for r in (M, N))
    out = []
    for skew in (0, 1):
        buf = torch.full((M * N + 128,), 7.0, dtype=torch.bfloat16, device="cuda")
        c = buf[64 + skew:64 + skew + M * N]
        assert (c.data_ptr() % 128 == 0) == (skew == 0)
        if kind == "bf16":
            binding.gemm_nt(a, b, c, M, N, K)
        else:
            binding.gemm_nt_fp8(a, b, c, M, N, K, out_dtype=I.BF16)
        assert bool((buf[:64 + skew] == 7.0).all()) and bool((buf[64 + skew + M * N:] == 7.0).all())
        out.append(c)
    assert torch.equal(*out)
    rows = torch.tensor([0, M // 2, M - 1], device="cuda")
    ref = a[rows].double() @ b.double().T
    err = (out[0].view(M, N)[rows].double() - ref).abs()
    # half an ulp of the bf16 result, and 2e-6 K for fp32 sums (see the top) or, on E4M3, whose matrix instruction adds its 64
    # products in a narrower frame, 2^-14 of the sum of their magnitudes
    slack = 2e-6 * K if kind == "bf16" else 2.0 ** -14 * (a[rows].double().abs() @ b.double().abs().T)
    assert bool((err <= 1.01 * U[I.BF16] * ref.abs() + slack).all())


def test_odd_n(env):
    _, _, G = env
    M, N, K = 130, 37, 96                     # rows of C are not aligned to more than an element
    a, b = I.make_ab(M, N, K, I.FP16, seed=7)
    c = run_gpu(env, a, b, I.FP16).double().cpu().numpy()
    check(c, G.gemm_nt(a, b, I.FP16), I.FP16, K, "odd N")


def test_exact_small_integers(env):
    # products and sums of small integers are exact in fp32 and in the 16-bit output: bit-exact result
    torch, _, G = env
    rng = np.random.Generator(np.random.Philox(5))
    M, N, K = 300, 280, 64
    a = I.to_bits(rng.integers(-3, 4, size=(M, K)).astype(np.float32), I.FP16)
    b = I.to_bits(rng.integers(-3, 4, size=(N, K)).astype(np.float32), I.FP16)
    c = run_gpu(env, a, b, I.FP16).double().cpu().numpy()
    assert np.array_equal(c, G.gemm_nt(a, b, I.FP16))


@pytest.mark.parametrize("K", [256, 8192, 16384])
def test_paper_sweep_sizes_sampled(env, K):
    # M = N = 8192 (the benchmark's launch configuration), sampled entries against the oracle
    torch, binding, G = env
    M = N = 8192
    a, b = I.make_ab(M, N, K, I.FP16, seed=900 + K)
    print("case gemm sweep K%d" % K, flush=True)
    c = run_gpu(env, a, b, I.FP16)
    idx = I.sample_entries(M, N, 96, seed=901 + K, always=[(0, 0), (M - 1, N - 1), (0, N - 1), (M - 1, 0), (255, 256), (4096, 4095)])
    ref = G.gemm_nt_samples(a, b, I.FP16, idx)
    ii = np.asarray(idx)
    got = c[ii[:, 0], ii[:, 1]].double().cpu().numpy()
    check(got, ref, I.FP16, K, "sweep K%d" % K)
    # a property that holds at any size: the sum over each row of C equals A times the column sums of B^T
    bs = torch.from_numpy(b.view(np.int16)).cuda().view(torch.float16).double().sum(dim=0)       # [K]
    af = torch.from_numpy(a.view(np.int16)).cuda().view(torch.float16).double()
    row_sums_ref = (af @ bs).cpu().numpy()
    row_sums = c.double().sum(dim=1).cpu().numpy()
    # each of the N entries of a row carries at most half an ulp of rounding, of random sign
    bound = 6.0 * np.sqrt(N) * U[I.FP16] * np.sqrt(K) * 4 + 1e-6 * K * N ** 0.5
    assert np.abs(row_sums - row_sums_ref).max() <= bound


def test_repeat_runs_are_bit_identical_and_errors(env):
    torch, binding, _ = env
    a, b = I.make_ab(512, 512, 256, I.BF16, seed=9)
    c0 = run_gpu(env, a, b, I.BF16).clone()
    for _ in range(3):
        assert torch.equal(run_gpu(env, a, b, I.BF16), c0)
    t = torch.zeros(64 * 64 + 16, dtype=torch.float16, device="cuda")
    c = torch.zeros(64 * 64, dtype=torch.float16, device="cuda")
    assert binding.gemm_nt_raw(t, t, c, 64, 64, 64, None, 0) == 0
    assert binding.gemm_nt_raw(t, t, c, 64, 64, 40, None, 0) == -2
    assert binding.gemm_nt_raw(t[1:], t, c, 64, 64, 64, None, 0) == -4
    assert binding.gemm_nt_raw(t, t, t, 64, 64, 64, None, 0) == -7
    torch.cuda.synchronize()
