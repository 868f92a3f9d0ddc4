"""Which attention calls take 128-row tiles with the keys shared out between the halves of a workgroup (host logic, no GPU).

``MEASURED`` holds calls on both sides of every line of the rule with the times of both forms on MI355X (us, three sets of
buffers in turn): the rule takes the faster form, or one that is at most 3 % slower."""
import pytest

# d, N, heads, causal, 8-bit floats, whole tiles, split tiles
MEASURED = [
    # one round
    (128, 128, 2, 0, 0, 8.2, 7.8), (64, 128, 2, 0, 0, 5.38, 5.23), (64, 64, 200, 0, 0, 4.46, 4.43), (128, 256, 100, 1, 0, 11.9, 10.8),
    (64, 200, 100, 0, 1, 6.96, 6.05), (64, 256, 8, 1, 1, 7.11, 6.15), (64, 100, 100, 0, 1, 4.81, 5.06), (64, 64, 8, 0, 1, 4.06, 4.47),
    (128, 256, 100, 0, 1, 10.2, 10.5), (128, 150, 100, 1, 1, 9.0, 10.7), (128, 257, 85, 0, 1, 10.6, 11.4), (128, 320, 66, 0, 1, 10.5, 11.0),
    (128, 352, 85, 0, 1, 12.3, 11.1), (128, 577, 51, 0, 1, 15.6, 13.3), (128, 320, 85, 1, 1, 11.6, 12.9), (128, 448, 64, 1, 1, 13.1, 14.5),
    (128, 400, 50, 1, 1, 12.8, 13.4), (128, 352, 42, 1, 1, 11.8, 11.6), (128, 640, 51, 1, 1, 15.7, 15.1), (128, 1024, 32, 1, 1, 21.9, 19.2),
    # more than one round without the mask
    (128, 1024, 64, 0, 0, 37.5, 49.9), (128, 1024, 64, 0, 1, 24.0, 33.0), (64, 512, 100, 0, 1, 10.4, 14.3), (64, 256, 400, 0, 0, 15.4, 18.8),
    # two rounds under the mask: the range of an XCD is half a head, one head or two
    (128, 7168, 8, 1, 0, 144.5, 113.5), (128, 3584, 16, 1, 0, 75.8, 63.5), (128, 15616, 4, 1, 0, 314.6, 305.5), (128, 7424, 8, 1, 1, 104.7, 72.2),
    # ... a short second round, or many rows
    (128, 2816, 12, 1, 0, 56.4, 41.0), (128, 5327, 7, 1, 0, 101.6, 77.2), (128, 6331, 7, 1, 0, 121.2, 108.3), (128, 3584, 10, 1, 1, 54.8, 42.8),
    (128, 10325, 5, 1, 1, 141.4, 117.7), (128, 11930, 5, 1, 1, 162.8, 148.7),
    # ... and neither
    (128, 3840, 17, 1, 0, 85.4, 106.0), (128, 6144, 9, 1, 0, 124.9, 142.0), (128, 2560, 21, 1, 0, 55.2, 61.9), (128, 2048, 32, 1, 0, 49.3, 55.9),
    (128, 2048, 21, 1, 0, 43.4, 47.8), (128, 1024, 64, 1, 0, 28.7, 38.8), (128, 3584, 18, 1, 1, 56.4, 67.2), (128, 2048, 32, 1, 1, 37.5, 43.2),
    (128, 2304, 27, 1, 1, 39.6, 47.6),
    # d = 64
    (64, 2816, 14, 1, 0, 49.9, 43.1), (64, 2048, 28, 1, 0, 37.9, 39.7), (64, 8192, 8, 1, 0, 139.2, 105.1), (64, 1024, 64, 1, 0, 22.0, 23.5),
    (64, 4060, 12, 1, 1, 52.8, 36.0), (64, 4096, 64, 1, 1, 155.6, 138.4), (64, 2048, 64, 1, 1, 56.6, 51.6), (64, 1280, 50, 1, 1, 20.1, 24.1),
]


# The same for the lines that more than one round of whole tiles brought (kernels with 16 x 16 MFMAs).
MEASURED_ROUNDS = [
    # one round, short E4M3 rows
    (128, 239, 65, 0, 1, 9.0, 8.3), (128, 251, 6, 0, 1, 8.8, 7.9), (128, 148, 127, 0, 1, 7.8, 8.5), (128, 227, 94, 1, 1, 9.3, 8.7), (128, 399, 47, 1, 1, 11.5, 9.7),
    (128, 123, 101, 1, 1, 6.6, 7.4), (128, 111, 132, 0, 1, 6.2, 7.2),
    # without the mask
    (64, 1905, 42, 0, 0, 64.8, 57.9), (64, 4510, 25, 0, 0, 152.9, 166.8), (64, 123, 340, 0, 0, 9.2, 8.2), (64, 300, 333, 0, 0, 22.2, 19.9), (64, 485, 348, 0, 0, 32.1, 37.4),
    (64, 2727, 81, 0, 0, 172.3, 175.0), (128, 3729, 26, 0, 0, 182.9, 228.4), (128, 135, 347, 0, 0, 20.7, 25.6), (128, 71, 268, 0, 0, 14.5, 13.3), (128, 38, 1168, 0, 0, 24.7, 26.9),
    (128, 5484, 16, 0, 1, 162.2, 138.2), (128, 4510, 23, 0, 1, 135.3, 157.3), (128, 4999, 28, 0, 1, 231.1, 219.8), (128, 281, 198, 0, 1, 20.0, 25.1),
    (64, 345, 131, 0, 1, 15.9, 12.7), (64, 954, 56, 0, 1, 16.3, 21.7),
    # under the mask
    (128, 6575, 11, 1, 0, 238.1, 163.1), (128, 4739, 21, 1, 0, 201.4, 159.2), (128, 3150, 40, 1, 0, 106.2, 119.6), (128, 742, 127, 1, 0, 43.1, 44.9),
    (128, 7599, 14, 1, 1, 195.9, 145.8), (128, 4833, 15, 1, 1, 83.2, 85.8), (128, 891, 100, 1, 1, 34.1, 35.1),
    (64, 80, 264, 1, 0, 11.4, 7.0), (64, 1926, 285, 1, 0, 315.7, 212.2), (64, 69, 2061, 1, 0, 44.2, 24.7), (64, 1024, 256, 1, 0, 57.9, 68.2), (64, 1846, 62, 1, 0, 66.0, 51.7),
    (64, 251, 1487, 1, 0, 60.7, 54.9),
]


@pytest.fixture(scope="module")
def lib():
    from paper_2510_14719_amd import binding
    return binding.load_library()


@pytest.mark.parametrize("d,N,heads,causal,fp8,whole,split", MEASURED + MEASURED_ROUNDS)
def test_the_faster_form_is_taken(lib, d, N, heads, causal, fp8, whole, split):
    rows = (lib.attn_fwd_fp8_call_rows if fp8 else lib.attn_fwd_call_rows)(1, heads, N, d, causal)
    assert rows in (128, 256)
    assert (split if rows == 128 else whole) <= 1.03 * min(whole, split)


def test_whole_tiles_beyond_the_largest_grid(lib):
    # one workgroup of 512 threads per split tile, less than 2^32 threads in a grid: whole tiles (persistent at d = 64 under the mask) take
    # what is larger, whatever the rule says of speed
    most = 2 ** 32 // 512 - 1
    for N, tiles in ((1, 1), (66, 1), (130, 2)):
        for f in (lib.attn_fwd_call_rows, lib.attn_fwd_fp8_call_rows):
            for causal in (0, 1):
                assert f(1, most // tiles + 1, N, 64, causal) == 256 and f(1, most // tiles + 1, N, 128, causal) == 256
        assert lib.attn_fwd_call_rows(1, most // tiles, N, 64, 1) == 128


def test_heads_count_over_the_batch_and_sizes_are_checked(lib):
    for f in (lib.attn_fwd_call_rows, lib.attn_fwd_fp8_call_rows):
        assert f(4, 2, 7424, 128, 1) == f(1, 8, 7424, 128, 1) == 128
        assert f(2 ** 15, 2 ** 15, 1024, 64, 0) == 256
        for bad in ((0, 1, 64, 64, 0), (1, 0, 64, 64, 0), (1, 1, 0, 64, 0), (1, 1, 64, 96, 0)):
            assert f(*bad) == -1
