"""GPU parity, scheme U: the HIP path (through the C ABI) against the CPU oracle.

Payload and header must match bit for bit; decoded values must match within
1e-6 * scale (they are in fact produced by the same single float32 multiply)."""
import numpy as np
import pytest

import synthetic_inputs as si
from oracle import accept_oracle as orc

from gpu_util import bytes_to_dev, dev_bytes, first_mismatch, out_to_numpy, to_dev, torch_mod

pytestmark = pytest.mark.gpu

KS = [2, 3, 4, 5, 6, 7, 8]


@pytest.fixture(scope="module")
def A():
    torch = torch_mod()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2311_05827_amd as pkg
    return pkg


def run_case(A, x, k, n, m, channels=0, in_bf16=False, out_bf16=False, rounding=0, seed=0, tag=""):
    torch = torch_mod()
    print("case", tag, "k", k, "n", n, "m", m, "C", channels, "bf16", in_bf16, out_bf16, "rnd", rounding, flush=True)
    xd, bits = to_dev(x, in_bf16)
    d = A.make_desc(A.UNIFORM, k, n, m, channels=channels, in_dtype=A.BF16 if in_bf16 else A.F32,
                    out_dtype=A.BF16 if out_bf16 else A.F32, rounding=rounding, seed=seed)
    header, payload = A.accept_compress(d, xd)
    xh = A.accept_decompress(d, header, payload)
    torch.cuda.synchronize()
    oh, op = orc.uniform_compress(bits if in_bf16 else x, k, n, m, channels, in_bf16, rounding, seed)
    assert dev_bytes(header) == oh, "header differs " + str(first_mismatch(dev_bytes(header), oh))
    mm = first_mismatch(dev_bytes(payload), op.tobytes())
    assert mm is None, "payload differs: " + mm
    oxh = orc.uniform_decompress(oh, op, k, n, m, channels, out_bf16)
    got = out_to_numpy(xh)
    if out_bf16:
        assert got.tolist() == oxh.tolist()
    else:
        scale = float(np.max(np.frombuffer(oh, dtype="<f4"))) * (2 ** (k - 1) - 1)
        assert np.all(np.abs(got.astype(np.float64) - oxh.astype(np.float64)) <= 1e-6 * scale)
        assert got.tobytes() == oxh.tobytes()
    return oh, op


@pytest.mark.parametrize("k", KS)
def test_multi_tile_with_ragged_tail(A, k):
    # three full 8192-element tiles plus a tail that is neither a multiple of 32 nor of 8
    N = 3 * 8192 + 777
    x = si.make_shape("grad_outliers", (1, N), 10 + k)
    run_case(A, x, k, 1, N, tag="ragged")
    x = si.make_shape("relu_normal", (3, 8455), 20 + k)
    run_case(A, x, k, 3, 8455, tag="relu")


@pytest.mark.parametrize("N", [1, 2, 3, 7, 8, 9, 31, 32, 33, 63, 64, 65, 255, 8191, 8192, 8193])
def test_tiny_and_boundary_sizes(A, N):
    for k in KS:
        x = si.make_shape("student_t3", (1, N), 100 + N)
        run_case(A, x, k, 1, N, tag="tiny")


@pytest.mark.parametrize("k", [3, 4, 8])
def test_odd_shapes(A, k):
    x = si.make_shape("student_t3", (3, 5, 7), 5)
    run_case(A, x, k, 3, 35, tag="3x5x7")
    x = si.make_shape("student_t3", (15, 127, 67), 6)
    run_case(A, x, k, 15, 127 * 67, tag="15x127x67")


@pytest.mark.parametrize("k", KS)
@pytest.mark.parametrize("in_bf16,out_bf16", [(True, False), (False, True), (True, True)])
def test_bf16_io(A, k, in_bf16, out_bf16):
    x = si.make_shape("relu_lognormal", (4, 5000), 30 + k)
    run_case(A, x, k, 4, 5000, in_bf16=in_bf16, out_bf16=out_bf16, tag="bf16")
    x = si.make_shape("grad", (2, 8192 + 13), 31 + k)
    run_case(A, x, k, 2, 8192 + 13, in_bf16=in_bf16, out_bf16=out_bf16, tag="bf16-tail")


def test_max_found_at_every_lane_and_block_position(A):
    """The range reduction must see every element: plant the maximum at many positions."""
    N = 5 * 4096 + 5
    base = (si.make_shape("grad", (1, N), 77) * np.float32(0.5)).astype(np.float32)
    for pos in list(range(0, 300, 7)) + [4095, 4096, 8191, 12345, N - 6, N - 5, N - 1]:
        x = base.copy()
        x[0, pos] = np.float32(-3.0)
        oh, _ = run_case(A, x, 8, 1, N, tag="maxpos%d" % pos)
        assert np.frombuffer(oh, dtype="<f4")[0] == np.float32(3.0) / np.float32(127)


def test_all_zero_tiny_and_denormal_tensors(A):
    for k in (2, 5, 8):
        run_case(A, np.zeros((2, 5000), np.float32), k, 2, 5000, tag="zeros")
        run_case(A, np.full((2, 5000), 1e-40, np.float32), k, 2, 5000, tag="denormal")
        run_case(A, np.full((1, 40), 2.0 ** -101, np.float32), k, 1, 40, tag="below-threshold")
        run_case(A, np.full((1, 40), 2.0 ** -100, np.float32), k, 1, 40, tag="at-threshold")
        x = np.zeros((1, 9000), np.float32)
        x[0, 4567] = -1.0
        run_case(A, x, k, 1, 9000, tag="single-spike")


def test_exact_ties_round_to_even(A):
    for k in KS:
        L = 2 ** (k - 1) - 1
        j = np.arange(-2 * L, 2 * L + 1)
        x = np.tile((j * 0.125 / 2).astype(np.float32), 70)[None, :]
        run_case(A, x, k, 1, x.size, tag="ties")


@pytest.mark.parametrize("k", [4, 6, 8])
@pytest.mark.parametrize("in_bf16", [False, True])
def test_per_channel_segmented(A, k, in_bf16):
    # segments of 1024 and 3136 elements (>= 512 and vector aligned): wave-per-segment range pass
    x = si.make_shape("relu_lognormal_chgain", (3, 5, 32, 32), 40 + k)
    run_case(A, x, k, 3, 5 * 1024, channels=5, in_bf16=in_bf16, out_bf16=in_bf16, tag="seg1024")
    x = si.make_shape("relu_lognormal_chgain", (5, 7, 56, 56), 41 + k)
    run_case(A, x, k, 5, 7 * 3136, channels=7, in_bf16=in_bf16, tag="seg3136")
    # a segment longer than one chunk (4096 vectors): 2 x 3 x 20000 floats
    x = si.make_shape("relu_lognormal_chgain", (2, 3, 20000), 42 + k)
    run_case(A, x, k, 2, 60000, channels=3, in_bf16=in_bf16, tag="seg20000")


@pytest.mark.parametrize("k", [2, 5, 8])
def test_per_channel_whole_tiles(A, k):
    """Tensors of whole 8192-element tiles with long segments: the quantize pass finishes the
    channels' ranges itself, tile by tile.  Tiles that touch more segments than there are
    channels, one segment over several tiles (two chunks per segment), many rows (several
    partial maxima per lane), float32 and bfloat16, and the same shapes one row short of whole
    tiles (separate U1b kernel) for comparison."""
    for n, C, seg in [(16, 3, 512), (4, 16, 512), (8, 40, 1024), (2, 5, 8192), (4, 2, 16384), (300, 4, 2048),
                      (64, 3, 1536), (1024, 1, 512)]:
        if C == 1:
            continue  # one channel is the per-tensor mode
        x = si.make_shape("relu_lognormal_chgain", (n, C, seg), 80 + k)
        gain = np.float32(10.0) ** np.linspace(-2, 2, C, dtype=np.float32)
        x = np.ascontiguousarray(x * gain[None, :, None], dtype=np.float32)
        assert (n * C * seg) % 8192 == 0
        run_case(A, x, k, n, C * seg, channels=C, tag="whole tiles seg%d C%d" % (seg, C))
        run_case(A, x, k, n, C * seg, channels=C, in_bf16=True, out_bf16=True, tag="whole tiles bf16")
        run_case(A, x[: n - 1], k, n - 1, C * seg, channels=C, tag="one row short") if (n - 1) * C * seg % 8192 else None
    x = si.make_shape("grad_outliers", (8, 4, 2048), 90 + k)
    run_case(A, x, k, 8, 8192, channels=4, rounding=1, seed=5, tag="whole tiles stochastic")


@pytest.mark.parametrize("k", [3, 8])
def test_more_tiles_than_workgroups(A, k):
    """Tensors of more than 2048 tiles: workgroups take several tiles each, last-read first, and
    step their channel position backwards; a few tiles after the last whole group of eight keep
    their plain places.  One range, one range per channel (with and without whole tiles) and
    one range per element."""
    T = 8192
    # one range: 2051 whole tiles (3 after the reversed part) and a ragged tail
    x = si.make_shape("grad_outliers", (1, 2051 * T + 77), 95 + k)
    run_case(A, x, k, 1, 2051 * T + 77, tag="2051 tiles + tail")
    # one range per channel, whole tiles (ranges finished tile by tile): 64 x 5 x 53248 = 2080 tiles
    x = si.make_shape("relu_lognormal_chgain", (64, 5, 53248), 96 + k)
    run_case(A, x, k, 64, 5 * 53248, channels=5, tag="2080 tiles per channel")
    run_case(A, x, k, 64, 5 * 53248, channels=5, in_bf16=True, out_bf16=True, tag="1040 tiles per channel bf16")
    # few rows, so few partial maxima per channel: the quantize pass finishes the ranges itself,
    # also for the workgroups that take two tiles (16 x 160 x 6656 = 2080 tiles of 2-3 segments)
    x = si.make_shape("relu_lognormal_chgain", (16, 160, 6656), 99 + k)
    run_case(A, x, k, 16, 160 * 6656, channels=160, tag="2080 tiles, ranges per tile")
    run_case(A, x, k, 16, 160 * 6656, channels=160, in_bf16=True, out_bf16=True, tag="1040 tiles bf16, ranges per tile")
    # the same one segment length off whole tiles (range table from the U1b kernel, ragged tail)
    x = si.make_shape("relu_lognormal_chgain", (64, 5, 53256), 97 + k)
    run_case(A, x, k, 64, 5 * 53256, channels=5, tag="2080 tiles + tail per channel")
    # channels-last: 266240 rows of 64 channels = 2080 tiles, and 5 rows more
    x = si.make_shape("grad", (266245, 64), 98 + k) * (np.arange(1, 65, dtype=np.float32)[None, :])
    x = np.ascontiguousarray(x, dtype=np.float32)
    run_case(A, x[:266240], k, 266240, 64, channels=64, tag="2080 tiles channels-last")
    run_case(A, x, k, 266245, 64, channels=64, tag="2080 tiles channels-last + tail")


@pytest.mark.parametrize("k", [3, 4, 8])
def test_per_channel_generic_geometries(A, k):
    # short aligned segments (vector quantize path, column range pass)
    x = si.make_shape("relu_lognormal_chgain", (6, 10, 12), 50 + k)
    run_case(A, x, k, 6, 120, channels=10, tag="seg12")
    x = si.make_shape("relu_lognormal_chgain", (40, 64, 8, 8), 51 + k)
    run_case(A, x, k, 40, 64 * 64, channels=64, tag="seg64")
    run_case(A, x, k, 40, 64 * 64, channels=64, in_bf16=True, out_bf16=True, tag="seg64-bf16")
    # segments that no 16-byte vector respects: element-wise path
    x = si.make_shape("relu_lognormal_chgain", (9, 11, 7), 52 + k)
    run_case(A, x, k, 9, 77, channels=11, tag="seg7")
    x = si.make_shape("relu_lognormal_chgain", (300, 33, 5), 53 + k)
    run_case(A, x, k, 300, 165, channels=33, in_bf16=True, tag="seg5-bf16")
    # one element per channel (channels-last 2-D tensor)
    x = si.make_shape("grad", (50, 96), 54 + k)
    run_case(A, x, k, 50, 96, channels=96, tag="seg1")
    # channels-last with many rows (several row blocks in the column pass), aligned and not
    x = si.make_shape("grad_outliers", (5000, 256), 55 + k)
    run_case(A, x, k, 5000, 256, channels=256, tag="channels-last 256")
    run_case(A, x, k, 5000, 256, channels=256, in_bf16=True, out_bf16=True, tag="channels-last 256 bf16")
    x = si.make_shape("relu_lognormal", (3001, 30, 11), 56 + k)
    run_case(A, x, k, 3001, 330, channels=30, tag="seg11 unaligned rows")
    x = si.make_shape("student_t3", (37, 1300, 3), 57 + k)
    run_case(A, x, k, 37, 3900, channels=1300, tag="seg3 wide")


@pytest.mark.parametrize("k", KS)
def test_channels_last_one_range_per_element(A, k):
    """Rows of C channels with one element each and a gain per channel spanning six decades: whole
    tiles (vector path, every element of a vector its own range) plus a ragged tail, float32 and
    bfloat16, nearest-even and stochastic; row lengths that no 16-byte vector divides take the plain path."""
    for rows, C in [(700, 64), (301, 136), (1237, 40), (530, 36), (2100, 8)]:
        x = si.make_shape("grad", (rows, C), 70 + k)
        gain = np.float32(10.0) ** np.linspace(-3, 3, C, dtype=np.float32)
        x = np.ascontiguousarray(x * gain[None, :], dtype=np.float32)
        run_case(A, x, k, rows, C, channels=C, tag="channels-last %d" % C)
        run_case(A, x, k, rows, C, channels=C, in_bf16=True, out_bf16=True, tag="channels-last %d bf16" % C)
    run_case(A, x, k, rows, C, channels=C, rounding=1, seed=77, tag="channels-last stochastic")


def test_channels_last_decoder_with_unaligned_header(A):
    """A header that is only 4-byte aligned (the contract's minimum) decodes to the same values."""
    torch = torch_mod()
    rows, C, k = 900, 64, 5
    x = si.make_shape("grad", (rows, C), 91) * (np.arange(1, C + 1, dtype=np.float32)[None, :])
    x = np.ascontiguousarray(x, dtype=np.float32)
    xd, _ = to_dev(x)
    d = A.make_desc(A.UNIFORM, k, rows, C, channels=C)
    header, payload = A.accept_compress(d, xd)
    ref = A.accept_decompress(d, header, payload)
    shifted = torch.empty(header.numel() + 4, dtype=torch.uint8, device=header.device)
    shifted[4:] = header
    got = A.accept_decompress(d, shifted[4:], payload)
    torch.cuda.synchronize()
    assert shifted[4:].data_ptr() % 16 == 4
    oh, op = orc.uniform_compress(x, k, rows, C, C)
    assert out_to_numpy(got).tobytes() == orc.uniform_decompress(oh, op, k, rows, C, C).tobytes()
    assert out_to_numpy(ref).tobytes() == out_to_numpy(got).tobytes()


@pytest.mark.parametrize("k", [2, 4, 7, 8])
def test_stochastic_rounding_bit_exact(A, k):
    x = si.make_shape("grad_outliers", (2, 8192 + 100), 60 + k)
    run_case(A, x, k, 2, 8292, rounding=1, seed=1234567, tag="stoch")
    run_case(A, x, k, 2, 8292, rounding=1, seed=(1 << 63) + 5, tag="stoch-bigseed")
    run_case(A, x, k, 4, 4146, channels=2, rounding=1, seed=9, in_bf16=True, tag="stoch-ch")


@pytest.mark.parametrize("k,bf16,seed", [(4, False, (1 << 64) - 3), (8, True, 11)])
def test_stochastic_rounding_over_many_tiles(A, k, bf16, seed):
    """More 8192-element tiles than workgroups, tiles in reversed order plus leftovers: the random
    state a workgroup carries from tile to tile is the one of the element's index."""
    N = 2061 * 8192 + 41
    run_case(A, si.make_shape("grad", (1, N), 64), k, 1, N, rounding=1, seed=seed, in_bf16=bf16, tag="stoch-tiles")


def per_channel_input(n, C, seg, seed):
    x = si.make_shape("grad", (n, C, seg), seed)
    gain = (np.float32(2.0) ** np.random.default_rng(seed).integers(-6, 7, C)).astype(np.float32)
    return np.ascontiguousarray(x * gain[None, :, None], dtype=np.float32)


@pytest.mark.parametrize("seg", [5, 6, 7, 9, 11, 49, 50, 196, 1023])
def test_segments_that_are_not_whole_vectors(A, seg):
    """Vectors across the border of two channels, and of the last channel and the next row's first."""
    for n, C, k, bf16, rounding in ((3, 2, 5, False, 0), (9, 37, 6, True, 0), (40, 5, 8, False, 1), (7, 300, 4, True, 1)):
        x = per_channel_input(n, C, seg, 300 + seg)
        run_case(A, x, k, n, C * seg, channels=C, in_bf16=bf16, out_bf16=bf16, rounding=rounding, seed=5, tag="straddling")
    if seg == 49:  # more tiles than workgroups
        x = per_channel_input(64, 5376, seg, 350)
        run_case(A, x, 3, 64, 5376 * seg, channels=5376, tag="straddling, many tiles")


@pytest.mark.parametrize("values,bf16", [(3 << 19, False), (1 << 21, True), (5 << 19, False), (5 << 19, True)])
@pytest.mark.parametrize("seg", [9, 201])
def test_straddling_segments_by_size(A, seg, values, bf16):
    """Both sides of the sizes from which such a tensor is compressed in vectors (1572864 and
    2097152 values) and decompressed in tiles (2621440 values)."""
    row = 41 * seg
    for n in (values // row, values // row + 1):
        assert (n * row >= values) == (n != values // row)
        x = per_channel_input(n, 41, seg, 360 + seg)
        x[n - 1, 40, seg - 1] = 100.0
        for rounding in (0, 1):
            run_case(A, x, 5, n, row, channels=41, in_bf16=bf16, out_bf16=bf16, rounding=rounding, seed=5, tag="straddling by size")


@pytest.mark.parametrize("seg", [512, 516, 520, 784, 1024, 1032, 2048, 2056, 4096, 4104, 8200, 20488])
def test_segment_lengths_of_the_range_pass(A, seg):
    """One, two, four and eight loads per lane and chunk, chunks that fill them and that do not."""
    for n, C, k, bf16 in ((3, 5, 4, False), (2, 17, 6, True), (13, 3, 8, seg % 8 == 0)):
        x = per_channel_input(n, C, seg, 400 + n)
        x[n - 1, C - 1, seg - 1] = 100.0   # the very last element of the tensor
        x[0, 0, 0] = -90.0
        run_case(A, x, k, n, C * seg, channels=C, in_bf16=bf16, out_bf16=bf16, tag="segments")


@pytest.mark.parametrize("n,C", [(1, 512), (65, 511), (65, 513), (520, 1000), (4099, 528), (3, 4097), (200, 300001)])
def test_channels_last_range(A, n, C):
    """Wide channels-last tensors: the fold of 16 channels per workgroup, ragged channel counts,
    one and many row blocks, and the largest value in the last row and channel."""
    x = per_channel_input(n, C, 1, 450 + n)
    x[n - 1, C - 1, 0] = 100.0
    x[0, 0, 0] = -90.0
    for k, bf16 in ((4, False), (7, True)):
        run_case(A, x, k, n, C, channels=C, in_bf16=bf16, out_bf16=bf16, tag="channels-last")


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 4 * 8192 - 1, 16 * 8192 - 1, 16 * 8192, 16 * 8192 + 1, 21 * 8192 + 5])
def test_single_columns_by_rows(A, rows):
    """Rows of 9 channels, which no 16-byte vector divides: a thread's share of the rows below, at and
    above the 16 and 4 that it takes at a time."""
    x = per_channel_input(rows, 9, 1, 460)
    x[rows - 1, 8, 0] = 100.0
    x[0, 0, 0] = -90.0
    for k, bf16 in ((4, False), (7, True)):
        run_case(A, x, k, rows, 9, channels=9, in_bf16=bf16, out_bf16=bf16, tag="single columns")


# One range, nearest rounding, 48 (bfloat16: 72) to 256 MiB: the end of the tensor is kept on the chip between the
# range and the quantizer.  256 workgroups, units of 16384 elements; per workgroup 7 (bfloat16: 14)
# units in registers, 2 (4) in local memory; what this does not hold, from the tenth (19th) round of units on, is read twice, 2 (4) units
# at a time and what is left over by a division in front of them.
HELD_ROUND = 256 * 16384


@pytest.mark.parametrize("k,N,bf16", [
    (8, 3 * HELD_ROUND, False),                      # the smallest, no tail
    (3, 3 * HELD_ROUND + 5 * 16384 + 8193, False),   # a few workgroups with one unit more, a tile and one element behind
    (5, 7 * HELD_ROUND + 16384, False),              # local memory comes into use
    (4, 10 * HELD_ROUND - 16384 * 7 + 33, False),    # one unit per workgroup is read twice, some have none
    (7, 7 * HELD_ROUND + 31, True),                  # bfloat16 below its own line: two reads
    (7, 9 * HELD_ROUND + 31, True),                  # the smallest in bfloat16
    (7, 12 * HELD_ROUND + 16384 * 64, False),        # four are read twice
    (5, 13 * HELD_ROUND + 16384 * 3 + 9, True),      # as many as there are slots
    (5, 14 * HELD_ROUND + 16384 * 3 + 9, True),      # local memory comes into use
    (6, 17 * HELD_ROUND + 16384 * 255, True),        # the largest that fits, but for a unit
    (6, 18 * HELD_ROUND + 16384 * 255, True),        # one, two, three per workgroup are read twice
    (3, 19 * HELD_ROUND + 16384 * 7 + 1, True),
    (8, 20 * HELD_ROUND + 16384, True),
    (2, 30 * HELD_ROUND + 8192, True),               # twelve
    (4, 30 * HELD_ROUND + 16384 * 9 + 77, True),     # thirteen
])
def test_held_pass(A, k, N, bf16):
    d = A.make_desc(A.UNIFORM, k, 1, N, in_dtype=A.BF16 if bf16 else A.F32)
    assert A.accept_stage_name(d, 0, 0) == ("range" if N == 7 * HELD_ROUND + 31 else "quantize_held")
    x = si.make_shape("grad", (1, N), 200 + k)
    x[0, N - 1 - N // 7] = 0.5  # the largest value, far from either end
    run_case(A, x, k, 1, N, in_bf16=bf16, out_bf16=bf16, tag="held")


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("tail", [0, 1, 63, 64, 65, 8191, 8192, 8193, 16383])
def test_held_pass_largest_value_at_the_end(A, tail, bf16):
    """The largest value in the last element, in the first one behind the last whole unit and in the
    last whole unit, whether the workgroups see each other's maxima or give up."""
    torch = torch_mod()
    k, N = 8, (9 if bf16 else 3) * HELD_ROUND + 16384 * 3 + tail
    print("held, tail", tail, "bf16", bf16, flush=True)
    base = si.make_shape("grad", (1, N), 230 + tail % 7)
    d = A.make_desc(A.UNIFORM, k, 1, N, in_dtype=A.BF16 if bf16 else A.F32)
    header, payload, ws = A.alloc_outputs(d, "cuda")
    for at in sorted({N - 1, N - max(tail, 1), N - tail - 1, N - tail - 16384}):
        x = base.copy()
        x[0, at] = -0.5
        xd, bits = to_dev(x, bf16)
        oh, op = orc.uniform_compress(bits if bf16 else x, k, 1, N, 0, bf16)
        for polls in (64, 0):
            A.accept_compress_polls(d, xd, header, payload, ws, polls)
            torch.cuda.synchronize()
            assert dev_bytes(header) == oh, (N - at, polls)
            assert first_mismatch(dev_bytes(payload), op.tobytes()) is None, (N - at, polls)


def test_held_pass_that_gives_up(A):
    """A workgroup that does not see the others' maxima in time finds them itself; whatever share of them does
    (0, some, none), the bytes are the same, and the workspace is ready for the next call."""
    torch = torch_mod()
    k, N = 5, 3 * HELD_ROUND + 16384 * 9 + 100
    xs = [torch.from_numpy(si.make_shape("grad", (N,), 220 + i) * np.float32(1 + i)).cuda() for i in range(2)]
    d = A.make_desc(A.UNIFORM, k, 1, N)
    assert [A.accept_stage_name(d, 0, i) for i in range(2)] == ["quantize_held", None]
    want = [orc.uniform_compress(x.cpu().numpy(), k, 1, N) for x in xs]
    header, payload, ws = A.alloc_outputs(d, "cuda")
    for polls in (0, 1, 2, 64, 0, 3, 64):
        for x, (oh, op) in zip(xs, want):
            payload.zero_()
            A.accept_compress_polls(d, x, header, payload, ws, polls)
            torch.cuda.synchronize()
            assert dev_bytes(header) == oh, polls
            assert first_mismatch(dev_bytes(payload), op.tobytes()) is None, polls


@pytest.mark.parametrize("k,N,bf16,largest_behind", [
    (5, 9 * HELD_ROUND + 33, False, True),             # the largest that fits
    (8, 8 * HELD_ROUND + 16384, False, False),         # one workgroup has a ninth unit
    (6, 17 * HELD_ROUND + 16384 * 5 + 77, True, True),   # bfloat16: some have an 18th, which fits
    (5, 9 * HELD_ROUND + 16384 * 5 + 33, False, True),   # some have a tenth: one unit of everyone's is read twice
    (8, 12 * HELD_ROUND + 16384 * 64 + 8193, False, False),  # four
    (6, 18 * HELD_ROUND + 16384 * 5 + 77, True, True),   # bfloat16: one
    (3, 20 * HELD_ROUND + 16384 * 250 + 1, True, False),  # three
])
def test_held_pass_of_more_than_fits_that_gives_up(A, k, N, bf16, largest_behind):
    """As above, for tensors that fill what can be kept, or of which only a part is: a workgroup that gives up reads all of its units
    again, those that it kept as well, by the loop that reads what was not kept."""
    torch = torch_mod()
    print("case", k, N, bf16, flush=True)
    d = A.make_desc(A.UNIFORM, k, 1, N, in_dtype=A.BF16 if bf16 else A.F32)
    assert [A.accept_stage_name(d, 0, i) for i in range(2)] == ["quantize_held", None]
    header, payload, ws = A.alloc_outputs(d, "cuda")
    for turn in range(2):
        x = si.make_shape("grad", (1, N), 225 + turn)
        x[0, N - 1 if largest_behind and turn == 1 else N // 3] = -0.5
        xd, bits = to_dev(x, bf16)
        oh, op = orc.uniform_compress(bits if bf16 else x, k, 1, N, 0, bf16)
        for polls in (0, 1, 2, 64):
            header.zero_()
            payload.zero_()
            A.accept_compress_polls(d, xd, header, payload, ws, polls)
            torch.cuda.synchronize()
            assert dev_bytes(header) == oh, (turn, polls)
            assert first_mismatch(dev_bytes(payload), op.tobytes()) is None, (turn, polls)


def test_held_pass_and_what_earlier_calls_left(A):
    """The mailboxes (64-bit words from byte 8192 on, value and number of the exchange) keep what the last call
    posted, or an earlier one where later calls had fewer workgroups.  The next call takes none of it for its own."""
    torch = torch_mod()
    k, N = 8, 3 * HELD_ROUND
    x = torch.from_numpy(si.make_shape("grad", (N,), 227)).cuda()
    oh, op = orc.uniform_compress(x.cpu().numpy(), k, 1, N)
    d = A.make_desc(A.UNIFORM, k, 1, N)
    header, payload, ws = A.alloc_outputs(d, "cuda")
    number = ws[8192 + 3 * 2048:8192 + 3 * 2048 + 1024].view(torch.int32)  # of exchanges so far, by workgroup
    A.accept_compress(d, x, header=header, payload=payload, workspace=ws)
    for back in (0, 1, 5):
        for boxes in (slice(0, 256), slice(3, 4)):
            torch.cuda.synchronize()
            now = int(number[0])
            assert number.tolist() == [now] * 256 and now > 0
            left = (max(now - back, 0) << 32) | int(np.float32(7.0).view(np.uint32))
            ws[8192:8192 + 2048].view(torch.int64)[boxes] = left
            for call in range(2):
                A.accept_compress(d, x, header=header, payload=payload, workspace=ws)
                torch.cuda.synchronize()
                assert dev_bytes(header) == oh, (back, boxes, call)
                assert first_mismatch(dev_bytes(payload), op.tobytes()) is None, (back, boxes, call)


def test_held_pass_on_two_streams_and_in_a_graph(A):
    """Calls that overlap on two streams (each with its own buffers) compete for the compute units
    the held pass waits on; a captured call is replayed on new inputs between eager ones."""
    torch = torch_mod()
    k, N = 6, 3 * HELD_ROUND + 16384 * 20 + 5
    xs = [torch.from_numpy(si.make_shape("grad", (N,), 240 + i) * np.float32(1 + i)).cuda() for i in range(3)]
    d = A.make_desc(A.UNIFORM, k, 1, N)
    want = [orc.uniform_compress(x.cpu().numpy(), k, 1, N) for x in xs]
    bufs = [A.alloc_outputs(d, "cuda") for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for turn in range(6):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                header, payload, ws = bufs[i]
                for rep in range(3):
                    A.accept_compress(d, xs[(turn + i + rep) % 3], header=header, payload=payload, workspace=ws)
        torch.cuda.synchronize()
        for i in range(2):
            oh, op = want[(turn + i + 2) % 3]
            assert dev_bytes(bufs[i][0]) == oh, (turn, i)
            assert first_mismatch(dev_bytes(bufs[i][1]), op.tobytes()) is None, (turn, i)
    header, payload, ws = bufs[0]
    x = xs[0].clone()
    with torch.cuda.stream(streams[0]):
        A.accept_compress(d, x, header=header, payload=payload, workspace=ws)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        A.accept_compress(d, x, header=header, payload=payload, workspace=ws)
    for i in (1, 2, 0, 1):
        x.copy_(xs[i])
        payload.zero_()
        g.replay()
        torch.cuda.synchronize()
        oh, op = want[i]
        assert dev_bytes(header) == oh and first_mismatch(dev_bytes(payload), op.tobytes()) is None, i
        A.accept_compress(d, xs[2], header=header, payload=payload, workspace=ws)  # eager, same workspace
        torch.cuda.synchronize()
        assert dev_bytes(header) == want[2][0]


def test_decoder_on_oracle_stream(A):
    """Feed the oracle's own header and payload to the GPU decoder."""
    torch = torch_mod()
    for k in KS:
        for N in (5, 64, 8192 * 2 + 50):
            x = si.make_shape("student_t3", (1, N), 70 + k)
            oh, op = orc.uniform_compress(x, k, 1, N)
            d = A.make_desc(A.UNIFORM, k, 1, N)
            xh = A.accept_decompress(d, bytes_to_dev(oh), bytes_to_dev(op.tobytes() + b"\0" * 16)[: op.size])
            torch.cuda.synchronize()
            assert xh.cpu().numpy().tobytes() == orc.uniform_decompress(oh, op, k, 1, N).tobytes()


def test_payload_tail_is_not_overwritten(A):
    """Bytes after ceil(N k / 8) belong to the caller."""
    torch = torch_mod()
    for k, N in [(3, 8192 + 5), (5, 77), (7, 3), (2, 9)]:
        x = si.make_shape("grad", (1, N), 80 + k)
        xd, _ = to_dev(x)
        d = A.make_desc(A.UNIFORM, k, 1, N)
        hb, pb = A.accept_packed_size(d)
        buf = torch.full((pb + 64,), 0xAB, dtype=torch.uint8, device="cuda")
        A.accept_compress(d, xd, payload=buf[:pb])
        torch.cuda.synchronize()
        assert buf[pb:].cpu().numpy().tolist() == [0xAB] * 64
        assert buf[:pb].cpu().numpy().tobytes() == orc.uniform_compress(x, k, 1, N)[1].tobytes()


# One range per channel, segments of whole 32s, a tensor that fits on the chip: one kernel, in which a workgroup
# has consecutive groups of 32 elements of the order channel, row, place, and channels may lie in several.
@pytest.mark.parametrize("n,C,seg,k,bf16", [
    (4, 5, 1024, 4, False),        # the smallest channels; whole channels per workgroup
    (3, 7, 1568, 5, True),         # shared channels, a last workgroup with little to do
    (130, 2, 32, 3, False),        # segments of one group
    (130, 2, 32, 8, True),
    (2, 3, 20000, 7, False),       # few channels, many workgroups each
    (1, 2, 300000, 2, True),
    (16, 300, 512, 6, False),      # channels of 256 groups, some shared
    (9, 100, 992, 7, True),        # a segment that no unit divides
    (33, 260, 1024, 4, False),     # three units per workgroup
    (33, 260, 1024, 5, True),
    (64, 100, 3136, 6, False),     # local memory comes into use
    (60, 256, 3136, 6, True),
    (7 * 64, 256, 256, 3, False),  # the most that fits, float32
    (7 * 64 + 1, 256, 256, 3, False),  # and one row more: range and quantizer
])
def test_channels_on_the_chip(A, n, C, seg, k, bf16):
    torch = torch_mod()
    print("case", n, C, seg, k, bf16, flush=True)
    x = si.make_shape("relu_lognormal_chgain", (n, C, seg), 300 + k)
    gain = np.float32(10.0) ** np.linspace(-2, 2, C, dtype=np.float32)
    x = np.ascontiguousarray(x * gain[None, :, None], dtype=np.float32)
    xd, bits = to_dev(x, bf16)
    d = A.make_desc(A.UNIFORM, k, n, C * seg, channels=C, in_dtype=A.BF16 if bf16 else A.F32)
    fits = n * C * seg <= (14 if bf16 else 7) * HELD_ROUND
    assert (A.accept_stage_name(d, 0, 0) == "quantize_channels") == fits
    oh, op = orc.uniform_compress(bits if bf16 else x, k, n, C * seg, C, bf16)
    header, payload, ws = A.alloc_outputs(d, "cuda")
    for polls in (64, 0, 64):  # seen by each other; every shared channel read by all that have a part of it
        payload.zero_()
        A.accept_compress_polls(d, xd, header, payload, ws, polls)
        torch.cuda.synchronize()
        assert dev_bytes(header) == oh, polls
        assert first_mismatch(dev_bytes(payload), op.tobytes()) is None, polls


@pytest.mark.parametrize("n,C,seg,k,bf16", [
    (1, 2, 12845056, 8, False),    # the largest form, both channels in 128 workgroups
    (2, 3, 4300032, 5, True),      # a workgroup in two channels
    (16, 4, 100352, 4, False),
    (64, 16, 25088, 6, False),
])
def test_few_large_channels_that_are_not_seen_in_time(A, n, C, seg, k, bf16):
    """Where workgroups look in vain, they share out what is missing of a channel: the bytes are the same, and it
    costs a few exchanges, not the whole channel once per workgroup (115 times as long, two channels of 51 MB)."""
    torch = torch_mod()
    print("case", n, C, seg, k, bf16, flush=True)
    x = si.make_shape("grad", (n, C, seg), 320 + k)
    x[n - 1, C - 1, seg - 1] = 0.5
    xd, bits = to_dev(x, bf16)
    d = A.make_desc(A.UNIFORM, k, n, C * seg, channels=C, in_dtype=A.BF16 if bf16 else A.F32)
    assert A.accept_stage_name(d, 0, 0) == "quantize_channels"
    oh, op = orc.uniform_compress(bits if bf16 else x, k, n, C * seg, C, bf16)
    header, payload, ws = A.alloc_outputs(d, "cuda")
    took = {}
    for polls in (64, 0, 1, 2, 64, 0):
        times = []
        for _ in range(5):
            payload.zero_()
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            A.accept_compress_polls(d, xd, header, payload, ws, polls)
            end.record()
            torch.cuda.synchronize()
            times.append(begin.elapsed_time(end))
        took[polls] = sorted(times)[2]
        assert dev_bytes(header) == oh, polls
        assert first_mismatch(dev_bytes(payload), op.tobytes()) is None, polls
    print(took, flush=True)
    assert took[0] < 8 * took[64], took


def test_channels_on_the_chip_on_two_streams_and_in_a_graph(A):
    """Workgroups of two calls compete for the compute units; one workspace serves descriptors with different
    numbers of workgroups; a captured call is replayed on new inputs between eager ones."""
    torch = torch_mod()
    n, C, seg, k = 40, 96, 3136, 6
    xs = [torch.from_numpy(si.make_shape("relu_lognormal_chgain", (n, C, seg), 310 + i) * np.float32(1 + i)).cuda() for i in range(3)]
    d = A.make_desc(A.UNIFORM, k, n, C * seg, channels=C)
    small = A.make_desc(A.UNIFORM, k, 6, C * seg, channels=C)
    want = [orc.uniform_compress(x.cpu().numpy(), k, n, C * seg, C) for x in xs]
    want_small = orc.uniform_compress(xs[0][:6].cpu().numpy(), k, 6, C * seg, C)
    bufs = [A.alloc_outputs(d, "cuda") for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for turn in range(4):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                header, payload, ws = bufs[i]
                for rep in range(3):
                    A.accept_compress(d, xs[(turn + i + rep) % 3], header=header, payload=payload, workspace=ws)
        torch.cuda.synchronize()
        for i in range(2):
            oh, op = want[(turn + i + 2) % 3]
            assert dev_bytes(bufs[i][0]) == oh, (turn, i)
            assert first_mismatch(dev_bytes(bufs[i][1]), op.tobytes()) is None, (turn, i)
    header, payload, ws = bufs[0]
    x = xs[0].clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        A.accept_compress(d, x, header=header, payload=payload, workspace=ws)
    for i in (1, 2, 0, 1):
        x.copy_(xs[i])
        payload.zero_()
        g.replay()
        torch.cuda.synchronize()
        oh, op = want[i]
        assert dev_bytes(header) == oh and first_mismatch(dev_bytes(payload), op.tobytes()) is None, i
        h, p = A.accept_compress(small, xs[0][:6].reshape(-1), workspace=ws)  # eager, same workspace
        torch.cuda.synchronize()
        assert dev_bytes(h) == want_small[0] and dev_bytes(p) == want_small[1].tobytes()


# One range, a tensor that stays in registers: one kernel.  Workgroups of at least 512 (stochastic: 128) groups of 32
# elements, at most 256 of them; up to 31 elements behind the last group.
@pytest.mark.parametrize("N,k,bf16,rounding", [
    (32, 4, False, 0),                        # one group
    (63, 3, True, 0),
    (512 * 32 + 31, 8, False, 0),             # one full workgroup and what is behind
    (512 * 32 + 32, 5, False, 0),             # a group more: two workgroups
    (1 << 17, 6, True, 0),
    (1 << 18, 6, False, 0),                   # 16 workgroups
    ((1 << 18) + 1, 7, False, 0),
    (31 * 512 * 32 + 31, 3, False, 0),        # the most workgroups that look at one set of boxes
    (31 * 512 * 32 + 32, 8, True, 0),         # and the fewest that have six
    ((3 << 19) - 1, 4, False, 0),             # the most in parts of 512 groups, float32
    (3 << 19, 8, False, 0),                   # and the fewest in parts of 256
    (256 * 512 * 32, 2, False, 0),            # 256 workgroups of a unit
    (256 * 512 * 32 + 33, 3, False, 0),       # of a unit and a group
    (2 * 256 * 512 * 32, 8, False, 0),
    (2 * 256 * 512 * 32 + 33, 6, False, 0),   # of two units and a group
    (3 * 256 * 512 * 32 - 1, 7, False, 0),    # the most, float32
    (3 * 256 * 512 * 32 + 7, 4, True, 0),     # beyond three units, bfloat16
    (128 * 32 + 5, 8, False, 1),              # stochastic: two workgroups
    (20480, 8, False, 1),
    (255 * 128 * 32 + 9, 4, True, 1),
    (4 * 256 * 512 * 32, 3, False, 1),        # the most, float32
    (3 << 20, 5, True, 1),                    # the most, bfloat16
])
def test_tensor_in_registers(A, N, k, bf16, rounding):
    torch = torch_mod()
    print("case", N, k, bf16, rounding, flush=True)
    seed = 12345 + N
    x = si.make_shape("grad", (1, N), 400 + k)
    x[0, N - 1 - N // 9] = 0.25
    d = A.make_desc(A.UNIFORM, k, 1, N, in_dtype=A.BF16 if bf16 else A.F32, rounding=rounding, seed=seed)
    assert A.accept_stage_name(d, 0, 0) == "quantize_whole"
    header, payload, ws = A.alloc_outputs(d, "cuda")
    for turn in range(2 if N < 1 << 20 else 1):
        if turn == 1:
            x[0, N - 1] = -0.5  # the largest value behind the last group
        xd, bits = to_dev(x, bf16)
        oh, op = orc.uniform_compress(bits if bf16 else x, k, 1, N, 0, bf16, rounding, seed)
        for polls in (64, 0, 1):  # seen by each other; workgroups find each other's maxima
            payload.zero_()
            A.accept_compress_polls(d, xd, header, payload, ws, polls)
            torch.cuda.synchronize()
            assert dev_bytes(header) == oh, polls
            assert first_mismatch(dev_bytes(payload), op.tobytes()) is None, polls
