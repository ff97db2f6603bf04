"""The few-lane kernels: the longest lanes, the numbers of lanes up to which they are taken, the block encoder's batches, the
packer behind it, short lanes in the row decoder."""
import numpy as np
import pytest
import torch

from oracle import pilc_oracle as orc
from paper_2206_05279_amd import binding as pb
from paper_2206_05279_amd import synth

pytestmark = pytest.mark.gpu

from gpu_util import DeviceWorkload, first_difference  # noqa: E402


def test_one_lane_of_more_than_2_to_the_27_symbols():
    h, w = 6700, 6690
    wl = synth.make_random_case(3, 1, 8, 8, 12, 0, 64)
    rng = np.random.default_rng(2)
    wl.h, wl.w, wl.lane_a = h, w, h * w
    wl.img = rng.integers(90, 166, size=(1, h, w, 3), dtype=np.uint8)
    wl.mu = np.full((1, h, w, 3), 128 * 256, dtype=np.uint16)
    wl.log_scale = np.full((1, h, w, 3), 3 * 4096, dtype=np.int16)
    assert 3 * h * w > 1 << 27
    rc, want = orc.encode(orc.make_geom(*wl.geom), wl.img, wl.mu, wl.log_scale, wl.chan_coef)
    assert rc == orc.OK
    d = DeviceWorkload(wl)
    _, nbytes = d.encode()
    got = d.coded_numpy()
    assert nbytes == want.size and np.array_equal(got, want), first_difference(got, want)


def _kernels(call):
    pb.pilc_set_timing(True)
    try:
        call()
        return [name for name, _ in pb.pilc_last_timing()]
    finally:
        pb.pilc_set_timing(False)


# Rows as long as one round of workgroups (two of 16 lanes on a compute unit) takes all lanes.
@pytest.mark.parametrize("over", [0, 1])
def test_decoder_takes_rows_for_one_round_of_workgroups(over):
    lanes = 32 * torch.cuda.get_device_properties(0).multi_processor_count + over
    wl = synth.make_random_case(9, lanes, 4, 4, 12, 0, 16)
    d = DeviceWorkload(wl)
    d.encode()
    assert ("k_decode_rows" in _kernels(d.decode)) == (over == 0)
    assert np.array_equal(d.decoded_numpy(), wl.img)


# The encoder's line by what a chunk of the lanes costs thread per lane: aligned tiles, tiles whose rows are not, flat
# lanes of whole lines, tiny lanes.  The container is the oracle's on both sides of it.
@pytest.mark.parametrize("h,w,mode,a,b,line", [
    (256, 256, 1, 16, 16, 32768), (256, 250, 1, 16, 16, 40960), (64, 61, 1, 8, 8, 36864),
    (32, 32, 0, 64, 0, 40960), (16, 16, 0, 32, 0, 28672)])
def test_encoder_takes_blocks_up_to_its_line(h, w, mode, a, b, line):
    per_image = -(-h // a) * -(-w // b) if mode else h * w // a
    for n in (line // per_image, line // per_image + 1):
        wl = synth.make_random_case(n, n, h, w, 12, mode, a, b) if mode else synth.make_random_case(n, n, h, w, 12, mode, a)
        rc, want = orc.encode(orc.make_geom(*wl.geom), wl.img, wl.mu, wl.log_scale, wl.chan_coef)
        assert rc == orc.OK
        d = DeviceWorkload(wl)
        assert ("k_encode_block" in _kernels(d.encode)) == (n * per_image <= line)
        got = d.coded_numpy()
        assert d.nbytes == want.size and np.array_equal(got, want), first_difference(got, want)


# Lanes of 512 pixels and more whose rows do not align stay with the block encoder for longer: tiles of 16 x 33, four a row
# of images of 16 x 129 (the last one 30 wide), on both sides of the line; the container is the same as the other encoder's.
@pytest.mark.parametrize("over", [0, 1])
def test_encoder_line_of_long_lanes_that_do_not_align(over):
    n = 114688 // 4 + over
    rng = np.random.default_rng(over)
    wl = synth.make_random_case(over, 1, 16, 129, 12, 1, 16, 33)
    wl.n = n
    wl.img = rng.integers(0, 256, size=(n, 16, 129, 3), dtype=np.uint8)
    wl.mu = wl.img.astype(np.uint16) << 8
    wl.log_scale = np.zeros(wl.img.shape, dtype=np.int16)
    wl.chan_coef = np.zeros((n, 3), dtype=np.int16)
    d = DeviceWorkload(wl)
    assert ("k_encode_block" in _kernels(d.encode)) == (over == 0)
    got = d.coded_numpy().copy()
    pb.pilc_set_kernel_policy(1 if over == 0 else 2)
    try:
        d.encode()
        assert np.array_equal(d.coded_numpy(), got)
    finally:
        pb.pilc_set_kernel_policy(0)


# Tiles of one or two whole chunks a row leave it sooner: tiles of 64 x 8, two an image of 64 x 9, and of 32 x 16, two of 32 x 17.
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("h,w,a,b", [(64, 9, 64, 8), (32, 17, 32, 16)])
def test_encoder_line_of_long_lanes_in_whole_chunks(h, w, a, b, over):
    n = 92160 // 2 + over
    rng = np.random.default_rng(over)
    wl = synth.make_random_case(over, 1, h, w, 12, 1, a, b)
    wl.n = n
    wl.img = rng.integers(0, 256, size=(n, h, w, 3), dtype=np.uint8)
    wl.mu = wl.img.astype(np.uint16) << 8
    wl.log_scale = np.zeros(wl.img.shape, dtype=np.int16)
    wl.chan_coef = np.zeros((n, 3), dtype=np.int16)
    d = DeviceWorkload(wl)
    assert ("k_encode_block" in _kernels(d.encode)) == (over == 0)
    got = d.coded_numpy().copy()
    pb.pilc_set_kernel_policy(1 if over == 0 else 2)
    try:
        d.encode()
        assert np.array_equal(d.coded_numpy(), got)
    finally:
        pb.pilc_set_kernel_policy(0)


# Batches of 20, 12 and 8 pixels (one workgroup on a compute unit, two, more): lanes of one pixel, of one less and more than
# a batch, of several; masses from 1 to 2^M - 255, states at both ends of what a mass renormalises.
@pytest.mark.parametrize("prec_bits", [10, 16])
@pytest.mark.parametrize("wild", [False, True])
@pytest.mark.parametrize("groups,pixels", [(0, (1, 19, 20, 21, 61)), (1, (1, 11, 12, 13, 37)), (2, (1, 7, 8, 9, 25))])
def test_block_encoder_at_the_edges_of_its_batches(groups, pixels, wild, prec_bits):
    lanes = 16 * groups * torch.cuda.get_device_properties(0).multi_processor_count + 35
    for px in pixels:
        wl = synth.make_random_case(prec_bits + px, lanes, 1, px, prec_bits, 0, px, wild=wild)
        if not wild:
            wl.log_scale[: lanes // 2] = -16384  # the narrowest law, at the pixel or off it
            wl.mu[: lanes // 4] = wl.img[: lanes // 4].astype(np.uint16) * 256
        rc, want = orc.encode(orc.make_geom(*wl.geom), wl.img, wl.mu, wl.log_scale, wl.chan_coef)
        assert rc == orc.OK
        d = DeviceWorkload(wl)
        assert "k_encode_block" in _kernels(d.encode)
        got = d.coded_numpy()
        assert d.nbytes == want.size and np.array_equal(got, want), first_difference(got, want)


# The packer that moves eight words at a time: lanes of no words, of one to nine and of many side by side, one, two and
# several of them a workgroup; short lanes, of which a workgroup has up to 16, and on both sides of that.
@pytest.mark.parametrize("lanes,pixels", [(70, 400), (70, 6000), (2300, 400), (5000, 400), (2048, 16), (2048, 32), (16384, 16),
                                          (16384, 32), (17407, 24), (17408, 24)])
def test_packer_of_long_lanes(lanes, pixels):
    wl = synth.make_random_case(pixels, lanes, 1, pixels, 16, 0, pixels)
    rng = np.random.default_rng(pixels)
    wl.mu[...] = wl.img.astype(np.uint16) * 256
    wl.log_scale[...] = -16384
    for lane in range(lanes):  # a pixel off its mean takes about a word
        far = rng.choice(pixels, size=min(pixels, lane % 70 if lane % 70 < 40 else 17 * (lane % 70)), replace=False)
        wl.mu[lane, 0, far, 0] ^= 0x4000
    wl.chan_coef[...] = 0
    rc, want = orc.encode(orc.make_geom(*wl.geom), wl.img, wl.mu, wl.log_scale, wl.chan_coef)
    assert rc == orc.OK
    d = DeviceWorkload(wl)
    assert "k_pack" in _kernels(d.encode)
    got = d.coded_numpy()
    assert d.nbytes == want.size and np.array_equal(got, want), first_difference(got, want)
    words = np.diff(want[64:64 + 4 * (lanes + 1)].view("<u4").astype(np.int64)) // 2 - 2
    assert words.min() < 8 <= words.max()


# What the second wavefront of the row decoder prepares goes as far as the longest lane of its wavefront: lanes of one pixel up to a
# batch of 16 and two more, alone, beside lanes of one pixel (edge tiles), with a shorter last lane; with and without that wavefront.
@pytest.mark.parametrize("lanes", [70, 5000])
@pytest.mark.parametrize("px", [1, 3, 4, 5, 8, 12, 13, 15, 16, 17, 20, 31, 33])
def test_row_decoder_on_short_lanes(px, lanes):
    cases = [(lanes, 1, px, 0, px, 0), (lanes // 2, 1, px + 1, 1, 1, px), (lanes * px - px // 2, 1, 1, 0, px, 0)]
    for i, (n, h, w, mode, a, b) in enumerate(cases):
        wl = synth.make_random_case(px + i, n, h, w, 12, mode, a, b)
        d = DeviceWorkload(wl)
        d.encode()
        assert "k_decode_rows" in _kernels(d.decode)
        assert np.array_equal(d.decoded_numpy(), wl.img)


# ... and a call with such lanes does not wait for pixels that they do not have (9.8 and 19.7 us; 15.1 when it did).
def test_row_decoder_of_one_pixel_a_lane_is_sooner_than_of_a_batch():
    times = []
    for px in (1, 16):
        wl = synth.make_random_case(px, 4096, 1, px, 12, 0, px)
        wl.mu[...] = wl.img.astype(np.uint16) << 8  # (every symbol in its window: no search)
        wl.log_scale[...] = 0
        wl.chan_coef[...] = 0
        d = DeviceWorkload(wl)
        d.encode()
        pb.pilc_set_timing(True)
        try:
            took = []
            for _ in range(40):
                d.decode()
                took += [ms for name, ms in pb.pilc_last_timing() if name == "k_decode_rows"]
        finally:
            pb.pilc_set_timing(False)
        times.append(1e3 * min(took))
    print("a pixel a lane: %.1f us, 16: %.1f us" % tuple(times))
    assert times[0] < 0.66 * times[1]
