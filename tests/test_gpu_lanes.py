"""The thread-per-lane kernels where they can go wrong: the decoder's guess of a symbol over the whole range of scales,
means and precisions, and chunks of pixels in arrays that are not aligned."""
import numpy as np
import pytest
import torch

from oracle import pilc_oracle as orc
from paper_2206_05279_amd import binding as pb
from paper_2206_05279_amd import synth

pytestmark = pytest.mark.gpu

from gpu_util import DeviceWorkload, first_difference  # noqa: E402


@pytest.fixture(autouse=True)
def thread_per_lane():
    pb.pilc_set_kernel_policy(1)
    yield
    pb.pilc_set_kernel_policy(0)


def _check(wl, device):
    rc, want = orc.encode(orc.make_geom(*wl.geom), wl.img, wl.mu, wl.log_scale, wl.chan_coef)
    assert rc == orc.OK
    _, nbytes = device.encode()
    got = device.coded_numpy()
    assert nbytes == want.size and np.array_equal(got, want), first_difference(got, want)
    assert device.decode() == pb.PILC_OK
    assert np.array_equal(device.decoded_numpy(), wl.img)


# Scales from the smallest to the largest that the format has (beyond both clamps at the ends); every
# value of a pixel under means at, near and far from it, at both ends of the range of values.
@pytest.mark.parametrize("prec_bits", [10, 12, 13, 16])
@pytest.mark.parametrize("log_scale", [-32768, -16384, -9000, 0, 8192, 12288, 20000, 24575, 32767])
def test_guess_over_the_range_of_the_law(prec_bits, log_scale):
    wl = synth.make_random_case(prec_bits, 6, 16, 48, prec_bits, 0, 16, wild=True)
    rng = np.random.default_rng(log_scale & 0xFFFF)
    wl.img[...] = np.arange(wl.img.size, dtype=np.uint32).reshape(wl.img.shape) % 256
    near = np.clip(wl.img * 256.0 + rng.normal(0, 700, wl.img.shape), 0, 65535)
    far = rng.choice([0, 1, 128, 32768, 65407, 65535], size=wl.img.shape)
    wl.mu[...] = np.where(rng.random(wl.img.shape) < 0.7, near, far).astype(np.uint16)
    wl.log_scale[...] = log_scale
    _check(wl, DeviceWorkload(wl))


# The same with more lanes than one wavefront a SIMD takes, where the decoder looks at one neighbour of the guessed edge (in
# rows of more than 32 pixels that do not align: with more than two take): all scales in one batch, chunks of single elements, of aligned eights and of pairs.
@pytest.mark.parametrize("prec_bits", [10, 13, 16])
@pytest.mark.parametrize("lane,rows,mode", [(3, 16, 0), (8, 16, 0), (16, 16, 0), (3, 16, 1), (35, 16, 0), (35, 32, 0)])
def test_guess_with_many_lanes(prec_bits, lane, rows, mode):
    n, h, w = 9, rows * lane, 512
    wl = synth.make_random_case(prec_bits, n, h, w, prec_bits, mode, 1 if mode else lane, lane, wild=True)
    assert n * h * w // lane > 4096 * rows
    rng = np.random.default_rng(lane)
    wl.img[...] = np.arange(wl.img.size, dtype=np.uint32).reshape(wl.img.shape) % 256
    near = np.clip(wl.img * 256.0 + rng.normal(0, 700, wl.img.shape), 0, 65535)
    far = rng.choice([0, 1, 128, 32768, 65407, 65535], size=wl.img.shape)
    wl.mu[...] = np.where(rng.random(wl.img.shape) < 0.7, near, far).astype(np.uint16)
    scales = np.array([-32768, -16384, -9000, 0, 8192, 12288, 20000, 24575, 32767], dtype=np.int16)
    wl.log_scale[...] = scales[:, None, None, None]
    _check(wl, DeviceWorkload(wl))


# Rows of lanes shorter and longer than a chunk of eight pixels, arrays that start on any element: the last chunk of
# the last row of the last image is the one that must not be read past.
@pytest.mark.parametrize("w", [1, 7, 8, 9, 15, 17, 24])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_chunks_of_unaligned_rows(w, shift):
    wl = synth.make_random_case(w, 3, 5, w, 12, 1, 2, 17)
    device = DeviceWorkload(wl)

    def moved(t):
        room = torch.empty(t.numel() + shift, dtype=t.dtype, device=t.device)
        room[shift:] = t.reshape(-1)
        return room[shift:].reshape(t.shape)

    device.img, device.mu, device.log_scale = moved(device.img), moved(device.mu), moved(device.log_scale)
    device.out = moved(device.out)
    _check(wl, device)


# Wide laws at the lowest precision, where the guess of one lane or other of a wavefront misses on nearly every symbol: going
# on from it takes a third more time than guesses that are all good (starting over with a search took two and a half times theirs).
@pytest.mark.parametrize("log_scale", [4.0, 4.6])
def test_wide_laws_decode_without_a_search(log_scale):
    n, h, w = 8, 512, 1024
    rng = np.random.default_rng(int(10 * log_scale))
    times = []
    for ls in (2.0, log_scale):
        wl = synth.make_random_case(4, 1, 8, 8, 10, 1, 16, 16)
        wl.n, wl.h, wl.w = n, h, w
        wl.img = rng.integers(0, 256, size=(n, h, w, 3), dtype=np.uint8)
        spread = rng.logistic(0.0, np.exp(ls), size=wl.img.shape)
        wl.mu = np.clip((wl.img + spread) * 256.0, 0, 65535).astype(np.uint16)
        wl.log_scale = np.full(wl.img.shape, int(ls * 4096), dtype=np.int16)
        wl.chan_coef = np.zeros((n, 3), dtype=np.int16)
        d = DeviceWorkload(wl)
        d.encode()
        took = []
        pb.pilc_set_timing(True)
        try:
            for _ in range(9):
                assert d.decode() == pb.PILC_OK
                took.append(dict(pb.pilc_last_timing())["k_decode_lanes"])
        finally:
            pb.pilc_set_timing(False)
        assert torch.equal(d.out, d.img)
        times.append(min(took))
    print("log-scale %.1f: %.0f us, 2.0: %.0f us" % (log_scale, 1e3 * times[1], 1e3 * times[0]))
    assert times[1] < 1.8 * times[0]


# The division of the encoder's step under masses of 1 up to the largest, at the precisions where quotients are smallest and
# largest (test_division_arithmetic.py has every mass).  With the narrowest law and the mean on the pixel a symbol has nearly all of the mass, off it a single count.
@pytest.mark.parametrize("prec_bits", [10, 11, 12, 16])
def test_division_from_the_smallest_to_the_largest_mass(prec_bits):
    wl = synth.make_random_case(prec_bits, 4, 32, 40, prec_bits, 0, 320)
    rng = np.random.default_rng(prec_bits)
    wl.mu[...] = np.clip(wl.img * 256.0 + 256 * rng.choice([0, 0, 0, 1, -1, 2, 9], size=wl.img.shape), 0, 65535).astype(np.uint16)
    wl.log_scale[...] = rng.integers(-16384, 24576, size=wl.img.shape).astype(np.int16)
    wl.log_scale[0] = -16384
    wl.log_scale[1] = 24575
    wl.chan_coef[...] = 0
    _check(wl, DeviceWorkload(wl))


# The longest lane that the thread-per-lane encoder takes, and one that is a pixel longer, which the block encoder takes whatever
# the policy says.  Every symbol has a mass of 1 and costs a word of 16 bits, so that the words' 32-bit places are used up to their end.
@pytest.mark.parametrize("pixels,policies,kernel", [
    ((2**25 - 1) // 3, (1,), "k_encode_lanes"), ((2**25 - 1) // 3 + 1, (1, 3), "k_encode_block")])
def test_longest_lane_thread_per_lane(pixels, policies, kernel):
    wl = synth.make_random_case(5, 1, 8, 8, 16, 0, 64)
    wl.h, wl.w, wl.lane_a = 1, pixels, pixels
    wl.img = np.random.default_rng(5).integers(100, 250, size=(1, 1, pixels, 3), dtype=np.uint8)
    wl.mu = np.zeros(wl.img.shape, dtype=np.uint16)
    wl.log_scale = np.full(wl.img.shape, -16384, dtype=np.int16)
    wl.chan_coef[...] = 0
    rc, want = orc.encode(orc.make_geom(*wl.geom), wl.img, wl.mu, wl.log_scale, wl.chan_coef)
    assert rc == orc.OK and want.size > 6 * pixels
    device = DeviceWorkload(wl)
    pb.pilc_set_timing(True)
    try:
        for policy in policies:
            pb.pilc_set_kernel_policy(policy)
            device.coded.zero_()
            device.encode()
            assert kernel in [name for name, _ in pb.pilc_last_timing()]
            got = device.coded_numpy()
            assert got.size == want.size and np.array_equal(got, want), first_difference(got, want)
    finally:
        pb.pilc_set_timing(False)
