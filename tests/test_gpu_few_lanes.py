"""The few-lane kernels: a lane whose words do not fit 32 bits of bytes from the first one (2^27 symbols and more), and
the numbers of lanes up to which they are taken."""
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
