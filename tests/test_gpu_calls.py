"""What a call of pilc_encode or pilc_decode says of itself: its own outcome, whatever other calls do at the same time and
wherever the outcome is kept (a place in pinned host memory, the workspace where none is free or wanted)."""
import os
import subprocess
import sys
import threading
import time

import numpy as np
import pytest
import torch

from oracle import pilc_oracle as orc
from paper_2206_05279_amd import binding as pb
from paper_2206_05279_amd import synth

pytestmark = pytest.mark.gpu

from gpu_util import DeviceWorkload  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# A thread captures a graph, which makes the runtime refuse another thread's wait for its stream: that call fails while its
# kernels (here the decoding of a damaged container) are still queued.  The next call's outcome must not be theirs.
_REFUSED_CALL = """
import sys, threading, time
sys.path[:0] = [%r, %r]
import torch
from paper_2206_05279_amd import binding as pb, synth
from gpu_util import DeviceWorkload

good, bad = (DeviceWorkload(synth.make_random_case(1, 4, 16, 16, 12, 0, 16)) for _ in range(2))
for d in (good, bad):
    d.encode()
    assert d.decode() == pb.PILC_OK
damaged = bad.coded.clone()
damaged[-40 - (bad.coded.numel() - bad.nbytes):] ^= 0x55
torch.cuda._sleep(1)
torch.cuda.synchronize()
since = time.perf_counter()
torch.cuda._sleep(1 << 24)
torch.cuda.synchronize()
a_second = int((1 << 24) / (time.perf_counter() - since))

def decode(d, coded, stream):
    return pb.pilc_decode(d.geom, coded, d.nbytes, d.mu, d.log_scale, d.chan_coef, d.workspace, d.out,
                          stream=stream, check=False)

first, second, side = (torch.cuda.Stream() for _ in range(3))
x = torch.zeros(64, device="cuda:0")
x.add_(1.0)
torch.cuda.synchronize()
with torch.cuda.stream(first):
    torch.cuda._sleep(a_second // 4)
with torch.cuda.stream(second):
    torch.cuda._sleep(a_second // 2)
refused = []
graph = torch.cuda.CUDAGraph()
try:
    with torch.cuda.graph(graph, stream=side):
        x.add_(1.0)
        t = threading.Thread(target=lambda: refused.append(decode(bad, damaged, first)))
        t.start()
        t.join()
        x.add_(1.0)
except Exception as e:
    print("the capture failed:", str(e)[:60])
print("refused call:", refused, "next call:", decode(good, good.coded, second))
print("damaged container:", decode(bad, damaged, first))
assert refused == [pb.PILC_E_HIP]
sys.stdout.flush()
import os
os._exit(0)
"""


def test_refused_call_leaves_nothing_to_the_next_one():
    run = subprocess.run([sys.executable, "-c", _REFUSED_CALL % (ROOT, os.path.join(ROOT, "tests"))], cwd=ROOT,
                         capture_output=True, text=True, timeout=100)
    print(run.stdout, run.stderr[-2000:])
    assert run.returncode == 0
    assert "next call: 0" in run.stdout and "damaged container: %d" % pb.PILC_E_CORRUPT in run.stdout


def _busy(stream, seconds):
    """Keeps the stream busy for about that long."""
    torch.cuda.synchronize()
    since = time.perf_counter()
    torch.cuda._sleep(1 << 24)
    torch.cuda.synchronize()
    per_second = (1 << 24) / (time.perf_counter() - since)
    with torch.cuda.stream(stream):
        torch.cuda._sleep(int(seconds * per_second))


class _Calls:
    """Calls that end well and calls that fail, with what each has to say."""

    def __init__(self, seed, policy_lanes):
        # few long lanes, or a lane a thread
        wl = synth.make_random_case(seed, 6, 16, 24, 12, 0, 24) if policy_lanes else synth.make_random_case(seed, 2, 32, 32, 14, 0, 512)
        rc, self.want = orc.encode(orc.make_geom(*wl.geom), wl.img, wl.mu, wl.log_scale, wl.chan_coef)
        assert rc == orc.OK
        self.d = DeviceWorkload(wl)
        self.stream = torch.cuda.Stream()
        self.good = torch.zeros_like(self.d.coded)
        self.good[:self.want.size] = torch.from_numpy(self.want).to("cuda:0")
        self.damaged = self.good.clone()
        self.damaged[self.want.size - 40:self.want.size] ^= 0x55
        self.other = self.good.clone()
        self.other[8:12] = 0  # another batch's header
        self.room = 64 + 4 * (orc.lane_count(orc.make_geom(*wl.geom)) + 1) + 64  # header, offsets and a little more
        torch.cuda.synchronize()

    def encode(self, capacity):
        d = self.d
        return pb.pilc_encode(d.geom, d.img, d.mu, d.log_scale, d.chan_coef, d.workspace, d.coded[:capacity], stream=self.stream, check=False)

    def decode(self, coded):
        d = self.d
        return pb.pilc_decode(d.geom, coded, self.want.size, d.mu, d.log_scale, d.chan_coef, d.workspace, d.out, stream=self.stream, check=False)

    def calls(self):
        """Calls, each with what it has to say."""
        return [(lambda: self.encode(self.d.coded.numel()), (pb.PILC_OK, self.want.size)),
                (lambda: self.decode(self.damaged), pb.PILC_E_CORRUPT),
                (lambda: self.encode(self.room)[0], pb.PILC_E_CAPACITY),
                (lambda: self.decode(self.good), pb.PILC_OK),
                (lambda: self.decode(self.other), pb.PILC_E_FORMAT)]


def _in_threads(jobs):
    """Runs the jobs at the same time and returns what they returned."""
    out = [None] * len(jobs)
    gate = threading.Barrier(len(jobs))

    def run(i):
        gate.wait()
        out[i] = jobs[i]()

    threads = [threading.Thread(target=run, args=(i,)) for i in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    return out


def test_calls_at_once_each_with_their_own_outcome():
    def rounds(c):
        for _ in range(20):
            for call, due in c.calls():
                assert call() == due
        return True

    many = [_Calls(20 + i, i % 2) for i in range(8)]
    assert _in_threads([lambda c=c: rounds(c) for c in many]) == [True] * 8


def test_more_calls_at_once_than_places():
    waiting = [_Calls(40, i % 2) for i in range(64)]
    late = [_Calls(60, i // 5 % 2) for i in range(10)]  # a buffer and a stream for each call of two rounds
    gate = torch.cuda.Stream()
    _busy(gate, 1.5)
    opened = torch.cuda.Event()
    opened.record(gate)
    for c in waiting + late:
        c.stream.wait_event(opened)

    def later(call):
        time.sleep(0.3)  # by now the others hold every place and wait for their streams
        return not opened.query() and call()

    jobs = [(lambda c=c: c.decode(c.good), pb.PILC_OK) if i % 3 else (lambda c=c: c.decode(c.damaged), pb.PILC_E_CORRUPT)
            for i, c in enumerate(waiting)]
    for i, c in enumerate(late):
        call, due = c.calls()[i % 5]
        jobs.append((lambda call=call: later(call), due))
    assert _in_threads([job for job, _ in jobs]) == [due for _, due in jobs]


@pytest.mark.parametrize("policy", [0, 1, 3])
def test_static_encode_says_what_does_not_fit(policy):
    c = _Calls(80, 1)
    d = c.d
    pb.pilc_set_kernel_policy(policy)
    try:
        for capacity, due in ((c.room, pb.PILC_E_CAPACITY), (d.coded.numel(), pb.PILC_OK), (c.want.size - 1, pb.PILC_E_CAPACITY)):
            rc, nbytes = pb.pilc_encode_static(d.geom, d.img, d.mu, d.log_scale, d.chan_coef, d.coded[:capacity], check=False)
            assert rc == due
            if due == pb.PILC_OK:
                assert nbytes == c.want.size and np.array_equal(d.coded[:nbytes].cpu().numpy(), c.want)
    finally:
        pb.pilc_set_kernel_policy(0)


@pytest.mark.parametrize("policy", [1, 2])
@pytest.mark.parametrize("lanes", [1, 2, 255, 257, 2047, 2049, 8191, 8192, 8193])
def test_packers_without_a_scan(lanes, policy):
    """Up to 8192 lanes the packers sum the lanes' bytes themselves, write the header and say what does not fit."""
    wl = synth.make_random_case(lanes, lanes, 1, 9, 12, 0, 9)
    rc, want = orc.encode(orc.make_geom(*wl.geom), wl.img, wl.mu, wl.log_scale, wl.chan_coef)
    assert rc == orc.OK
    d = DeviceWorkload(wl)

    def encode(capacity):
        return pb.pilc_encode(d.geom, d.img, d.mu, d.log_scale, d.chan_coef, d.workspace, d.coded[:capacity], check=False)
    pb.pilc_set_kernel_policy(policy)
    try:
        for capacity in (d.coded.numel(), want.size):
            d.coded.fill_(0x5A)
            rc, nbytes = encode(capacity)
            assert rc == pb.PILC_OK and nbytes == want.size
            assert np.array_equal(d.coded[:nbytes].cpu().numpy(), want) and bool((d.coded[nbytes:] == 0x5A).all())
        d.coded.fill_(0x5A)
        assert encode(want.size - 1)[0] == pb.PILC_E_CAPACITY
        assert bool((d.coded[64 + 4 * (lanes + 1):] == 0x5A).all())
    finally:
        pb.pilc_set_kernel_policy(0)


@pytest.mark.parametrize("lanes", [4096, 4097])
def test_packers_of_long_lanes_have_a_scan(lanes):
    """With a workgroup of the packer for every lane, 4096 lanes are the most whose counts every workgroup sums."""
    wl = synth.make_random_case(lanes, lanes, 1, 2731, 12, 0, 2731)
    rc, want = orc.encode(orc.make_geom(*wl.geom), wl.img, wl.mu, wl.log_scale, wl.chan_coef)
    assert rc == orc.OK
    d = DeviceWorkload(wl)
    pb.pilc_set_timing(True)
    try:
        rc, nbytes = d.encode()
        names = [name for name, _ in pb.pilc_last_timing()]
    finally:
        pb.pilc_set_timing(False)
    assert ("scan" in names) == (lanes > 4096), names
    assert nbytes == want.size and np.array_equal(d.coded[:nbytes].cpu().numpy(), want)
