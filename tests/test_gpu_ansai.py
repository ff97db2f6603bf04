"""GPU parity of the table-driven coder (Sec. 3.2 Algs. 3-4) against the CPU reference: the
tables entry by entry, the container byte for byte, the decoded symbols, and the error codes,
through the C ABI, on shapes that span several wavefronts, ragged rows and every table path."""
import struct

import numpy as np
import pytest
import torch

from oracle import ansai_oracle as ao
from paper_2206_05279_amd import binding as pb
from paper_2206_05279_amd import synth_pieces as sp

pytestmark = pytest.mark.gpu

from gpu_util import DevicePieces, first_difference  # noqa: E402


def _logistic(m, d, x=256):
    return lambda rng: sp.logistic_masses(m, d, x)


def _random(m, d, x, conc=0.3):
    return lambda rng: sp.random_masses(rng, m, d, x, conc)


# name, M, masses, pieces, count, uniform symbols
CASES = [
    ("one symbol", 12, _logistic(12, 8), 1, 1, False),
    ("one wavefront", 12, _logistic(12, 8), 64, 64, False),
    ("ragged pieces and rows", 12, _logistic(12, 8), 65, 1000, False),
    ("odd count", 10, _logistic(10, 3), 130, 257, False),
    ("short rows", 12, _logistic(12, 8), 7, 33, False),
    ("count 1, many pieces", 12, _logistic(12, 8), 300, 1, False),
    ("count 3", 12, _logistic(12, 8), 129, 3, False),
    ("M15 tables in global memory", 15, _logistic(15, 2), 200, 999, False),
    ("M13 wide entries in LDS", 13, _logistic(13, 1), 100, 500, False),
    ("5 symbols", 6, _random(6, 3, 5), 96, 700, False),
    ("M1 two symbols", 1, lambda rng: np.array([[1, 1]], dtype=np.uint32), 50, 300, False),
    ("peaky masses", 11, _random(11, 4, 40, 0.05), 128, 1000, False),
    ("model does not fit", 12, _logistic(12, 8), 70, 640, True),
    ("40 distributions, encode tables in global memory", 9, _random(9, 40, 256, 1.0), 70, 200, False),
    ("255 distributions", 8, _random(8, 255, 256, 1.0), 64, 100, False),
    ("4096 pieces of 1000", 12, _logistic(12, 8), 4096, 1000, False),
    ("M14 random", 14, _random(14, 2, 256, 1.0), 77, 130, False),
    # between one wavefront per SIMD and a full workgroup: seven wavefronts per decode workgroup
    ("100,000 short pieces", 12, _logistic(12, 8), 100000, 24, False),
    # the stream of vector indices (Sec. 3.1): one static law, 16x16 indices per 32x32 image, K = 256
    ("vector-index stream", 12, lambda rng: sp.index_stream_masses(12), 3000, 256, False),
]


@pytest.fixture(params=range(len(CASES)), ids=[c[0] for c in CASES], scope="module")
def case(request):
    name, m, make, pieces, count, uniform = CASES[request.param]
    rng = np.random.default_rng(500 + request.param)
    mass = make(rng)
    sym, dist = sp.draw_pieces(mass, m, pieces, count, seed=900 + request.param, uniform_sym=uniform, threads=1)
    print("case", name, "M", m, "D,X", mass.shape, "pieces", pieces, "count", count, flush=True)
    dp = DevicePieces(m, mass, sym, dist)
    return dp


def test_tables_match_the_reference(case):
    dp = case
    got = dp.table_views()
    ref = ao.build_tables(dp.m, dp.mass_np)
    for name, g, r in zip(("delta", "phi", "theta", "nbits", "next"), got, ref):
        assert np.array_equal(g.astype(np.int64), r.astype(np.int64)), name


def test_container_is_byte_identical(case):
    dp = case
    rc, ref = ao.encode(dp.m, dp.mass_np, dp.sym_np, dp.dist_np)
    assert rc == ao.OK
    dp.encode()
    got = dp.coded_numpy()
    assert got.size == ref.size and np.array_equal(got, ref), first_difference(got, ref)


def test_decode_returns_the_symbols(case):
    dp = case
    dp.encode()
    dp.decode()
    assert np.array_equal(dp.decoded_numpy(), dp.sym_np)
    # and a container made by the reference decodes the same way
    rc, ref = ao.encode(dp.m, dp.mass_np, dp.sym_np, dp.dist_np)
    buf = torch.zeros(ref.size + 16, dtype=torch.uint8, device="cuda:0")
    buf[: ref.size] = torch.from_numpy(ref).cuda()
    dp.decode(coded=buf, nbytes=ref.size)
    assert np.array_equal(dp.decoded_numpy(), dp.sym_np)


@pytest.mark.parametrize("m,d", [(12, 8), (15, 2), (13, 1)], ids=["M12", "M15", "M13"])
@pytest.mark.parametrize("count", [1, 2, 7, 8, 9, 31, 32, 33, 40, 63, 64, 65, 95, 127, 128, 129, 136, 255, 300])
def test_rows_of_every_length_decode(count, m, d):
    """Row lengths around the eight symbols of a group, the 32 that pass through LDS together and the 128
    that are fetched together, at every alignment of the rows; symbols drawn uniformly, so that the rare
    ones with the longest codes come as often as the others; arrays of fewer than 16 bytes among them."""
    mass = sp.logistic_masses(m, d)
    for pieces in (1, 3, 67, 200):
        print("M", m, "D", d, "count", count, "pieces", pieces, flush=True)
        sym, dist = sp.draw_pieces(mass, m, pieces, count, seed=count + pieces, uniform_sym=True, threads=1)
        dp = DevicePieces(m, mass, sym, dist)
        rc, ref = ao.encode(m, mass, sym, dist)
        assert rc == ao.OK
        buf = torch.zeros(ref.size + 16, dtype=torch.uint8, device="cuda:0")
        buf[: ref.size] = torch.from_numpy(ref).cuda()
        dp.decode(coded=buf, nbytes=ref.size)
        assert np.array_equal(dp.decoded_numpy(), sym)


@pytest.mark.parametrize("m,d", [(9, 90), (9, 91), (9, 94), (9, 95), (11, 23), (11, 24)])
def test_tables_that_just_fit_beside_the_rows(m, d):
    """Decode tables around the size up to which they are kept in LDS: the most laws that leave room for four
    wavefronts' rows, the least and the most that leave room for three, and one law more, whose tables stay
    in global memory; as many wavefronts as the library likes, one, and as many as fit."""
    mass = sp.logistic_masses(m, d)
    sym, dist = sp.draw_pieces(mass, m, 900, 77, seed=d, uniform_sym=True, threads=1)
    dp = DevicePieces(m, mass, sym, dist)
    rc, ref = ao.encode(m, mass, sym, dist)
    assert rc == ao.OK
    buf = torch.zeros(ref.size + 16, dtype=torch.uint8, device="cuda:0")
    buf[: ref.size] = torch.from_numpy(ref).cuda()
    try:
        for waves in (0, 1, 12):
            print("M", m, "D", d, "waves", waves, flush=True)
            pb.pilc_set_ansai_decode_waves(waves)
            dp.decode(coded=buf, nbytes=ref.size)
            assert np.array_equal(dp.decoded_numpy(), sym)
    finally:
        pb.pilc_set_ansai_decode_waves(0)


@pytest.mark.parametrize("m,d,count,pieces", [(12, 8, 641, 209_500), (10, 3, 1001, 134_150), (13, 1, 4001, 33_601), (15, 2, 1000, 134_300),
                                              (15, 1, 20_003, 6_713), (12, 8, 640, 209_800), (12, 8, 639, 210_100)])
def test_long_rows_of_a_large_batch_decode(m, d, count, pieces):
    """Rows of 640 symbols and more in a batch of 2^27 and more are cut at the array's lines: every alignment of the
    rows, tables in LDS and in global memory, a last wavefront that is not full; and on the other side of the
    line, rows of whole half lines and rows of 639.  Symbols drawn uniformly, by the library's encoder
    (compared with the reference in the cases above)."""
    print("M", m, "D", d, "count", count, "pieces", pieces, flush=True)
    assert pieces * count >= 1 << 27
    rng = np.random.default_rng(count)
    sym = rng.integers(0, 256, (pieces, count), dtype=np.uint8)
    dist = rng.integers(0, d, (pieces, count), dtype=np.uint8)
    dp = DevicePieces(m, sp.logistic_masses(m, d), sym, dist)
    dp.encode()
    dp.decode()
    assert torch.equal(dp.out, dp.sym)


def test_every_workgroup_shape_of_the_decoder_gives_the_same_symbols():
    """One input through workgroups of 1 .. 12 wavefronts (as many as fit beside the tables), for
    tables in LDS with 16-bit and with 32-bit entries and for tables in global memory."""
    for m, d, pieces, count in ((12, 8, 2000, 300), (13, 1, 1500, 200), (15, 2, 1500, 200)):
        mass = sp.logistic_masses(m, d)
        sym, dist = sp.draw_pieces(mass, m, pieces, count, seed=77 + m, threads=1)
        dp = DevicePieces(m, mass, sym, dist)
        rc, ref = ao.encode(m, mass, sym, dist)
        assert rc == ao.OK
        dp.encode()
        assert np.array_equal(dp.coded_numpy(), ref)
        try:
            for waves in range(1, 13):
                print("M", m, "D", d, "wavefronts per workgroup", waves, flush=True)
                pb.pilc_set_ansai_decode_waves(waves)
                dp.decode()
                assert np.array_equal(dp.decoded_numpy(), sym), waves
        finally:
            pb.pilc_set_ansai_decode_waves(0)
    with pytest.raises(pb.PilcError):
        pb.pilc_set_ansai_decode_waves(13)


# ---------------------------------------------------------------- errors
@pytest.fixture(scope="module")
def small():
    m, mass = 10, sp.logistic_masses(10, 4)
    sym, dist = sp.draw_pieces(mass, m, 70, 100, seed=3, threads=1)
    return DevicePieces(m, mass, sym, dist)


def test_capacity_and_workspace(small):
    dp = small
    _, nbytes = dp.encode()
    assert dp.max_coded == ao.max_coded_bytes(70, 100, 10)
    rc, _ = dp.encode(check=False, capacity=((nbytes - 1) // 16) * 16)
    assert rc == pb.PILC_E_CAPACITY
    rc, _ = dp.encode(check=False, capacity=64)
    assert rc == pb.PILC_E_CAPACITY
    rc, n2 = dp.encode(check=False, capacity=nbytes)
    assert rc == pb.PILC_OK and n2 == nbytes
    ws = dp.workspace
    dp.workspace = ws[: ws.numel() - 256]
    try:
        assert dp.encode(check=False)[0] == pb.PILC_E_WORKSPACE
        assert dp.decode(check=False) == pb.PILC_E_WORKSPACE
    finally:
        dp.workspace = ws


def test_bad_arguments(small):
    dp = small
    dp.encode()
    good = dp.shape
    for field, value in (("pieces", 0), ("count", 0), ("prec_bits", 0), ("prec_bits", 16), ("num_dist", 0),
                         ("num_dist", 256), ("num_sym", 1), ("num_sym", 257)):
        shape = pb.make_ansai_shape(good.pieces, good.count, good.prec_bits, good.num_dist, good.num_sym)
        setattr(shape, field, value)
        dp.shape = shape
        try:
            assert dp.encode(check=False)[0] == pb.PILC_E_ARG, field
            assert dp.decode(check=False) == pb.PILC_E_ARG, field
        finally:
            dp.shape = good
    assert pb.pilc_ansai_table_bytes(3, 1, 256) == 0           # 2^M below the alphabet size
    # misaligned arrays
    pad = torch.zeros(dp.sym.numel() + 16, dtype=torch.uint8, device="cuda:0")
    off1 = pad[1: 1 + dp.sym.numel()].view(dp.sym.shape)
    assert dp.encode(check=False, sym=off1)[0] == pb.PILC_E_ARG
    assert dp.decode(check=False, dist=off1) == pb.PILC_E_ARG
    # a shape the tables were not built for
    other = pb.make_ansai_shape(good.pieces, good.count, good.prec_bits, good.num_dist - 1, good.num_sym)
    dp.shape = other
    try:
        assert dp.encode(check=False)[0] == pb.PILC_E_ARG
    finally:
        dp.shape = good
    big = pb.make_ansai_shape(1 << 24, 1 << 10, 12, 8, 256)
    with pytest.raises(pb.PilcError) as e:
        pb.pilc_ansai_workspace_size(big)
    assert e.value.code == pb.PILC_E_TOO_LARGE


def test_bad_masses_and_indices(small):
    dp = small
    mass = dp.mass_np.copy()
    mass[1, 7] += 1                                            # a row that does not sum to 2^M
    bad = DevicePieces(dp.m, mass, dp.sym_np, dp.dist_np, build=False)
    rc = pb.pilc_ansai_build_tables(bad.m, bad.d, bad.x, bad.mass, bad.tables, check=False)
    assert rc == pb.PILC_E_ARG
    assert bad.encode(check=False)[0] == pb.PILC_E_ARG         # the blob is marked unusable
    mass = dp.mass_np.copy()
    mass[2, 0] += mass[2, 1]
    mass[2, 1] = 0                                             # an empty symbol
    bad = DevicePieces(dp.m, mass, dp.sym_np, dp.dist_np, build=False)
    assert pb.pilc_ansai_build_tables(bad.m, bad.d, bad.x, bad.mass, bad.tables, check=False) == pb.PILC_E_ARG
    # an index beyond D in the data
    dist = dp.dist_np.copy()
    dist[69, 99] = 4
    assert ao.encode(dp.m, dp.mass_np, dp.sym_np, dist)[0] == ao.E_ARG
    assert dp.encode(check=False, dist=torch.from_numpy(dist).cuda())[0] == pb.PILC_E_ARG
    dp.encode()
    assert dp.decode(check=False, dist=torch.from_numpy(dist).cuda()) in (pb.PILC_E_ARG, pb.PILC_E_CORRUPT)
    # a symbol beyond X
    m, mass = 6, sp.random_masses(np.random.default_rng(1), 6, 2, 5)
    sym, dist = sp.draw_pieces(mass, m, 10, 50, seed=4, threads=1)
    sym[3, 3] = 5
    assert ao.encode(m, mass, sym, dist)[0] == ao.E_ARG
    assert DevicePieces(m, mass, sym, dist).encode(check=False)[0] == pb.PILC_E_ARG


def _damaged(dp, coded, edit):
    c = coded.copy()
    edit(c)
    rc_ref, back_ref = ao.decode(dp.m, dp.mass_np, dp.dist_np, c)
    buf = torch.zeros(c.size + 16, dtype=torch.uint8, device="cuda:0")
    buf[: c.size] = torch.from_numpy(c).cuda()
    rc = dp.decode(coded=buf, nbytes=c.size, check=False)
    return rc_ref, back_ref, rc, dp.decoded_numpy()


def test_damaged_containers_agree_with_the_reference(small):
    dp = small
    dp.encode()
    coded = dp.coded_numpy()
    pieces = dp.shape.pieces
    offs = np.frombuffer(coded.tobytes(), dtype="<u4", count=pieces + 1, offset=64)
    body = 64 + 4 * (pieces + 1)

    def put(at, value):
        def edit(c):
            c[at:at + 4] = np.frombuffer(struct.pack("<I", value), np.uint8)
        return edit

    def flip(at, mask):
        def edit(c):
            c[at] ^= mask
        return edit

    edits = {
        "magic": flip(0, 1),
        "pieces field": put(8, pieces + 1),
        "payload size": put(48, int(offs[-1]) + 4),
        "state below 2^M": put(body + int(offs[1]), 5),
        "state above 2^(M+1)": put(body + int(offs[65]), 3000),
        "bit count": flip(body + int(offs[2]) + 4, 0x40),
        "offset moved": put(64 + 4 * 66, int(offs[66]) + 4),
        "offset beyond payload": put(64 + 4 * 3, int(offs[-1]) + 8),
        "payload bit": flip(body + int(offs[3]) + 9, 0x10),
        "payload bit in last piece": flip(body + int(offs[69]) + 8, 0x01),
    }
    for name, edit in edits.items():
        rc_ref, back_ref, rc, back = _damaged(dp, coded, edit)
        want = {ao.OK: pb.PILC_OK, ao.E_FORMAT: pb.PILC_E_FORMAT, ao.E_CORRUPT: pb.PILC_E_CORRUPT}[rc_ref]
        assert rc == want, name
        if rc == pb.PILC_OK:
            assert np.array_equal(back, back_ref), name
    # truncation is a size mismatch
    assert dp.decode(nbytes=coded.size - 4, check=False) == pb.PILC_E_FORMAT
    assert dp.decode(nbytes=32, check=False) == pb.PILC_E_FORMAT


def test_timing_names(small):
    dp = small
    pb.pilc_set_timing(True)
    try:
        dp.encode()
        names = [n for n, _ in pb.pilc_last_timing()]
        assert names == ["total", "k_ansai_encode", "scan", "k_ansai_pack"]
        dp.decode()
        names = [n for n, _ in pb.pilc_last_timing()]
        assert names == ["total", "k_ansai_check_header", "k_ansai_decode"]
    finally:
        pb.pilc_set_timing(False)


def test_centering_matches_the_reference():
    rng = np.random.default_rng(5)
    for n in (1, 15, 16, 17, 4097, 1 << 20):
        r = rng.integers(0, 256, n, dtype=np.uint8)
        mu = rng.integers(0, 256, n, dtype=np.uint8)
        dr, dmu = torch.from_numpy(r).cuda(), torch.from_numpy(mu).cuda()
        out = torch.full_like(dr, 0x5A)
        pb.pilc_ansai_center(dr, dmu, out)
        assert np.array_equal(out.cpu().numpy(), ao.center(r, mu)), n
        back = torch.empty_like(dr)
        pb.pilc_ansai_center(out, dmu, back, inverse=True)
        assert np.array_equal(back.cpu().numpy(), r), n
        pb.pilc_ansai_center(out, dmu, out, inverse=True)                  # in place
        assert np.array_equal(out.cpu().numpy(), r), n
    pad = torch.zeros(64, dtype=torch.uint8, device="cuda:0")
    assert pb.pilc_ansai_center(pad[1:33], pad[:32], pad[32:], check=False) == pb.PILC_E_ARG


# Pieces of one wavefront whose words differ in number as much as they can (a law of one very likely symbol against one of
# equally likely ones), rows that end beside the edges of a line, of its quarters and of a block of words.
@pytest.mark.parametrize("pieces", [1, 63, 65, 130])
@pytest.mark.parametrize("count", [1, 4, 15, 16, 17, 31, 32, 33, 127, 128, 129, 255, 257, 640])
def test_pieces_of_very_different_lengths(pieces, count):
    m, x = 15, 200
    mass = np.ones((2, x), dtype=np.uint32)
    mass[0, 7] = (1 << m) - (x - 1)
    mass[1] = (1 << m) // x
    mass[1, 0] += (1 << m) - mass[1].sum()
    rng = np.random.default_rng(1000 * pieces + count)
    dist = np.broadcast_to((np.arange(pieces) % 3 == 0)[:, None], (pieces, count)).astype(np.uint8).copy()
    sym = np.where(dist == 0, 7, rng.integers(0, x, (pieces, count))).astype(np.uint8)
    sym[1::2] = np.where(rng.random(sym[1::2].shape) < 0.1, rng.integers(0, x, sym[1::2].shape), sym[1::2])
    rc, want = ao.encode(m, mass, sym, dist)
    assert rc == ao.OK
    dp = DevicePieces(m, mass, sym, dist)
    _, nbytes = dp.encode()
    got = dp.coded_numpy()
    assert nbytes == want.size and np.array_equal(got, want), first_difference(got, want)
    assert dp.decode() == pb.PILC_OK
    assert np.array_equal(dp.decoded_numpy(), sym)


# A last group of sixteen that is not full, of pieces with few and with many words, beside full ones and alone.
@pytest.mark.parametrize("pieces", [1, 2, 15, 17, 31, 33, 79, 81])
@pytest.mark.parametrize("count", [9, 40, 600, 1300])
def test_last_pieces_of_a_batch(pieces, count):
    m, x = 12, 256
    mass = np.full((1, x), (1 << m) // x, dtype=np.uint32)
    rng = np.random.default_rng(pieces * 10000 + count)
    sym = rng.integers(0, x, (pieces, count)).astype(np.uint8)
    dist = np.zeros((pieces, count), dtype=np.uint8)
    rc, want = ao.encode(m, mass, sym, dist)
    assert rc == ao.OK
    dp = DevicePieces(m, mass, sym, dist)
    _, nbytes = dp.encode()
    got = dp.coded_numpy()
    assert nbytes == want.size and np.array_equal(got, want), first_difference(got, want)


def _pack_time(m, mass, sym, dist):
    """Fastest of some launches of the packer, in microseconds; what was packed decodes."""
    dp = DevicePieces(m, mass, sym, dist)
    times = []
    pb.pilc_set_timing(True)
    try:
        for _ in range(5):
            dp.encode()
            times.append(1e3 * dict(pb.pilc_last_timing())["k_ansai_pack"])
    finally:
        pb.pilc_set_timing(False)
    assert dp.decode() == pb.PILC_OK
    assert np.array_equal(dp.decoded_numpy(), sym)
    return min(times)


# One piece in sixteen with a word or two beside pieces of a thousand words: the others of its group are not held up.
def test_short_pieces_beside_long_ones():
    m, pieces, count = 15, 8192, 4000
    mass = np.ones((2, 256), dtype=np.uint32)
    mass[0] = (1 << m) // 256
    mass[1, 7] = (1 << m) - 255
    rng = np.random.default_rng(11)
    took = []
    for short in (False, True):
        sym = rng.integers(0, 256, (pieces, count), dtype=np.uint8)
        dist = np.zeros((pieces, count), dtype=np.uint8)
        if short:
            dist[5::16] = 1
            sym[5::16] = 7
        took.append(_pack_time(m, mass, sym, dist))
    print("pack: %.0f us, with short pieces %.0f us" % tuple(took))
    assert took[1] < 2.0 * took[0]


# Pieces of four words, which are long enough for sixteen bytes a thread, take about what pieces of three words take.
def test_pieces_of_few_words():
    rng = np.random.default_rng(12)
    mass = np.full((1, 256), 16, dtype=np.uint32)
    took = []
    for count in (12, 16):
        sym = rng.integers(0, 256, (400000, count), dtype=np.uint8)
        took.append(_pack_time(12, mass, sym, np.zeros_like(sym)))
    print("pack: %.0f us for three words, %.0f us for four" % tuple(took))
    assert took[1] < 1.7 * took[0]
