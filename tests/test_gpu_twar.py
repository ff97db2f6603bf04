"""GPU parity of the Three-Way AR residual transform (Sec. 3.1 eqs. (2)-(4)) against the CPU
reference, through the C ABI: residuals and recovered images byte for byte, on shapes that
cover several images per wavefront, bands of 64 rows, tiles in LDS, and the kernel that decodes
along the diagonals with its bands together, one at a time and in several launches."""
import numpy as np
import pytest
import torch

from oracle import twar_oracle as to
from paper_2206_05279_amd import binding as pb

pytestmark = pytest.mark.gpu

ONE = 1 << 14
SHAPES = [(1, 1, 1), (3, 32, 32), (5, 7, 9), (2, 64, 64), (7, 16, 16), (2, 33, 5), (1, 100, 37),
          (1, 130, 300), (2, 3, 700), (513, 32, 32), (1, 200, 64),
          # taller than a wavefront: one row more than a band, two whole bands, 25 bands, a full-size frame
          (3, 65, 16), (2, 128, 48), (1, 1600, 32), (2, 1080, 1920),
          # bands that follow each other: 11, 33, 7 and 5 of them, the last with 60, 52, 1 and 1 rows; eight whole ones
          (2, 700, 64), (1, 2100, 160), (3, 385, 32), (3, 257, 32), (2, 512, 48),
          # many images, the bands of which go one at a time
          (256, 800, 16),
          # more groups of small images: eight images a group, rows of 27 dwords, an odd number of
          # groups, 17-row images (13 idle threads), many groups with a single-image group at the end
          (9, 8, 8), (40, 32, 36), (11, 64, 64), (100, 17, 16), (24577, 32, 32),
          # tiles copied a byte, 4 bytes or 16 bytes at a time (image sizes 105, 36 and 3960 bytes,
          # the last with 33-row images), each with many groups and a short last one
          (4001, 5, 7), (7001, 3, 4), (1300, 33, 40)]


def models(rng):
    yield "plane", [[-ONE, ONE, ONE], [ONE // 2, -ONE // 2, ONE], [ONE // 2, -ONE // 2, ONE]], [0, 0, 0]
    yield "random", rng.integers(-ONE, ONE + 1, (3, 3)).tolist(), rng.integers(-64 * ONE, 64 * ONE, 3).tolist()
    yield "extreme", [[32767] * 3, [-32768] * 3, [32767, -32768, 1]], [1 << 30, -(1 << 30), 12345]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_forward_and_inverse_match_the_reference(shape):
    rng = np.random.default_rng(sum(shape))
    img = rng.integers(0, 256, shape + (3,), dtype=np.uint8)
    if shape[1] >= 16:  # some structure, so that predictions matter
        img = (img // 8 + np.linspace(0, 200, shape[2]).astype(np.uint8)[None, None, :, None]).astype(np.uint8)
    d_img = torch.from_numpy(img).cuda()
    for name, wq, bq in models(rng):
        print("shape", shape, "model", name, flush=True)
        ref = to.forward(to.make_params(wq, bq), img)
        p = pb.make_twar_params(wq, bq)
        d_res = torch.full_like(d_img, 0x5A)
        pb.pilc_twar_forward(p, d_img, d_res)
        assert np.array_equal(d_res.cpu().numpy(), ref), name
        d_back = torch.full_like(d_img, 0xA5)
        pb.pilc_twar_inverse(p, d_res, d_back)
        assert np.array_equal(d_back.cpu().numpy(), img), name
        # and the reference's own inverse agrees on a residual that is not a forward image
        noise = rng.integers(0, 256, img.shape, dtype=np.uint8)
        d_noise = torch.from_numpy(noise).cuda()
        pb.pilc_twar_inverse(p, d_noise, d_back)
        assert np.array_equal(d_back.cpu().numpy(), to.inverse(to.make_params(wq, bq), noise)), name


def test_thirty_frames_come_back_every_time():
    """The workload bench.py times (30 frames of 1080 x 1920, 17 bands each, 510 workgroups that
    follow each other through words in global memory): the inverse of the forward transform is the
    image, on five calls in a row into a buffer poisoned before each, compared on the device.  A
    band that took a word of the band above before it was there would decode the rest of its rows wrongly."""
    g = torch.Generator().manual_seed(11)
    img = torch.randint(0, 256, (30, 1080, 1920, 3), dtype=torch.uint8, generator=g).cuda()
    p = pb.make_twar_params([[-ONE, ONE, ONE], [ONE // 2, -ONE // 2, ONE], [ONE // 2, -ONE // 2, ONE]], [0, 0, 0])
    res = torch.empty_like(img)
    back = torch.empty_like(img)
    pb.pilc_twar_forward(p, img, res)
    # two frames of the residual against the CPU reference
    assert np.array_equal(res[:2].cpu().numpy(), to.forward(to.make_params(
        [[-ONE, ONE, ONE], [ONE // 2, -ONE // 2, ONE], [ONE // 2, -ONE // 2, ONE]], [0, 0, 0]), img[:2].cpu().numpy()))
    for turn in range(5):
        back.fill_(0xA5 ^ turn)
        pb.pilc_twar_inverse(p, res, back)
        assert torch.equal(back, img), turn


def test_bands_give_up_a_wait_that_is_never_answered():
    """A band of a tall image waits for the last row of the band above.  With that row made to
    publish nothing (a switch that exists for this test) and a bound of 20 microseconds the band
    below must give up, every kernel must end, and the call must say PILC_E_TIMEOUT; the next
    ordinary call works."""
    rng = np.random.default_rng(5)
    img = rng.integers(0, 256, (2, 700, 64, 3), dtype=np.uint8)
    wq, bq = [[ONE // 2, ONE // 4, ONE // 4]] * 3, [0, 0, 0]
    p = pb.make_twar_params(wq, bq)
    d_res = torch.from_numpy(to.forward(to.make_params(wq, bq), img)).cuda()
    d_back = torch.zeros_like(d_res)
    try:
        pb.pilc_set_one_pass_wait(2000, True)
        assert pb.pilc_twar_inverse(p, d_res, d_back, check=False) == pb.PILC_E_TIMEOUT
    finally:
        pb.pilc_set_one_pass_wait(0, False)
    assert pb.pilc_twar_inverse(p, d_res, d_back, check=False) == pb.PILC_OK
    assert np.array_equal(d_back.cpu().numpy(), img)


# Rows of any width at any address, decoded along the anti-diagonals: one group of 64 rows and one row
# more, the most and one more than a band, several bands, images that share a group of rows, widths
# around the 16 columns of a block and the narrowest there are, photographs.
@pytest.mark.parametrize("offset", [0, 1, 7], ids=lambda o: "at%d" % o)
@pytest.mark.parametrize("shape", [(1, 65, 16), (2, 65, 17), (1, 128, 31), (3, 129, 33), (2, 300, 47), (1, 700, 85),
                                   (5, 20, 333), (3, 64, 97), (65, 1, 129), (2, 33, 1000), (2, 1365, 2047)],
                         ids=lambda s: "x".join(map(str, s)))
def test_any_width_at_any_address(shape, offset):
    print("shape", shape, "offset", offset, flush=True)
    rng = np.random.default_rng(sum(shape) + offset)
    noise = rng.integers(0, 256, shape + (3,), dtype=np.uint8)
    _, wq, bq = list(models(rng))[offset % 3]
    ref = to.inverse(to.make_params(wq, bq), noise)
    size = noise.size

    def at_offset(fill):
        whole = torch.full((size + 64,), fill, dtype=torch.uint8, device="cuda:0")
        return whole, whole[16 + offset:16 + offset + size].view(noise.shape)
    p = pb.make_twar_params(wq, bq)
    _, d_noise = at_offset(0x33)
    d_noise.copy_(torch.from_numpy(noise))
    whole_back, d_back = at_offset(0xA5)
    pb.pilc_twar_inverse(p, d_noise, d_back)
    assert np.array_equal(d_back.cpu().numpy(), ref)
    whole_res, d_res = at_offset(0x5A)
    pb.pilc_twar_forward(p, d_back, d_res)
    assert np.array_equal(d_res.cpu().numpy(), noise)
    # nothing beside either array has been written
    for whole, fill in ((whole_back, 0xA5), (whole_res, 0x5A)):
        assert bool((whole[:16 + offset] == fill).all()) and bool((whole[16 + offset + size:] == fill).all()), fill


# Images of more than 64 rows on either side of each line between tiles and diagonals (by how many there are and how
# wide); from 191 images of 150 rows on, bands of the diagonals in several shapes (their lines: test_lines_of_bands).
@pytest.mark.parametrize("offset", [0, 1], ids=lambda o: "at%d" % o)
@pytest.mark.parametrize("shape", [(256, 65, 24), (257, 97, 24), (257, 97, 28), (300, 65, 36), (300, 65, 40), (512, 97, 36),
                                   (513, 97, 36), (513, 97, 40), (768, 97, 84), (769, 97, 84), (769, 129, 27),
                                   (769, 129, 29), (769, 96, 39), (769, 96, 41), (1023, 70, 83), (1024, 70, 83),
                                   (1030, 65, 15), (191, 150, 64), (192, 150, 64), (40, 128, 191), (40, 128, 192),
                                   (127, 512, 64), (128, 512, 64), (128, 512, 192), (128, 770, 192), (111, 1000, 192)],
                         ids=lambda s: "x".join(map(str, s)))
def test_both_sides_of_every_line(shape, offset):
    print("shape", shape, "offset", offset, flush=True)
    rng = np.random.default_rng(sum(shape) + offset)
    noise = rng.integers(0, 256, shape + (3,), dtype=np.uint8)
    _, wq, bq = list(models(rng))[1 + offset]
    size = noise.size
    d_noise, d_back = (torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda:0") for _ in range(2))
    d_noise[16 + offset:16 + offset + size] = torch.from_numpy(noise.reshape(-1)).cuda()
    pb.pilc_twar_inverse(pb.make_twar_params(wq, bq), d_noise[16 + offset:16 + offset + size].view(noise.shape),
                         d_back[16 + offset:16 + offset + size].view(noise.shape))
    back = d_back.cpu().numpy()
    assert np.array_equal(back[16 + offset:16 + offset + size], to.inverse(to.make_params(wq, bq), noise).reshape(-1))
    assert (back[:16 + offset] == 0xA5).all() and (back[16 + offset + size:] == 0xA5).all()


@pytest.mark.parametrize("shape", [(70, 1080, 1920), (23, 150, 50000), (1, 4100, 65535), (6000, 129, 100), (250, 200, 2047),
                                   (190, 300, 3200)],
                         ids=lambda s: "x".join(map(str, s)))
def test_more_bands_than_one_launch_takes(shape):
    """More bands than there is room for the rows they pass on: several launches with all bands of an image, over
    the images (62 and 8 frames, 13 and 10 wide images), whose rows pass through the same words; for an image
    with more bands than that by itself, over its bands; and so many images that bands go one at a time, a
    launch each, or as many wide ones as make up a round of workgroups and more bands than a launch takes (and somewhat fewer, which
    go together)."""
    print("shape", shape, flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(3)
    img = torch.randint(0, 256, shape + (3,), dtype=torch.uint8, device="cuda:0", generator=g)
    p = pb.make_twar_params([[-ONE, ONE, ONE], [ONE // 2, -ONE // 2, ONE], [ONE // 2, -ONE // 2, ONE]], [0, 0, 0])
    res, back = torch.empty_like(img), torch.full_like(img, 0xA5)
    pb.pilc_twar_forward(p, img, res)
    pb.pilc_twar_inverse(p, res, back)
    assert torch.equal(back, img)


def test_more_calls_at_once_than_sets_of_words():
    """Eight threads with a stream each: the calls that find no set of words free go a band at a time."""
    import threading
    g = torch.Generator(device="cuda:0").manual_seed(4)
    img = torch.randint(0, 256, (2, 900, 1001, 3), dtype=torch.uint8, device="cuda:0", generator=g)
    p = pb.make_twar_params([[-ONE, ONE, ONE], [ONE // 2, -ONE // 2, ONE], [ONE // 2, -ONE // 2, ONE]], [0, 0, 0])
    res = torch.empty_like(img)
    pb.pilc_twar_forward(p, img, res)
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            back = torch.full_like(img, i)
            for _ in range(6):
                pb.pilc_twar_inverse(p, res, back, stream=stream)
                if not torch.equal(back, img):
                    wrong.append(i)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


# Either side of the lines of csrc/pilc_twar_rules.hpp that batches of up to some 130 MB reach: one at a time or together (two
# bands by strips and blocks, by how rounds are filled, long rows), then together with a compute unit each or two to one
# (eight bands by strips, by strips times blocks, seven bands, long rows of many and of two bands).  The last ones are odd sizes on
# no line.
LINES = [(255, 70, 64), (256, 70, 64), (384, 70, 240), (385, 70, 240), (513, 70, 641), (513, 70, 642), (512, 70, 642),
         (410, 130, 64), (411, 130, 64), (450, 193, 258), (451, 193, 258), (470, 129, 658), (471, 129, 658),
         (512, 193, 258), (513, 193, 258), (614, 193, 258), (615, 193, 258), (768, 193, 258), (769, 193, 258),
         (819, 449, 98), (820, 449, 98), (230, 200, 881), (230, 200, 882), (211, 70, 1681), (211, 70, 1682),
         (210, 70, 1682), (100, 450, 34), (101, 450, 34), (124, 450, 50), (125, 450, 50), (150, 450, 66),
         (151, 450, 66), (103, 450, 304), (104, 450, 304), (103, 448, 304), (119, 400, 66), (120, 400, 66),
         (20, 400, 65), (20, 400, 66), (20, 400, 209), (20, 400, 210), (96, 449, 689), (96, 449, 690), (95, 449, 690),
         (60, 321, 1009), (60, 321, 1010), (140, 200, 1010), (141, 200, 1010), (141, 200, 1009), (140, 130, 1682),
         (141, 130, 1682), (281, 70, 1521), (281, 70, 1522), (280, 70, 1522)]


@pytest.mark.parametrize("shape", LINES + [(383, 130, 64), (384, 130, 64), (384, 200, 161), (384, 200, 162), (143, 131, 161),
                                           (144, 131, 161), (132, 129, 176), (132, 129, 194), (20, 140, 945), (20, 140, 946),
                                           (1, 65, 1), (1, 127, 17), (1, 193, 33)], ids=lambda s: "x".join(map(str, s)))
def test_lines_of_bands(shape):
    print("shape", shape, flush=True)
    rng = np.random.default_rng(sum(shape))
    noise = rng.integers(0, 256, shape + (3,), dtype=np.uint8)
    _, wq, bq = list(models(rng))[1]
    d_back = torch.full(noise.shape, 0xA5, dtype=torch.uint8, device="cuda:0")
    pb.pilc_twar_inverse(pb.make_twar_params(wq, bq), torch.from_numpy(noise).cuda(), d_back)
    assert np.array_equal(d_back.cpu().numpy(), to.inverse(to.make_params(wq, bq), noise))


def test_more_launches_than_marks():
    """The words that bands pass on carry the mark of their launch, of which there are 255: 600 calls in a row on two
    images by turns, of different heights, so that words of all earlier launches stand where a band looks."""
    rng = np.random.default_rng(12)
    wq, bq = [[ONE // 2, ONE // 4, ONE // 4]] * 3, [3 * ONE, 0, 0]
    p, q = pb.make_twar_params(wq, bq), to.make_params(wq, bq)
    images = [rng.integers(0, 256, s, dtype=np.uint8) for s in ((1, 140, 100, 3), (2, 200, 61, 3))]
    residuals = [torch.from_numpy(to.forward(q, i)).cuda() for i in images]
    images = [torch.from_numpy(i).cuda() for i in images]
    for turn in range(600):
        back = torch.full_like(images[turn % 2], 0xA5)
        pb.pilc_twar_inverse(p, residuals[turn % 2], back)
        assert torch.equal(back, images[turn % 2]), turn


def test_bad_arguments():
    img = torch.zeros((2, 4, 4, 3), dtype=torch.uint8, device="cuda:0")
    out = torch.zeros_like(img)
    p = pb.make_twar_params([[0] * 3] * 3, [0] * 3)
    assert pb.pilc_twar_forward(p, img, img, check=False) == pb.PILC_E_ARG      # in place is not allowed
    assert pb.pilc_twar_inverse(p, img, img, check=False) == pb.PILC_E_ARG
    bad = pb.make_twar_params([[0] * 3] * 3, [(1 << 30) + 1, 0, 0])
    assert pb.pilc_twar_forward(bad, img, out, check=False) == pb.PILC_E_ARG
    empty = torch.zeros((0, 4, 4, 3), dtype=torch.uint8, device="cuda:0")
    assert pb.lib().pilc_twar_forward(0, 4, 4, img.data_ptr(), None, out.data_ptr(), None) == pb.PILC_E_ARG
    del empty
