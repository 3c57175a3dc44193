"""Position-split scans without slot records (the call without allocation), with
every layout and launch form, against the oracle; and the automatic rule on both
sides of its lines, a filter of 8 MiB and an image of more than 512 MiB, against
the contiguous scan."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import assert_same_matches, gpu_flags_and_matches, oracle_flags_and_matches
from paper_0901_1307_amd import carve

pytestmark = pytest.mark.gpu
SECTOR = 512


def _noalloc(idx, image, tau0=0, any_tau=False):
    ids = torch.full((image.numel() // SECTOR,), -1, dtype=torch.int64, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    carve.scan_image_noalloc(idx, image, ids, count, tau0, int(any_tau))
    return ids[:int(count)].cpu().numpy().astype(np.uint64)


# (blocks per CU, tiles per chunk): waves for all sectors, a capped grid, runs of tiles
@pytest.mark.parametrize("kind", [carve.CARVE_SIG_DJB2_64, carve.CARVE_SIG_CRC64_ISO])
@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("shape", [(0, 0), (2, 1), (0, 3)])
def test_split_without_allocation(shape, layout, kind):
    rng = np.random.default_rng(layout)
    masters = rng.integers(0, 256, (500, SECTOR), dtype=np.uint8)
    offsets = [0, 200, 203, 500]
    idx = carve.build_master_index(torch.from_numpy(masters).reshape(-1).cuda(), offsets, sig_kind=kind, layout=layout)
    idx.set_scan_config(*shape, carve.CARVE_SPLIT_ON)
    for n in (1, 7, 8, 127, 128, 129, 511, 513, 5000, 40_003):   # (the last: several tiles a wave of the capped grid)
        image = rng.integers(0, 256, (n, SECTOR), dtype=np.uint8)
        for j in {0, n - 1, *range(0, n, 11)}:
            image[j] = masters[int(rng.integers(0, 500))]
        dev = torch.from_numpy(image).reshape(-1).cuda()
        for tau0 in (0, 5):
            want_flags, want = oracle_flags_and_matches(masters, offsets, image.reshape(-1), tau0, False, sig_kind=kind)
            assert np.array_equal(_noalloc(idx, dev, tau0), want_flags)
            flags, matches, _ = gpu_flags_and_matches(idx, dev, tau0)
            assert np.array_equal(flags, want_flags)
            assert_same_matches(matches, want)


@pytest.fixture(scope="module")
def large():
    """A million masters and an image of 512 MiB and 65 sectors with copies of them in it."""
    g = torch.Generator(device="cuda").manual_seed(3)
    n, m = (1 << 20) + 65, 1 << 20
    masters = torch.randint(-2**62, 2**62, (m * 64,), device="cuda", generator=g).view(torch.uint8).view(m, SECTOR)
    image = torch.randint(-2**62, 2**62, (n * 64,), device="cuda", generator=g).view(torch.uint8).view(n, SECTOR)
    at = torch.cat([torch.randperm(n, device="cuda", generator=g)[:20_000], torch.arange(n - 80, n, device="cuda")])
    image[at] = masters[torch.randint(m, (at.numel(),), device="cuda", generator=g)]
    return masters.view(-1), image.view(-1)


# bits per master: filters of 4 and of 8 MiB; sectors: the last image of the one-launch compaction, one sector and
# one word more
@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1, (1 << 20) + 64, (1 << 20) + 65])
def test_automatic_rule(large, bits, n):
    masters, image = large
    idx = carve.build_master_index(masters, [0, 1 << 19, 1 << 20], bloom_bits_per_key=bits)
    assert idx.stats()["bloom_bytes"] == (bits // 32) * (4 << 20)
    img = image[:n * SECTOR]
    got = {}
    for split in (carve.CARVE_SPLIT_AUTO, carve.CARVE_SPLIT_OFF, carve.CARVE_SPLIT_ON):
        idx.set_scan_config(0, 0, split)
        got[split] = gpu_flags_and_matches(idx, img, 3)[:2] + (_noalloc(idx, img, 3),)
    flags, matches, ids = got[carve.CARVE_SPLIT_OFF]
    assert len(matches) > 1000 and np.array_equal(flags, ids)
    for split in (carve.CARVE_SPLIT_AUTO, carve.CARVE_SPLIT_ON):
        assert np.array_equal(got[split][0], flags) and np.array_equal(got[split][2], flags)
        assert_same_matches(got[split][1], matches)


def test_whole_mid_image():
    """8 GiB against a million masters, split (claims and all in the capped form) and contiguous."""
    cfg = synth.CONFIGS["mid"]
    ms = synth.master_set(cfg, device="cuda")
    image = synth.disk_image(cfg, ms, device="cuda").data
    idx = carve.build_master_index(ms.sectors, ms.file_offsets, bloom_bits_per_key=32)
    idx.set_scan_config(0, 0, carve.CARVE_SPLIT_OFF)
    flags, matches, _ = gpu_flags_and_matches(idx, image)
    assert len(flags) > 10_000
    for shape in ((0, 0), (3, 2)):
        idx.set_scan_config(*shape, carve.CARVE_SPLIT_ON)
        got = gpu_flags_and_matches(idx, image)
        assert np.array_equal(got[0], flags) and np.array_equal(_noalloc(idx, image), flags)
        assert_same_matches(got[1], matches)
