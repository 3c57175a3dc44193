"""The scans at the edges of their parts (16 sectors),
tiles (64), clusters and positions, under both launch forms (waves for all
sectors, and the persistent grid that a launch shape asks for), with both
signatures, against the oracle: signatures of bytes that stress the signed
digits of djb2 on the matrix cores, and flags and records of ragged images."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_same_matches, gpu_flags_and_matches, oracle_flags_and_matches
from paper_0901_1307_amd import carve

pytestmark = pytest.mark.gpu
SECTOR = 512


def _sectors(n, seed):
    """Random sectors, and among them constant, alternating and single-byte ones."""
    rng = np.random.default_rng(seed)
    s = rng.integers(0, 256, (n, SECTOR), dtype=np.uint8)
    for i in range(0, n, 7):
        s[i] = (0, 255, 128, 127)[(i // 7) % 4]
    for i in range(3, n, 11):
        s[i] = 128
        s[i, (i * 37) % SECTOR] = 255 * (i % 2)
    s[5 % n, ::2], s[5 % n, 1::2] = 255, 0
    return s


@pytest.mark.parametrize("kind", [carve.CARVE_SIG_DJB2_64, carve.CARVE_SIG_CRC64_ISO])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 200, 1029])
def test_signatures(n, kind):
    s = _sectors(n, n)
    got = carve.sector_signatures(torch.from_numpy(s).reshape(-1).cuda(), sig_kind=kind).cpu().numpy().view(np.uint64)
    assert np.array_equal(got, oracle.sector_signatures(s.reshape(-1), 4, sig_kind=kind))


# (blocks per CU, tiles per chunk): waves for all sectors, then the persistent grid
@pytest.mark.parametrize("kind", [carve.CARVE_SIG_DJB2_64, carve.CARVE_SIG_CRC64_ISO])
@pytest.mark.parametrize("shape", [(0, 0), (2, 1), (0, 3)])
@pytest.mark.parametrize("split", [carve.CARVE_SPLIT_OFF, carve.CARVE_SPLIT_ON])
@pytest.mark.parametrize("n", [1, 8, 15, 16, 17, 127, 128, 129, 511, 512, 513, 2000])
def test_ragged_images(n, split, shape, kind):
    rng = np.random.default_rng(n)
    masters = _sectors(300, 1)
    offsets = [0, 100, 107, 300]
    image = rng.integers(0, 256, (n, SECTOR), dtype=np.uint8)
    for j in {0, n - 1, n // 2, n // 3, *range(0, n, 13)}:
        image[j] = masters[int(rng.integers(0, 300))]
    idx = carve.build_master_index(torch.from_numpy(masters).reshape(-1).cuda(), offsets, sig_kind=kind)
    idx.set_scan_config(shape[0], shape[1], split)
    dev = torch.from_numpy(image).reshape(-1).cuda()
    sc = None
    for tau0, any_tau in ((0, False), (5, False), (3, True)):
        flags, matches, sc = gpu_flags_and_matches(idx, dev, tau0, any_tau, sc)
        want_flags, want = oracle_flags_and_matches(masters, offsets, image.reshape(-1), tau0, any_tau, sig_kind=kind)
        assert np.array_equal(flags, want_flags)
        assert_same_matches(matches, want)
