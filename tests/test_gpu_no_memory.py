"""Scan objects after a scan that asked for more device memory than there is:
their results are refused, nothing is launched on buffers given up to make room,
and the object serves the next scan. The requests are far past the card's memory
(one image listed many times, or the windows of a very large one), so each fails
at once."""
import numpy as np
import pytest
import torch

from gpu_util import assert_same_matches, oracle_flags_and_matches
from paper_0901_1307_amd import carve

pytestmark = pytest.mark.gpu
SECTOR = 512


def _refused(f):
    with pytest.raises(carve.CarveError) as e:
        f()
    assert e.value.code == carve.CARVE_EINVAL


def _masters(unit):
    rng = np.random.default_rng(1)
    return rng.integers(0, 256, (32, unit), dtype=np.uint8)


def test_batch_larger_than_memory():
    masters = _masters(SECTOR)
    idx = carve.build_master_index(torch.from_numpy(masters).reshape(-1).cuda(), [0, 32])
    small = np.random.default_rng(2).integers(0, 256, (200, SECTOR), dtype=np.uint8)
    small[::3] = masters[np.arange(0, 200, 3) % 32]
    image = torch.from_numpy(small).reshape(-1).cuda()
    flags, matches = oracle_flags_and_matches(masters, [0, 32], small.reshape(-1), 0, True)
    big = torch.zeros(1 << 30, dtype=torch.uint8, device="cuda")
    b = carve.Batch()
    for _ in range(2):
        carve.scan_batch(idx, [(image, 0, carve.CARVE_TAU_ANY)], batch=b)
        carve.confirm_enqueue(idx, b)
        assert np.array_equal(carve.batch_flagged_sectors(b, 0).numpy().astype(np.uint64), flags)
        assert_same_matches(carve.batch_confirm_matches(idx, b)[list(matches.dtype.names)], matches)
        with pytest.raises(carve.CarveError) as e:   # 16 bytes for each of 2^35 sectors
            carve.scan_batch(idx, [(big, 0, 0)] * (1 << 14), batch=b)
        assert e.value.code == carve.CARVE_ENOMEM
        out = torch.zeros(24 * 64, dtype=torch.uint8, device="cuda")
        _refused(lambda: carve.confirm_enqueue(idx, b))
        _refused(lambda: carve.batch_confirm_matches(idx, b, out))
        _refused(lambda: carve.batch_flagged_sectors(b, carve.CARVE_ALL_IMAGES))
        _refused(lambda: carve.batch_flag_counts(b))
        _refused(lambda: carve.scan_counts(b))


def test_windows_larger_than_memory():
    masters = _masters(64)
    idx = carve.build_fragment_index(torch.from_numpy(masters).reshape(-1).cuda(), [0, 32])
    image = torch.zeros(1 << 16, dtype=torch.uint8, device="cuda")
    image[4096:4096 + 32 * 64] = torch.from_numpy(masters).reshape(-1).cuda()
    torch.cuda.empty_cache()
    big = torch.empty(80 << 30, dtype=torch.uint8, device="cuda")
    sc = carve.Scan()
    out = torch.zeros(16 * 64, dtype=torch.uint8, device="cuda")
    ids = torch.zeros(64, dtype=torch.int64, device="cuda")
    for _ in range(2):
        carve.scan_fragments(idx, image, scan=sc)
        rec = carve.confirm_matches(idx, sc)
        assert np.array_equal(rec["disk_sector"], 1024 + 16 * np.arange(32))
        with pytest.raises(carve.CarveError) as e:   # 12 bytes for each of 20 G windows
            carve.scan_fragments(idx, big, scan=sc)
        assert e.value.code == carve.CARVE_ENOMEM
        _refused(lambda: carve.confirm_enqueue(idx, sc))
        _refused(lambda: carve.confirm_enqueue(idx, sc, out))
        _refused(lambda: carve.confirm_matches(idx, sc, out))
        _refused(lambda: carve.flagged_sectors_enqueue(sc, ids))
        _refused(lambda: carve.flagged_sectors(sc))
        _refused(lambda: carve.scan_counts(sc))
    del big
    torch.cuda.empty_cache()
