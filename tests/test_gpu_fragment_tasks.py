"""The fragment scan's two kernels at their edges: the largest image of one
task (1024 windows) per wave and the smallest of more, whole and partial last
tasks, with runs in which every window passes both filters (more candidates
than a wave queues at once), against the CPU oracle element by element."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_same_matches, dev_bytes
from paper_0901_1307_amd import carve

pytestmark = pytest.mark.gpu

TASK = 4096      # bytes of image a task starts windows in
WAVES = 16       # of a block; one block per CU


@pytest.mark.parametrize("bloom", [0, carve.CARVE_BLOOM_OFF])
@pytest.mark.parametrize("extra", [-1, 0, 1, 64, 1023, 1025])
def test_one_and_more_tasks_per_wave(extra, bloom):
    """A full grid's tasks and `extra` windows."""
    waves = WAVES * torch.cuda.get_device_properties(0).multi_processor_count
    n_windows = waves * (TASK // 4) + extra
    n_bytes = 4 * (n_windows - 1) + 64
    rng = np.random.default_rng(1000 + extra)
    files = [rng.integers(0, 256, 64 * int(n), dtype=np.uint8).tobytes() for n in rng.integers(1, 40, 100)]
    period = rng.integers(0, 256, 4, dtype=np.uint8).tobytes()
    files.append(period * 16)
    img = rng.integers(0, 256, n_bytes, dtype=np.uint8)
    for at in [0, TASK - 32, 1000 * TASK - 4, (waves - 1) * TASK + 8, n_bytes - 64]:   # across tasks, and the ends
        img[at:at + 64] = np.frombuffer(files[at % 100][:64], np.uint8)
    for at, n in [(40 * TASK, 3 * TASK), (77 * TASK + 100, 300), (n_bytes - 700, 600)]:
        img[at:at + n] = np.frombuffer(period * (n // 4), np.uint8)
    for i in rng.integers(100, waves - 2, 500):   # whole files, at any 4-byte offset
        f = np.frombuffer(files[int(i) % 100], np.uint8)
        at = int(i) * TASK + 4 * int(rng.integers(0, 400))
        img[at:at + len(f)] = f
    frag_data, offsets = oracle.pack_fragment_files(files)
    idx = carve.build_fragment_index(dev_bytes(frag_data.tobytes()), offsets, bloom_bits_per_key=bloom)
    sc = carve.scan_fragments(idx, dev_bytes(img.tobytes()))
    f = carve.flagged_sectors(sc).numpy().astype(np.uint64)
    m = carve.confirm_matches(idx, sc)
    ox = oracle.FragmentIndex(frag_data, offsets, threads=oracle.default_threads())
    wf = ox.flag_windows(img, threads=oracle.default_threads())
    assert len(wf) > 3 * 1024
    assert np.array_equal(f, wf)
    assert_same_matches(m, ox.confirm_windows(img, wf))
