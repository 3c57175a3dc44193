"""Flagged ids and records at the edges of the compaction and of the record
offsets: hit words on both sides of a block's chunk, of the one-launch form and
of the wide chunks; batches whose images start and end there. Images are zero
bytes with master units copied to chosen places, so the flags and records are
known without scanning anything."""
import numpy as np
import pytest
import torch

from gpu_util import assert_same_matches, gpu_flags_and_matches, oracle_flags_and_matches
from paper_0901_1307_amd import carve

pytestmark = pytest.mark.gpu
SECTOR, FRAGMENT = 512, 64
N_MASTERS = 64


def _random(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=g)


def _places(n_units, chunk):
    """Unit ids around word, chunk and end boundaries (units are 64 to a word)."""
    edges = {0, 63, 64, n_units - 1, n_units - 64, n_units // 2}
    for m in (1, 2, 63, 64, 4096):
        edges |= {64 * chunk * m - 1, 64 * chunk * m}
    rng = np.random.default_rng(n_units)
    edges |= set(int(v) for v in rng.integers(0, n_units, 300))
    return np.array(sorted(e for e in edges if 0 <= e < n_units), dtype=np.int64)


def _check(idx, sc, places, masters_of):
    assert np.array_equal(carve.flagged_sectors(sc).numpy(), places)
    rec = carve.confirm_matches(idx, sc)
    assert np.array_equal(rec["disk_sector"].astype(np.int64), places)
    assert np.array_equal(rec["sector_in_file"].astype(np.int64), masters_of)


# words: one block and its end, the one-launch form's end, summed chunks of 1024 words
@pytest.mark.parametrize("n_words", [1, 255, 256, 257, 1025, 16384, 16385])
def test_sector_ids_at_chunk_edges(n_words):
    masters = _random(N_MASTERS * SECTOR, 1).view(N_MASTERS, SECTOR)
    idx = carve.build_master_index(masters.view(-1), [0, N_MASTERS])
    n = n_words * 64 - 3
    image = torch.zeros(n, SECTOR, dtype=torch.uint8, device="cuda")
    places = _places(n, 1024 if n_words > 16384 else 256)
    which = (places * 7) % N_MASTERS
    image[torch.from_numpy(places).cuda()] = masters[torch.from_numpy(which).cuda()]
    sc = carve.scan_image(idx, image.view(-1), tau_mode=carve.CARVE_TAU_ANY)
    _check(idx, sc, places, which)
    ids = torch.full((len(places) + 1,), -1, dtype=torch.int64, device="cuda")
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    carve.scan_image_noalloc(idx, image.view(-1), ids, count, tau_mode=carve.CARVE_TAU_ANY)
    assert int(count) == len(places)
    assert np.array_equal(ids.cpu().numpy(), np.append(places, -1))


# words: chunks of 4096 summed in the emitting blocks, and past 4096 of them scanned first
@pytest.mark.parametrize("n_words", [(1 << 22) + 1, (1 << 24) + 1])
def test_window_ids_in_wide_chunks(n_words):
    frags = _random(N_MASTERS * FRAGMENT, 2)
    idx = carve.build_fragment_index(frags, [0, N_MASTERS])
    windows = n_words * 64 - 5
    image = torch.zeros(windows * 4 + 60, dtype=torch.uint8, device="cuda")
    places = _places(windows, 4096)
    places = places[np.append(True, np.diff(places) >= 16)]   # whole fragments, not overlapping
    which = (places * 5) % N_MASTERS
    at = torch.from_numpy(places).cuda()[:, None] * 4 + torch.arange(FRAGMENT, device="cuda")
    image[at] = frags.view(N_MASTERS, FRAGMENT)[torch.from_numpy(which).cuda()]
    sc = carve.scan_fragments(idx, image)
    _check(idx, sc, places, which)


# images of 64-sector words; empty ones, ones that start on and beside a chunk's edge, empty ones at the end
@pytest.mark.parametrize("words", [[0, 0, 255, 1, 0, 256, 3, 0, 0], [256, 256, 0], [5],
                                   [16384, 0, 1, 1023, 1024, 7, 0]])
def test_batch_images_at_chunk_edges(words):
    masters = _random(N_MASTERS * SECTOR, 3).view(N_MASTERS, SECTOR)
    idx = carve.build_master_index(masters.view(-1), [0, N_MASTERS])
    images, want, recs = [], [], []
    for i, w in enumerate(words):
        n = max(0, w * 64 - i % 5)
        img = torch.zeros(n, SECTOR, dtype=torch.uint8, device="cuda")
        places = _places(n, 256) if n else np.empty(0, dtype=np.int64)
        which = (places + i) % N_MASTERS
        if n:
            img[torch.from_numpy(places).cuda()] = masters[torch.from_numpy(which).cuda()]
        images.append((img.view(-1), 0, carve.CARVE_TAU_ANY))
        want.append(places)
        recs.append(np.stack([np.full_like(places, i), places, which], 1))
    b = carve.scan_batch(idx, images)
    assert carve.batch_flag_counts(b).tolist() == [len(p) for p in want]
    got = carve.batch_flagged_sectors(b, carve.CARVE_ALL_IMAGES).numpy()
    assert np.array_equal(got, np.concatenate(want))
    r = carve.batch_confirm_matches(idx, b)
    got = np.stack([r["image"], r["disk_sector"], r["sector_in_file"]], 1).astype(np.int64)
    assert np.array_equal(got, np.concatenate(recs))


# lengths of a signature's candidate list on both sides of the mask's short form (32) and of its ranks (63)
@pytest.mark.parametrize("length", [1, 31, 32, 33, 62, 63, 64, 70])
@pytest.mark.parametrize("any_tau", [False, True])
def test_candidate_list_lengths(length, any_tau):
    rng = np.random.default_rng(length)
    a = rng.integers(40, 200, SECTOR, dtype=np.uint8)
    b = a.copy()
    b[100] += 1   # the same djb2: 33 * 1 less 33
    b[101] -= 33
    masters = np.where(np.arange(length)[:, None] % 3 == 1, b, a).astype(np.uint8)
    offsets = [0, length // 2, length]
    image = rng.integers(0, 256, (200, SECTOR), dtype=np.uint8)
    image[::5], image[1::7] = a, b
    idx = carve.build_master_index(torch.from_numpy(masters).reshape(-1).cuda(), offsets)
    flags, matches, _ = gpu_flags_and_matches(idx, torch.from_numpy(image).reshape(-1).cuda(), 3, any_tau)
    want_flags, want = oracle_flags_and_matches(masters, offsets, image.reshape(-1), 3, any_tau)
    assert np.array_equal(flags, want_flags)
    assert_same_matches(matches, want)


# flagged units on both sides of the confirmation's ranges: a block's 32 sectors, 2048 blocks of them, two passes each
@pytest.mark.parametrize("flagged", [0, 1, 31, 33, 2048 * 32 - 1, 2048 * 32, 2048 * 32 + 1, 2048 * 64 + 5])
def test_record_offsets_at_range_edges(flagged):
    masters = _random(8 * SECTOR, 4).view(8, SECTOR)
    masters[5], masters[6] = masters[2], masters[2]   # three records for master 2, 5 and 6
    idx = carve.build_master_index(masters.view(-1), [0, 8])
    n = 2048 * 64 + 300
    image = torch.zeros(n, SECTOR, dtype=torch.uint8, device="cuda")
    places = torch.from_numpy(np.sort(np.random.default_rng(flagged).permutation(n)[:flagged])).cuda()
    which = torch.arange(flagged, device="cuda") % 8
    image[places] = masters[which]
    sc = carve.scan_image(idx, image.view(-1), tau_mode=carve.CARVE_TAU_ANY)
    assert carve.flagged_sectors(sc).numel() == flagged
    rec = carve.confirm_matches(idx, sc)
    triple = ((which == 2) | (which == 5) | (which == 6)).cpu().numpy()
    repeat = np.where(triple, 3, 1)
    assert np.array_equal(rec["disk_sector"].astype(np.int64), np.repeat(places.cpu().numpy(), repeat))
    master = [[2, 5, 6] if t else [int(w)] for t, w in zip(triple, which.tolist())]
    assert np.array_equal(rec["sector_in_file"], np.array(sum(master, []), dtype=np.uint32))
