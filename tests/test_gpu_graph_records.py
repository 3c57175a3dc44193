"""Records read after replays of a captured scan and confirmation: more of them
than the confirmation has room for, then fewer and others, and the other way
round. Each replay's records are those of the bytes it scanned, whatever an
earlier copy-out had to produce again. The images are copies of master units, so
the records are known without scanning anything."""
import numpy as np
import pytest
import torch

from paper_0901_1307_amd import carve

pytestmark = pytest.mark.gpu
SECTOR, FRAGMENT, N = 512, 64, 4096


def _random(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda", generator=g)


def _captured(enqueue):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        enqueue()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            enqueue()
    return g


def _check(rec, units, masters_of):
    """masters_of: a row per unit, the masters that it equals, ascending."""
    assert np.array_equal(rec["disk_sector"].astype(np.int64), np.repeat(units, masters_of.shape[1]))
    assert np.array_equal(rec["sector_in_file"].astype(np.int64), masters_of.reshape(-1))


# records go to the object's own buffer (room for n/8 + 4096 of them), or to a buffer of the caller with less room
@pytest.mark.parametrize("kind", ["image", "image, own buffer", "batch"])
def test_more_and_fewer_records_than_room(kind):
    masters = _random(8 * SECTOR, 1).view(8, SECTOR)
    masters[6], masters[7] = masters[2], masters[2]   # three records for 2, 6 and 7
    idx = carve.build_master_index(masters.view(-1), [0, 8])
    img = torch.zeros(N, SECTOR, dtype=torch.uint8, device="cuda")
    room = torch.zeros(16 * 100, dtype=torch.uint8, device="cuda")
    state = carve.Batch() if kind == "batch" else carve.Scan()
    any_ = carve.CARVE_TAU_ANY

    def step():
        if kind == "batch":
            carve.scan_batch(idx, [(img[:1024].view(-1), 0, any_), (img[1024:].view(-1), 0, any_)], batch=state)
            carve.confirm_enqueue(idx, state)
        else:
            carve.scan_image(idx, img.view(-1), tau_mode=any_, scan=state)
            carve.confirm_enqueue(idx, state, room if kind == "image, own buffer" else None)

    g = _captured(step)
    for share, master in ((1, 2), (2, 3), (4, 2), (1, 2), (1, 4), (0, 1)):
        img.zero_()
        at = torch.arange(0, N, share, device="cuda") if share else torch.empty(0, dtype=torch.int64, device="cuda")
        img[at] = masters[master]
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        units = at.cpu().numpy()
        same = np.tile([[2, 6, 7] if master == 2 else [master]], (len(units), 1))
        for _ in range(2):
            if kind == "batch":
                rec = carve.batch_confirm_matches(idx, state)
                assert np.array_equal(rec["image"], np.repeat(units >= 1024, same.shape[1]))
                rec["disk_sector"] += 1024 * rec["image"].astype(np.uint64)
            else:
                rec = carve.confirm_matches(idx, state)
            _check(rec, units, same)


@pytest.mark.parametrize("order", ["dense first", "sparse first"])
def test_more_and_fewer_windows_than_room(order):
    """A window scan's confirmation has room for 2^20 flagged windows at least;
    past that it is done again when the records are fetched."""
    fragments = _random(4 * FRAGMENT, 2).view(4, FRAGMENT)
    fragments[1] = 0
    idx = carve.build_fragment_index(fragments.view(-1), [0, 4])
    img = torch.zeros(6 << 20, dtype=torch.uint8, device="cuda")
    n = (img.numel() - FRAGMENT) // 4 + 1
    state = carve.Scan()

    def step():
        carve.scan_fragments(idx, img, scan=state)
        carve.confirm_enqueue(idx, state)

    img.copy_(_random(img.numel(), 3))
    g = _captured(step)
    noise = _random(img.numel(), 4)
    for dense in ((1, 0, 1, 0) if order == "dense first" else (0, 1, 0)):
        if dense:
            img.zero_()
            units, same = np.arange(n), np.ones((n, 1), dtype=np.int64)
        else:
            img.copy_(noise)
            img[4096:4096 + 3 * FRAGMENT] = fragments[[2, 0, 3]].view(-1)
            units, same = np.array([1024, 1040, 1056]), np.array([[2], [0], [3]])
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(carve.flagged_sectors(state).numpy(), units)
        _check(carve.confirm_matches(idx, state), units, same)


@pytest.mark.parametrize("n_words", [9, 16, 23])
def test_captured_scan_beside_a_split_scan(n_words):
    """A graph of a contiguous scan, replayed after the same object scanned the
    image split by position (whose words are eight to a group)."""
    masters = _random(64 * SECTOR, 5).view(64, SECTOR)
    idx = carve.build_master_index(masters.view(-1), [0, 64])
    n = 64 * n_words - 5
    img = torch.zeros(n, SECTOR, dtype=torch.uint8, device="cuda")
    at = torch.arange(0, n, 7, device="cuda")
    img[at] = masters[at % 64]
    state = carve.Scan()
    g = _captured(lambda: carve.scan_image(idx, img.view(-1), tau_mode=carve.CARVE_TAU_ANY, scan=state))
    idx.set_scan_config(0, 0, carve.CARVE_SPLIT_ON)
    for rep in range(3):
        carve.scan_image(idx, img.view(-1), scan=state)
        assert np.array_equal(carve.flagged_sectors(state).numpy(), at.cpu().numpy())
        others = [_random(1 << 20, rep) for _ in range(8)]   # takes what was freed, if anything was
        img[at[rep]] = 0
        at = at[at != at[rep]]
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(carve.flagged_sectors(state).numpy(), at.cpu().numpy())
        del others
