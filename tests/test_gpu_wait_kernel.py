"""scan_wait_kernel from a scan object's first scan on: the other stream waits for
the scan kernel and not for what is enqueued behind it on the scan's stream."""
import pytest
import torch

from paper_0901_1307_amd import carve

pytestmark = pytest.mark.gpu
SECTOR = 512


@pytest.mark.parametrize("kind", ["djb2", "crc", "split", "capped", "capped split", "runs", "batch", "windows", "timed"])
def test_first_scan_of_an_object(kind):
    data = torch.randint(0, 256, (64 * SECTOR,), dtype=torch.uint8, device="cuda")
    image = torch.randint(0, 256, (8192 * SECTOR,), dtype=torch.uint8, device="cuda")
    image[:data.numel()] = data
    if kind == "windows":
        idx = carve.build_fragment_index(data, [0, data.numel() // 64])
    else:
        idx = carve.build_master_index(data, [0, 64], sig_kind=int(kind == "crc"))
        idx.set_scan_config(1 if "capped" in kind else 0, 2 if kind == "runs" else 0,
                            carve.CARVE_SPLIT_ON if "split" in kind else carve.CARVE_SPLIT_OFF)
    ours, other = torch.cuda.Stream(), torch.cuda.Stream()

    def scan():
        if kind == "batch":
            return carve.scan_batch(idx, [(image, 0, 0)])
        if kind == "timed":   # (the object's second scan: timing is switched on for an object that there is)
            sc = carve.scan_image(idx, image)
            sc.set_timing(True)
            return carve.scan_image(idx, image, scan=sc)
        return carve.scan_fragments(idx, image) if kind == "windows" else carve.scan_image(idx, image)

    scan()                                   # (the code objects are loaded)
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    with torch.cuda.stream(ours):
        sc = scan()
        torch.cuda._sleep(100_000_000)       # tens of milliseconds at least
        end = torch.cuda.Event()
        end.record()
    carve.scan_wait_kernel(sc, other)
    other.synchronize()
    assert not end.query()                   # what came behind the scan is still running
    torch.cuda.synchronize()
    assert carve.scan_counts(sc)[0] > 0


def test_first_wait_after_many_scans():
    """An object scanned many times without a wait: its first wait is for all that its stream holds,
    the next ones are for the kernel alone again."""
    data = torch.randint(0, 256, (64 * SECTOR,), dtype=torch.uint8, device="cuda")
    image = torch.cat([data] * 128)
    idx = carve.build_master_index(data, [0, 64])
    ours, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(ours):
        sc = carve.scan_image(idx, image)
        for n in range(2, 20):
            carve.scan_image(idx, image, scan=sc)
        for alone in (False, True, True):
            carve.scan_image(idx, image, scan=sc)
            torch.cuda._sleep(100_000_000)
            end = torch.cuda.Event()
            end.record()
            carve.scan_wait_kernel(sc, other)
            other.synchronize()
            assert end.query() != alone
            torch.cuda.synchronize()
    assert carve.scan_counts(sc)[0] == 128 * 64


def test_two_streams_in_one_capture():
    """Objects made during a capture, the second one's stream joined by scan_wait_kernel."""
    data = torch.randint(0, 256, (64 * SECTOR,), dtype=torch.uint8, device="cuda")
    image = torch.cat([data] * 16)
    idx = carve.build_master_index(data, [0, 64])
    ours, other = torch.cuda.Stream(), torch.cuda.Stream()
    first, second = carve.Scan(), carve.Scan()
    with torch.cuda.stream(ours):
        carve.scan_image(idx, image)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=ours, capture_error_mode="relaxed"):
            carve.scan_image(idx, image, scan=first)
            carve.scan_wait_kernel(first, other)
            with torch.cuda.stream(other):
                carve.scan_image(idx, image, tau_mode=carve.CARVE_TAU_ANY, scan=second)
                carve.confirm_enqueue(idx, second)
            ours.wait_stream(other)
            carve.confirm_enqueue(idx, first)
    for gone in range(3):
        image[gone * SECTOR:(gone + 1) * SECTOR] = 0
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert carve.scan_counts(first) == carve.scan_counts(second) == (16 * 64 - gone - 1, 16 * 64 - gone - 1)
