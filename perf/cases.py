"""The work a program has this library do, as cases that can be timed.

A case is one pass through the Python binding's public entry points on seeded
inputs made on the GPU. Seven kinds of work, over the sizes the library is used
at:

* disk     one device-resident image against a resident index of master
           sectors: the step that waits once (scan, confirmation into a device
           buffer, ids into a device buffer, both counts);
* flow     one buffer without cluster alignment, in the allocation-free call
           of a tight loop (nothing is read back);
* batch    many images of uneven sizes in one call, per-image counts, ids and
           records;
* serve    jobs handed to the request loop, polled until all are done, their
           results fetched and released;
* windows  every 64-byte window of an image against a resident index of
           fragments (logos and small files embedded in others);
* build    a new set of master files: the index built, and the first image
           scanned with it;
* ingest   an image in pinned host memory, streamed through device buffers.

Images follow the synthetic recipe of the repository's workloads: random bytes
with clusters copied from the master files (some of them with their first
sectors overwritten), zero clusters and low-entropy clusters.
"""
import math

import numpy as np
import torch

from paper_0901_1307_amd import carve

SECTOR, CLUSTER, WINDOW = 512, 8, 64
KIB, MIB, GIB = 1 << 10, 1 << 20, 1 << 30


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # one captured network flow buffer, as a tight loop scans it: latency
        dict(name="flow 64 KiB", kind="flow", bytes=64 * KIB, masters=1 << 22, crc=False, hits=0.25, zero=0.02,
             low=0.02, low_masters=16),
        # one small disk (the 64 MiB configuration of the tests and the benchmark)
        dict(name="disk 64 MiB", kind="disk", bytes=64 * MIB, masters=4096, crc=False, any=False, tau0=0, hits=0.05,
             zero=0.02, low=0.0, low_masters=0),
        # a partition cut out of a disk: an odd size, a tail, not starting on a cluster, many hits
        dict(name="partition 700 MB, ragged", kind="disk", bytes=700_000_123, masters=65_537, crc=False, any=False,
             tau0=5, hits=0.15, zero=0.05, low=0.02, low_masters=8),
        # the benchmark's 8 GiB disk against a million master sectors
        dict(name="disk 8 GiB", kind="disk", bytes=8 * GIB, masters=1 << 20, crc=False, any=False, tau0=0, hits=0.01,
             zero=0.05, low=0.0, low_masters=0),
        # half of the benchmark's large disk against its 16 M master sectors: an index beyond the L2s
        dict(name="disk 32 GiB, 16M masters", kind="disk", bytes=32 * GIB, masters=1 << 24, crc=False, any=False,
             tau0=0, hits=0.001, zero=0.0, low=0.10, low_masters=64),
        # recorded traffic, the other signature, any position, the served index's 4 M masters
        dict(name="traffic 2 GB, CRC-64, any", kind="disk", bytes=2_000_000_512, masters=1 << 22, crc=True, any=True,
             tau0=0, hits=0.02, zero=0.02, low=0.02, low_masters=16),
        # a folder of small and middling disk images and flow buffers in one call
        dict(name="batch of 256", kind="batch", images=256, low_bytes=64 * KIB, high_bytes=64 * MIB, masters=1 << 20,
             crc=False, hits=0.025, zero=0.05, low=0.0, low_masters=0),
        # a burst of requests to the serving loop
        dict(name="serve a burst of 48", kind="serve", images=48, low_bytes=64 * KIB, high_bytes=16 * MIB,
             masters=1 << 22, crc=False, hits=0.02, zero=0.02, low=0.02, low_masters=16),
        # embedded files in one document or memory dump
        dict(name="windows 16 MiB", kind="windows", bytes=16 * MIB, files=120),
        # the logos configuration: 2,000 files of 2 to 32 KiB in 2 GiB
        dict(name="windows 2 GiB", kind="windows", bytes=2 * GIB, files=2000),
        # a new master set of a million sectors, and a first small disk scanned with it
        dict(name="build 1M masters", kind="build", bytes=64 * MIB, masters=1 << 20, crc=False, any=False, tau0=0,
             hits=0.05, zero=0.05, low=0.0, low_masters=0),
        # a disk read into pinned host memory
        dict(name="ingest 256 MiB", kind="ingest", bytes=256 * MIB, chunk=64 * MIB, masters=1 << 20, crc=False,
             any=False, tau0=0, hits=0.01, zero=0.05, low=0.0, low_masters=0),
    ]


def _log_uniform(rng, low, high):
    return int(math.exp(rng.uniform(math.log(low), math.log(high))))


def draw(rng):
    kind = rng.choice(["disk", "disk", "disk", "flow", "batch", "serve", "windows", "windows", "build", "ingest"])
    if kind == "windows":
        return dict(kind=kind, bytes=_log_uniform(rng, MIB, 2 * GIB), files=_log_uniform(rng, 60, 2000))
    c = dict(kind=kind, masters=_log_uniform(rng, 4096, 1 << 22), crc=rng.random() < 0.2,
             hits=rng.uniform(0.0, 0.1), zero=rng.choice([0.0, 0.02, 0.05]), low=rng.choice([0.0, 0.02]),
             low_masters=rng.choice([0, 8, 16]))
    if kind == "disk":
        c.update(bytes=_log_uniform(rng, MIB, 16 * GIB), any=rng.random() < 0.25, tau0=rng.randrange(8))
        if rng.random() < 0.2:
            c["masters"] = _log_uniform(rng, 1 << 22, 1 << 24)
    elif kind == "flow":
        c.update(bytes=_log_uniform(rng, 16 * KIB, 16 * MIB))
    elif kind == "build":
        c.update(bytes=_log_uniform(rng, 4 * MIB, 256 * MIB), any=False, tau0=0)
    elif kind == "ingest":
        c.update(bytes=_log_uniform(rng, 16 * MIB, 256 * MIB), chunk=rng.choice([16 * MIB, 64 * MIB]), any=False,
                 tau0=rng.randrange(8))
    else:
        c.update(images=rng.randrange(4, 257 if kind == "batch" else 65), low_bytes=rng.choice([4 * KIB, 64 * KIB]),
                 high_bytes=rng.choice([MIB, 16 * MIB, 64 * MIB]) if kind == "batch" else rng.choice([MIB, 16 * MIB]))
    return c


def _sizes(case):
    """The images of a batch or burst: (bytes, tau0, any position), the same for every seed. Sizes are
    spread over their logarithm; images under 1 MiB are flow buffers, matched at any position."""
    rng = np.random.default_rng(case["images"])
    lo, hi = math.log(case["low_bytes"]), math.log(case["high_bytes"])
    out = []
    for u, t in zip(rng.uniform(lo, hi, case["images"]), rng.integers(0, 8, case["images"])):
        n = int(math.exp(u)) // SECTOR * SECTOR
        out.append((n, 0 if n < MIB else int(t), n < MIB))
    return out


def work(case):
    if case["kind"] in ("batch", "serve"):
        read = sum(n for n, _, _ in _sizes(case))
    else:
        read = case["bytes"]
    if case["kind"] == "windows":
        return {"bytes": read + read // 4 // 8, "flops": 0}      # one flag bit per window
    n = read / SECTOR
    if case["kind"] == "build":
        read += case["masters"] * (SECTOR + 8)                   # the master sectors, a signature each
    # one flag bit per sector, and per hit: its bytes and the master's, an id and a record
    return {"bytes": read + n / 8 + n * case["hits"] * (2 * SECTOR + 24), "flops": 0}


# ------------------------------------------------------------------ the inputs
def _generator(seed, salt):
    return torch.Generator(device="cuda").manual_seed(seed * 1_000_003 + salt)


def _random_bytes(n, g):
    out = torch.empty((n + 7) // 8, dtype=torch.int64, device="cuda")
    for s in range(0, out.numel(), 1 << 27):
        out[s:s + (1 << 27)].random_(-2**63, None, generator=g)
    return out.view(torch.uint8)[:n]


def _patterns(g):
    """The pool of 4-byte patterns that low-entropy clusters and masters repeat."""
    return torch.randint(-2**31, 2**31, (4096,), dtype=torch.int64, device="cuda", generator=g).to(torch.int32)


def _masters(case, seed):
    """Packed master sectors, the files' sector offsets, the first sector of every whole cluster and the
    pattern pool. About 1,000 sectors a file at random cut points; one sector in a thousand is a copy."""
    n, g = case["masters"], _generator(seed, 1)
    cuts = torch.randint(1, n, (max(1, n // 1024),), device="cuda", generator=g).unique().tolist()
    offsets = [0] + cuts + [n]
    data, pool = _random_bytes(n * SECTOR, g).view(n, SECTOR), _patterns(g)
    pairs = torch.randperm(n, device="cuda", generator=g)[:2 * (n // 1000)].view(2, -1)
    data[pairs[0]] = data[pairs[1]]
    if case["low_masters"]:
        at = torch.randperm(n, device="cuda", generator=g)[:case["low_masters"]]
        data.view(torch.int32)[at] = pool[:case["low_masters"], None].expand(-1, SECTOR // 4)
    off = torch.tensor(offsets, device="cuda")
    clusters = (off[1:] - off[:-1]) // CLUSTER
    first = torch.repeat_interleave(off[:-1], clusters)
    within = torch.arange(first.numel(), device="cuda") - torch.repeat_interleave(clusters.cumsum(0) - clusters,
                                                                                  clusters)
    return data, offsets, first + CLUSTER * within, pool


def _image(case, seed, salt, n_bytes, tau0, masters):
    """A disk image: random, with copied (at least one), zero and low-entropy clusters at its cluster boundaries."""
    data, _, starts, pool = masters
    g = _generator(seed, salt)
    img = _random_bytes(n_bytes, g)
    lead = -tau0 % CLUSTER
    n_clusters = max(0, n_bytes // SECTOR - lead) // CLUSTER
    sectors = img[:n_bytes // SECTOR * SECTOR].view(-1, SECTOR)
    u = torch.rand(n_clusters, device="cuda", generator=g)
    if n_clusters:
        u[u.argmin()] = -1.0
    copied = (u < case["hits"]).nonzero()[:, 0]
    kept = torch.rand(copied.numel(), device="cuda", generator=g)
    skip = torch.where(kept < 0.3, 1 + (kept * 1000).long() % 3, 0)     # leading sectors since overwritten
    src = starts[torch.randint(max(1, starts.numel()), (copied.numel(),), device="cuda", generator=g)] \
        if starts.numel() else copied[:0]
    step = torch.arange(CLUSTER, device="cuda")
    keep = step[None, :] >= skip[:src.numel(), None]
    to, frm = (lead + copied[:src.numel(), None] * CLUSTER + step)[keep], (src[:, None] + step)[keep]
    for s in range(0, to.numel(), 1 << 20):
        sectors[to[s:s + (1 << 20)]] = data[frm[s:s + (1 << 20)]]
    for low, share in ((False, case["zero"]), (True, case["low"])):
        a = case["hits"] + (case["zero"] if low else 0.0)
        at = ((u >= a) & (u < a + share)).nonzero()[:, 0]
        pick = pool[torch.randint(pool.numel(), (at.numel(),), device="cuda", generator=g)] * int(low)
        for i in range(CLUSTER):
            for s in range(0, at.numel(), 1 << 20):
                sectors.view(torch.int32)[lead + at[s:s + (1 << 20)] * CLUSTER + i] = \
                    pick[s:s + (1 << 20), None].expand(-1, SECTOR // 4)
    return img


def _fragments(case, seed):
    """Files of 2 to 32 KiB, and an image with whole copies of them: one in each of three in four 64 KiB
    stretches, four of five on a 4-byte boundary."""
    g = _generator(seed, 2)
    u = torch.rand(case["files"], dtype=torch.float64, device="cuda", generator=g)
    sizes = torch.exp(math.log(2 * KIB) + u * math.log(16)).long()
    ends = sizes.cumsum(0)
    data = _random_bytes(int(ends[-1]), g)
    n, stretch = case["bytes"], 64 * KIB
    img = _random_bytes(n, g)
    copies = (n // stretch) * 3 // 4
    slot = torch.randperm(n // stretch, device="cuda", generator=g)[:copies]
    which = torch.randint(case["files"], (copies,), device="cuda", generator=g)
    place = slot * stretch + torch.randint(8 * KIB, (copies,), device="cuda", generator=g) * 4
    place += torch.where(torch.rand(copies, device="cuda", generator=g) < 0.2, 1 + which % 3, 0)
    for s in range(0, copies, 2048):
        length = sizes[which[s:s + 2048]]
        within = torch.arange(int(length.sum()), device="cuda") - torch.repeat_interleave(length.cumsum(0) - length,
                                                                                         length)
        at = torch.repeat_interleave(place[s:s + 2048], length) + within
        img[at] = data[torch.repeat_interleave((ends - sizes)[which[s:s + 2048]], length) + within]
    pieces = [data[e - z:e] for e, z in zip(ends.tolist(), sizes.tolist())]
    return pieces, img


# ------------------------------------------------------------------ a user's program
def _index(case, masters):
    return carve.build_master_index(masters[0].view(-1), masters[1], sig_kind=int(case["crc"]))


def _room(case):
    """Ids and records that a program provides for: all of them, and some more."""
    if case["kind"] == "windows":
        return case["bytes"] // 4 // 64 + 4096
    n = sum(n for n, _, _ in _sizes(case)) if case["kind"] in ("batch", "serve") else case["bytes"]
    return int(n // SECTOR * (1.3 * case["hits"] + 1 / 64)) + 4096


def _outputs(case, device="cuda", record=16):
    """Room for the ids and the records of a pass."""
    return dict(ids=torch.full((_room(case),), -1, dtype=torch.int64, device=device),
                records=torch.zeros(_room(case) * record, dtype=torch.uint8, device=device))


def prepare(case, seed):
    kind = case["kind"]
    if kind == "windows":
        pieces, img = _fragments(case, seed)
        packed, offsets = carve.pack_fragment_files(pieces)
        return dict(kind=kind, image=img, index=carve.build_fragment_index(packed, offsets), scan=None,
                    **_outputs(case))
    masters = _masters(case, seed)
    if kind in ("batch", "serve"):
        jobs = [(_image(case, seed, 10 + i, n, t, masters), t, int(any_))
                for i, (n, t, any_) in enumerate(_sizes(case))]
        index = _index(case, masters)
        if kind == "serve":
            return dict(kind=kind, jobs=jobs, server=carve.Server(index, budget_bytes=4 * GIB),
                        **_outputs(case, "cpu"))
        return dict(kind=kind, jobs=jobs, index=index, batch=None, ids=_outputs(case, "cpu")["ids"],
                    records=_outputs(case, record=24)["records"])
    if kind == "flow":
        return dict(kind=kind, index=_index(case, masters), image=_image(case, seed, 3, case["bytes"], 0, masters),
                    ids=_outputs(case)["ids"], count=torch.zeros(1, dtype=torch.int64, device="cuda"))
    img = _image(case, seed, 3, case["bytes"], case["tau0"], masters)
    state = dict(kind=kind, image=img, tau0=case["tau0"], any=int(case["any"]))
    if kind == "ingest":
        state["image"] = torch.empty(img.numel(), dtype=torch.uint8, pin_memory=True).copy_(img)
        state.update(ingest=carve.Ingest(_index(case, masters), chunk_bytes=case["chunk"]), **_outputs(case, "cpu"))
        return state
    state.update(scan=None, **_outputs(case))
    if kind == "build":
        state.update(masters=masters[0].view(-1), offsets=masters[1], sig=int(case["crc"]))
    else:
        state["index"] = _index(case, masters)
    return state


def _step(index, scan, s):
    """Confirmation, ids and counts behind a scan; the host waits once, for the counts."""
    carve.confirm_enqueue(index, scan, s["records"])
    carve.flagged_sectors_enqueue(scan, s["ids"])
    flagged, confirmed = carve.scan_counts(scan)
    return dict(ids=s["ids"], records=s["records"], flagged=flagged, confirmed=confirmed)


def _keep(s, ids, records):
    """Host results into the program's own arrays."""
    s["ids"].numpy()[:len(ids)] = ids
    s["records"].numpy()[:records.nbytes] = records.view(np.uint8)
    return dict(ids=s["ids"], records=s["records"], flagged=len(ids), confirmed=len(records))


def run(s):
    kind = s["kind"]
    if kind == "flow":
        carve.scan_image_noalloc(s["index"], s["image"], s["ids"], s["count"], tau_mode=carve.CARVE_TAU_ANY)
        return dict(ids=s["ids"], count=s["count"])
    if kind == "windows":
        s["scan"] = carve.scan_fragments(s["index"], s["image"], scan=s["scan"])
        return _step(s["index"], s["scan"], s)
    if kind == "disk":
        s["scan"] = carve.scan_image(s["index"], s["image"], s["tau0"], s["any"], scan=s["scan"])
        return _step(s["index"], s["scan"], s)
    if kind == "build":
        index = carve.build_master_index(s["masters"], s["offsets"], sig_kind=s["sig"])
        scan = carve.scan_image(index, s["image"], s["tau0"], s["any"])
        out = _step(index, scan, s)
        out["signatures"] = index.stats()["n_unique_signatures"]
        return out
    if kind == "batch":
        s["batch"] = carve.scan_batch(s["index"], s["jobs"], batch=s["batch"])
        carve.confirm_enqueue(s["index"], s["batch"])
        confirmed = carve.batch_confirm_matches(s["index"], s["batch"], s["records"])
        ids = carve.batch_flagged_sectors(s["batch"], carve.CARVE_ALL_IMAGES)
        s["ids"][:ids.numel()] = ids
        return dict(ids=s["ids"], records=s["records"], confirmed=confirmed,
                    flagged=carve.batch_flag_counts(s["batch"]).astype(np.int64))
    if kind == "ingest":
        s["ingest"].scan(s["image"], s["tau0"], s["any"])
        return _keep(s, s["ingest"].flagged(), s["ingest"].matches())
    jobs = [s["server"].submit(t, tau0, any_) for t, tau0, any_ in s["jobs"]]
    left = len(jobs)
    while left:
        left -= len(s["server"].poll())
    flags = [s["server"].flags(j) for j in jobs]
    records = [s["server"].matches(j) for j in jobs]
    for j in jobs:
        s["server"].release(j)
    out = _keep(s, np.concatenate(flags), np.concatenate(records))
    out["flagged"] = np.array([len(f) for f in flags], dtype=np.int64)
    return out


# ------------------------------------------------------------------ the same, plainly, in 64 bits
def _signed(x):
    x &= 2**64 - 1
    return x - 2**64 if x >= 2**63 else x


def _djb2(rows):
    """djb2 of each row of bytes (Eq. (1) unrolled: a sum with the powers of 33, modulo 2^64)."""
    n = rows.shape[1]
    w = torch.tensor([_signed(33**(n - 1 - b)) for b in range(n)], device=rows.device)
    init = _signed(5381 * 33**n)
    return torch.cat([(rows[s:s + (1 << 17)].long() * w).sum(1) + init for s in range(0, rows.shape[0], 1 << 17)]
                     or [torch.empty(0, dtype=torch.int64, device=rows.device)])


def _crc64(rows):
    """CRC-64/GO-ISO of each row of bytes, a byte at a time through its table."""
    table = []
    for b in range(256):
        for _ in range(8):
            b = (b >> 1) ^ (0xD800000000000000 if b & 1 else 0)
        table.append(_signed(b))
    table = torch.tensor(table, device=rows.device)
    out = []
    for s in range(0, rows.shape[0], 1 << 20):
        cols = rows[s:s + (1 << 20)].t().contiguous()
        crc = torch.full((cols.shape[1],), -1, dtype=torch.int64, device=rows.device)
        for col in cols:
            crc = table[(crc ^ col.long()) & 255] ^ ((crc >> 8) & (2**56 - 1))
        out.append(~crc)
    return torch.cat(out or [torch.empty(0, dtype=torch.int64, device=rows.device)])


def _pairs(signatures, order, sig, unit):
    """(unit, master) for every unit whose signature a master has; order sorts the masters' signatures."""
    a, b = torch.searchsorted(signatures, sig), torch.searchsorted(signatures, sig, right=True)
    n = b - a
    within = torch.arange(int(n.sum()), device=sig.device) - torch.repeat_interleave(n.cumsum(0) - n, n)
    return torch.repeat_interleave(unit, n), order[torch.repeat_interleave(a, n) + within]


def _records(unit, master, offsets, image=None):
    """The records of (unit, master) pairs, as the bytes the library returns."""
    off = torch.tensor(offsets, device=unit.device)
    f = torch.searchsorted(off, master, right=True) - 1
    cols = [unit & 0xFFFFFFFF, unit >> 32, f, master - off[f]]
    if image is not None:
        cols += [image, torch.zeros_like(unit)]
    return torch.stack(cols, 1).to(torch.int32).view(torch.uint8).reshape(-1)


class _Plain:
    """The masters' signatures in order, and the flags and matches of an image."""

    def __init__(self, case, seed):
        self.masters = _masters(case, seed)
        self.data, self.offsets = self.masters[:2]
        self.hash = _crc64 if case["crc"] else _djb2
        self.signatures, self.order = self.hash(self.data).sort(stable=True)
        off = torch.tensor(self.offsets, device="cuda")
        ids = torch.arange(self.data.shape[0], device="cuda")
        self.position = (ids - off[torch.searchsorted(off, ids, right=True) - 1]) % CLUSTER

    def scan(self, img, tau0, any_):
        """Flagged sectors, and the (sector, master) pairs that are equal byte for byte."""
        rows = img[:img.numel() // SECTOR * SECTOR].view(-1, SECTOR)
        found = []
        for s in range(0, rows.shape[0], 1 << 20):
            sig = self.hash(rows[s:s + (1 << 20)])
            at = torch.searchsorted(self.signatures, sig).clamp(max=self.signatures.numel() - 1)
            maybe = (self.signatures[at] == sig).nonzero()[:, 0]
            unit, master = _pairs(self.signatures, self.order, sig[maybe], maybe + s)
            if not any_:
                ok = self.position[master] == (unit + tau0) % CLUSTER
                unit, master = unit[ok], master[ok]
            same = torch.cat([(rows[unit[k:k + (1 << 18)]] == self.data[master[k:k + (1 << 18)]]).all(1)
                              for k in range(0, unit.numel(), 1 << 18)] or [unit.bool()])
            found.append((unit.unique(), unit[same], master[same]))
        return [torch.cat(x) for x in zip(*found)] if found else [self.order[:0]] * 3


def _plain_windows(case, seed):
    pieces, img = _fragments(case, seed)
    data, offsets = carve.pack_fragment_files(pieces)
    data = data.view(-1, WINDOW)
    signatures, order = _djb2(data).sort(stable=True)
    words = img[:img.numel() // 4 * 4].view(-1, 4)
    n = (img.numel() - WINDOW) // 4 + 1
    weights = torch.tensor([33**3, 33**2, 33, 1], device="cuda")
    found = []
    for s in range(0, n, 1 << 24):
        e = min(n, s + (1 << 24))
        d = (words[s:e + 15].long() * weights).sum(1)
        sig = torch.full((e - s,), 5381, dtype=torch.int64, device="cuda")
        for k in range(16):
            sig = sig * 33**4 + d[k:k + e - s]
        at = torch.searchsorted(signatures, sig).clamp(max=signatures.numel() - 1)
        maybe = (signatures[at] == sig).nonzero()[:, 0]
        unit, master = _pairs(signatures, order, sig[maybe], maybe + s)
        flat = words.reshape(-1)
        step = torch.arange(WINDOW, device="cuda")
        same = torch.cat([(flat[unit[k:k + (1 << 20), None] * 4 + step] == data[master[k:k + (1 << 20)]]).all(1)
                          for k in range(0, unit.numel(), 1 << 20)] or [unit.bool()])
        found.append((unit.unique(), unit[same], master[same]))
    flags, unit, master = [torch.cat(x) for x in zip(*found)]
    return _padded(case, flags, _records(unit, master, offsets), unit.numel())


def _padded(case, flags, records, confirmed):
    """Ids and records in the room that a program provides."""
    ids = torch.full((_room(case),), -1, dtype=torch.int64, device="cuda")
    ids[:flags.numel()] = flags
    data = torch.zeros(_room(case) * (24 if case["kind"] == "batch" else 16), dtype=torch.uint8, device="cuda")
    data[:records.numel()] = records
    return dict(ids=ids, records=data, flagged=flags.numel(), confirmed=confirmed)


def exact(case, seed):
    kind = case["kind"]
    if kind == "windows":
        return _plain_windows(case, seed)
    plain = _Plain(case, seed)
    if kind in ("batch", "serve"):
        flags, records, counts = [], [], []
        for i, (n, t, any_) in enumerate(_sizes(case)):
            f, unit, master = plain.scan(_image(case, seed, 10 + i, n, t, plain.masters), t, any_)
            flags.append(f)
            counts.append(f.numel())
            records.append(_records(unit, master, plain.offsets,
                                    torch.full_like(unit, i) if kind == "batch" else None))
        records = torch.cat(records)
        out = _padded(case, torch.cat(flags), records, records.numel() // (24 if kind == "batch" else 16))
        out["flagged"] = np.array(counts, dtype=np.int64)
        return out
    flow = kind == "flow"
    tau0 = 0 if flow else case["tau0"]
    flags, unit, master = plain.scan(_image(case, seed, 3, case["bytes"], tau0, plain.masters), tau0,
                                     flow or case["any"])
    out = _padded(case, flags, _records(unit, master, plain.offsets), unit.numel())
    if flow:
        return dict(ids=out["ids"], count=torch.tensor([flags.numel()]))
    if kind == "build":
        out["signatures"] = plain.signatures.unique().numel()
    return out
