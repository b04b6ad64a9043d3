"""Workloads of the GPU page cache for timing: each case is one pass of a reader over files
the cache holds (served from GPU memory) or does not hold (fetched by the host threads from a
memory file system, so that the host link and not a disk is the limit).

Three kinds, one per public launcher:

* ``list``: ``runner.ListReader``, blocks reading one file at given offsets;
* ``batch``: ``runner.BatchReader``, one persistent launch over many files of uneven sizes;
* ``serve``: ``runner.serve``, a stream of whole-file requests.

A case gives its sizes in bytes. ``cached``: the files fit the cache and were read once
before; otherwise the file is larger than the cache, so a pass finds at most the tail that
the previous pass left.
"""
import math
import os
import random
import tempfile

import numpy as np
import torch

from paper_2109_05366_amd import gfs, runner

KiB, MiB = 1 << 10, 1 << 20
CONSUMERS = {"checksum": 0, "histogram": 1, "none": 2}


def _list(name, **over):
    c = {"name": name, "kind": "list", "page": 64 * KiB, "cache": 256 * MiB, "ra_cap": 1 * MiB, "cached": True,
         "file": 64 * MiB, "blocks": 64, "reads": 16, "read": 64 * KiB, "pitch": 0, "pattern": "strided",
         "consumer": "checksum", "threads": 256, "advice": "normal", "ra_async": False, "policy": "shared"}
    c.update(over)
    return c


def listed():
    return [
        # the smallest call: one block reads 4 KiB that the cache holds (a kernel that looks
        # up one small object); its launch and the chain of one hit are all there is
        _list("one_read", blocks=1, reads=1, read=4 * KiB, file=1 * MiB + 40, cache=16 * MiB, consumer="none"),
        # a small file read again: 64 blocks, 64 KiB strides of 64 MiB (the small plain configuration)
        _list("small_file"),
        # a data set that stays in the cache, read whole: the all-hit configuration, reads alone
        _list("resident_stream", file=512 * MiB, cache=1024 * MiB, blocks=512, reads=16, consumer="none"),
        # the same through 4 KiB pages in 128 KiB reads (the small-page configuration, second epoch on)
        _list("resident_small_pages", page=4 * KiB, file=256 * MiB, cache=512 * MiB, ra_cap=64 * KiB, blocks=1024,
              reads=2, read=128 * KiB),
        # byte histograms over 256 KiB pages in half-page reads (the large-stream configuration's
        # reader over a file that fits)
        _list("resident_histogram", page=256 * KiB, file=512 * MiB, cache=1024 * MiB, blocks=1024, reads=4,
              read=128 * KiB, consumer="histogram"),
        # lookups of packed records: 4080 bytes at multiples of 4093, so at every byte alignment,
        # in random order, pages crossed now and then
        _list("resident_records", file=128 * MiB + 777, cache=256 * MiB, blocks=512, reads=64, read=4080, pitch=4093,
              pattern="records", consumer="none"),
        # many files of uneven, ragged sizes in one persistent launch, second epoch on
        {"name": "resident_batch", "kind": "batch", "page": 64 * KiB, "cache": 1024 * MiB, "ra_cap": 1 * MiB,
         "cached": True, "files": 64, "median": 4 * MiB, "unit": 1 * MiB, "per_file": 8, "threads": 256},
        # a burst of whole-file requests over a pool that the cache holds
        {"name": "resident_serve", "kind": "serve", "page": 256 * KiB, "cache": 512 * MiB, "ra_cap": 4 * MiB,
         "cached": True, "files": 16, "median": 4 * MiB, "requests": 64, "chunk": 1 * MiB, "threads": 256,
         "noalloc": False},
        # a file larger than the cache streamed through it with readahead: the headline
        # configuration's pages, reads and consumer
        _list("stream", page=256 * KiB, file=1024 * MiB + 24 * KiB + 8, cache=512 * MiB, ra_cap=4 * MiB, cached=False,
              blocks=512, reads=17, read=128 * KiB, consumer="histogram"),
        # every block its own part of the file, asynchronous readahead
        _list("own_parts", file=512 * MiB, cache=256 * MiB, ra_cap=4 * MiB, cached=False, blocks=256, reads=32,
              pattern="chunked", ra_async=True),
        # 4 KiB pages fetched through 64 KiB windows
        _list("small_pages", page=4 * KiB, file=256 * MiB, cache=64 * MiB, ra_cap=64 * KiB, cached=False, blocks=1024,
              reads=2, read=128 * KiB),
        # single pages at random, readahead switched off for the file by its advice
        _list("random_pages", file=512 * MiB, cache=128 * MiB, cached=False, blocks=1024, reads=8, pattern="random",
              advice="random"),
    ]


def _log(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["cached", "cached", "records", "streamed", "random", "batch", "serve"])
    if kind == "batch":
        page = rng.choice([16, 64, 256]) * KiB
        return {"kind": "batch", "page": page, "cache": 1024 * MiB, "ra_cap": 1 * MiB, "cached": True,
                "files": _log(rng, 3, 63), "median": _log(rng, 256 * KiB, 4 * MiB), "unit": _log(rng, 4, 64) * 16 * KiB + 16,
                "per_file": rng.choice([1, 4, 8, 16]), "threads": 256}
    if kind == "serve":
        return {"kind": "serve", "page": rng.choice([64, 256]) * KiB, "cache": 512 * MiB, "ra_cap": 4 * MiB, "cached": True,
                "files": _log(rng, 2, 15), "median": _log(rng, 128 * KiB, 4 * MiB), "requests": _log(rng, 1, 60),
                "chunk": _log(rng, 2, 7) * 16 * KiB, "threads": 256, "noalloc": rng.random() < 0.5}
    c = _list("")
    del c["name"]
    c["threads"] = rng.choice([64, 128, 256, 256])
    c["consumer"] = rng.choice(["checksum", "histogram", "none"])
    if kind == "records":
        pitch = _log(rng, 300, 20000) | 1
        c.update(pattern="records", pitch=pitch, read=max(16, pitch // 16 * 16), page=rng.choice([4, 64, 256]) * KiB,
                 file=_log(rng, 1 * MiB, 128 * MiB), blocks=_log(rng, 1, 1000), reads=_log(rng, 8, 60))
        return c
    c["blocks"] = _log(rng, 1, 1000)
    if kind == "random":
        policy = rng.choice(["shared", "shared", "private"])
        page = rng.choice([16, 64] if policy == "private" else [16, 64, 256]) * KiB   # private: a share of 512 is a page or more
        c.update(pattern="random", advice="random", cached=False, page=page, read=page, cache=64 * MiB,
                 file=_log(rng, 3 * 64 * MiB, 400 * MiB), blocks=min(c["blocks"], 32 * MiB // page), threads=256,
                 policy=policy, ra_cap=0 if policy == "private" else 1 * MiB)
        c["reads"] = max(1, min(32, 128 * MiB // (page * c["blocks"])))
        return c
    page = rng.choice([4, 16, 64, 256]) * KiB
    c["page"] = page
    c["pattern"] = rng.choice(["strided", "chunked"])
    if kind == "cached":
        c["read"] = max(16, _log(rng, 256, 2 * MiB) // 16 * 16)
        size = min(_log(rng, 64 * KiB, 400 * MiB), 48 * c["read"] * c["blocks"])
        c["cache"] = 512 * MiB
    else:
        c["read"] = rng.choice([1, 2, 4, 8]) * 16 * KiB
        size = _log(rng, 24 * MiB, 32 * MiB if page < 64 * KiB else 256 * MiB)
        size = min(size, 4096 * c["read"] * c["blocks"])
        c.update(cached=False, ra_cap=rng.choice([0, 64 * KiB, 1 * MiB, 4 * MiB]) // page * page, ra_async=rng.random() < 0.3)
        # room for a read of every block and some more, and less than the file
        share = max(c["read"], page) * 5 // 4
        c["blocks"] = min(c["blocks"], 128 * MiB // share)
        c["cache"] = max(64 * page, c["blocks"] * share // page * page)
        size = max(size, c["cache"] * 3 // 2)
    c["file"] = size
    c["reads"] = -(-size // (c["read"] * c["blocks"]))
    return c


def _sizes(case):
    """File sizes of a batch or a pool: lognormal about the median, a multiple of 8 bytes."""
    r = random.Random("%d files of %d" % (case["files"], case["median"]))
    return [int(min(max(r.lognormvariate(math.log(case["median"]), 0.9), 8 * KiB), 8 * case["median"])) // 8 * 8
            for _ in range(case["files"])]


def _requested(case):
    r = random.Random("%d requests" % case["requests"])
    return [r.randrange(case["files"]) for _ in range(case["requests"])]


def _offsets(case, seed):
    b = np.arange(case["blocks"], dtype=np.uint64)[:, None]
    k = np.arange(case["reads"], dtype=np.uint64)[None, :]
    read = np.uint64(case["read"])
    if case["pattern"] == "strided":
        return (b + np.uint64(case["blocks"]) * k) * read
    if case["pattern"] == "chunked":
        return (b * np.uint64(case["reads"]) + k) * read
    pitch = case["pitch"] if case["pattern"] == "records" else case["page"]
    at = np.random.RandomState(seed % (1 << 32)).randint(0, case["file"] // pitch, (case["blocks"], case["reads"]))
    return at.astype(np.uint64) * np.uint64(pitch)


def _delivered(case):
    if case["kind"] == "batch":
        return sum(_sizes(case))
    if case["kind"] == "serve":
        sizes = _sizes(case)
        return sum(sizes[i] for i in _requested(case))
    end = _offsets(case, 1).astype(np.int64)
    return int(np.clip(case["file"] - end, 0, case["read"]).sum())


def work(case):
    """Every delivered byte is read once and written once."""
    return {"bytes": 2 * _delivered(case), "flops": 0}


def _contents(total, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    words = torch.randint(-(1 << 63), (1 << 63) - 1, (total // 8 + 1,), dtype=torch.int64, device="cuda", generator=g)
    return words.cpu().numpy().view(np.uint8)[:total]


class State:
    """An open cache, its files and the reader's buffers. The files have no name any more once
    they are open, so they go when the cache closes."""

    def __init__(self, case, seed):
        self.case = case
        cfg = dict(page_size=case["page"], cache_bytes=case["cache"], ra_cap_bytes=case["ra_cap"])
        if case.get("ra_async"):
            cfg["ra_async"] = 1
        if case.get("policy") == "private":
            cfg.update(policy=gfs.GFS_POLICY_PRIVATE, private_slots=512)
        self.cache = gfs.PageCache(runner.make_config(**cfg))
        sizes = _sizes(case) if case["kind"] != "list" else [case["file"]]
        data = _contents(sum(sizes), seed)
        self.ids, at = [], 0
        for n in sizes:
            self.ids.append(self._open(data[at:at + n]))
            at += n
        if case["kind"] == "list":
            if case["advice"] == "random":
                self.cache.fadvise(self.ids[0], gfs.GFS_ADV_RANDOM)
            self.reader = runner.ListReader(_offsets(case, seed), case["read"], CONSUMERS[case["consumer"]],
                                            case["threads"])
            self.reader.buf.zero_()
        elif case["kind"] == "batch":
            self.reader = runner.BatchReader(self.ids, sizes, case["unit"], case["per_file"], threads=case["threads"])
        else:
            self.requests = [self.ids[i] for i in _requested(case)]
        if case["cached"]:
            run(self)
            if case["kind"] == "list" and case["consumer"] == "none":
                torch.cuda.synchronize()
                self.reader.buf.zero_()

    def _open(self, data):
        fd, path = tempfile.mkstemp(dir="/dev/shm" if os.path.isdir("/dev/shm") else None)
        try:
            with os.fdopen(fd, "wb", buffering=0) as f:
                view = memoryview(data)
                while len(view):
                    view = view[f.write(view[:256 * MiB]):]
            return self.cache.open(path)
        finally:
            os.unlink(path)

    def __del__(self):
        cache = getattr(self, "cache", None)
        if cache is not None:
            torch.cuda.synchronize()
            cache.close()


def prepare(case, seed):
    return State(case, seed)


def run(state):
    case = state.case
    if case["kind"] == "serve":
        records, _ = runner.serve(state.cache, state.requests, [0] * len(state.requests), case["cache"],
                                  chunk_bytes=case["chunk"], threads=case["threads"], noalloc=case["noalloc"])
        return {"csum": records["csum"].view(np.int64), "result": records["result"]}
    r = state.reader
    if case["kind"] == "batch":
        r.launch(state.cache)
        return {"csum": r.csum, "hist": r.hist, "status": r.status.sum()}
    r.launch(state.cache, state.ids[0])
    return {"out": r.buf if r.out is None else r.out, "status": r.status}


def _csum(data):
    words = len(data) // 4 * 4
    tail = int.from_bytes(data[words:].tobytes(), "little")
    return (int(data[:words].copy().view("<u4").sum(dtype=np.uint64)) + tail) % (1 << 64)


def _signed(values):
    return np.array(values, dtype=np.uint64).view(np.int64)


def exact(case, seed):
    if case["kind"] != "list":
        sizes = _sizes(case)
        data, at, files = _contents(sum(sizes), seed), 0, []
        for n in sizes:
            files.append(data[at:at + n])
            at += n
        sums = [_csum(f) for f in files]
        if case["kind"] == "serve":
            asked = _requested(case)
            return {"csum": _signed([sums[i] for i in asked]), "result": np.array([sizes[i] for i in asked], dtype=np.int64)}
        hist = np.concatenate([np.bincount(f, minlength=256) for f in files]).astype(np.int32)
        return {"csum": _signed(sums), "hist": hist, "status": sum(sizes)}
    data = _contents(case["file"], seed)
    out, status = [], []
    for row in _offsets(case, seed).astype(np.int64):
        parts = [data[o:o + case["read"]] for o in row]
        status.append(sum(len(p) for p in parts))
        if case["consumer"] == "checksum":
            out.append(sum(_csum(p) for p in parts) % (1 << 64))
        elif case["consumer"] == "histogram":
            out.append(sum(np.bincount(p, minlength=256) for p in parts).astype(np.int32))
        else:
            buf = np.zeros(case["read"], dtype=np.uint8)
            for p in parts:
                buf[:len(p)] = p
            out.append(buf)
    out = _signed(out) if case["consumer"] == "checksum" else np.concatenate(out)
    return {"out": out, "status": np.array(status, dtype=np.int64)}
