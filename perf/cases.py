"""What the snapshot library is timed on: snapshots, restores, batched plans and
on-demand restores as a checkpointing program calls them, from one small
allocation to gigabytes in many.

A case is a dict of plain values:

  op        "snapshot" (crum_snapshot), "noalloc" (crum_snapshot_noalloc),
            "restore" (crum_restore), "plan" (crum_plan_launch) or "lazy"
            (crum_lazy_open, touches, finish, close)
  nbytes    bytes of the region table, about (cut into whole pages)
  page      page size
  regions   allocations in the table (in each request of a plan)
  dirty     share of the pages that differ from the shadow; -1: no shadow
            (a first snapshot, every page dirty)
  runs      dirty pages come in runs (geometric, mean 32), as in the
            many-allocations workload; else they are scattered
  update    CRUM_UPDATE_SHADOW; a snapshot that updates its shadows follows a
            step of the application that writes the same pages again
  verify    CRUM_VERIFY (restores)
  host      the image is in pinned host memory; else it stays in device memory
  requests  requests of a plan (sizes log-uniform over a factor of 64)
  touches   accesses announced to an on-demand restore before it finishes
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1808_00117_amd as crum
from paper_1808_00117_amd import _lib as C

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30
FIELDS = dict(op="snapshot", nbytes=MiB, page=4 * KiB, regions=1, dirty=0.05, runs=False,
              update=False, verify=False, host=True, requests=0, touches=0)


def _case(name, **kw):
    return dict(FIELDS, name=name, **kw)


def listed():
    return [
        # the smallest request of the batched workload, taken alone: one small
        # allocation, all latency
        _case("snap_1m", nbytes=1 * MiB),
        # the plain workload: one 64 MiB allocation, 4 KiB pages, 5 % changed
        _case("snap_plain_64m", nbytes=64 * MiB),
        # a serving client's checkpoint: one region, 64 KiB pages, shadow kept up to date
        _case("snap_client_update", nbytes=500 * MiB, page=64 * KiB, dirty=0.12, update=True),
        # the many-allocations workload, scaled: 64 allocations, 64 KiB pages, clustered
        _case("snap_many_host", nbytes=1800 * MiB, page=64 * KiB, regions=64, dirty=0.09,
              runs=True),
        # the same at half of its full size, the image kept in device memory
        # (h_image NULL) for a rollback without the host
        _case("snap_many_device", nbytes=8 * GiB, page=64 * KiB, regions=64, dirty=0.09,
              runs=True, host=False),
        # fine pages, many scattered changes, shadows kept up to date, device image
        _case("snap_fine_update", nbytes=1537 * MiB + 20 * KiB, regions=7, dirty=0.37,
              update=True, host=False),
        # a first snapshot: no shadow yet, every page packed, 2 MiB pages
        _case("snap_first_full", nbytes=1 * GiB, page=2 * MiB, regions=5, dirty=-1.0,
              host=False),
        # the allocation-free entry point in a tight loop, odd sizes, 16 KiB pages
        _case("noalloc_odd", op="noalloc", nbytes=37 * MiB + 48 * KiB, page=16 * KiB, regions=11,
              dirty=0.10),
        # a restart from a host image, every page verified before the first write
        _case("restore_host", op="restore", nbytes=600 * MiB, page=64 * KiB, regions=9,
              dirty=0.30, runs=True, verify=True),
        # a rollback from an image in device memory, verified, shadows refreshed
        _case("restore_device", op="restore", nbytes=3 * GiB, page=4 * KiB, regions=16,
              dirty=0.25, verify=True, update=True, host=False),
        # the batched workload, fewer requests: one plan, mixed 4 and 64 KiB pages
        _case("plan_mixed", op="plan", nbytes=800 * MiB, regions=6, dirty=0.20, runs=True,
              requests=24),
        # a restart on demand: random accesses first, then the rest
        _case("lazy_restore", op="lazy", nbytes=256 * MiB, page=64 * KiB, regions=4, dirty=0.25,
              runs=True, verify=True, touches=48),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["snapshot"] * 4 + ["noalloc", "restore", "restore", "plan", "lazy"])
    host = op in ("plan", "lazy") or rng.random() < 0.5
    # a host image's dirty pages cross the link, so those tables are smaller
    top = {"lazy": 256 * MiB, "plan": 800 * MiB, "noalloc": 1 * GiB}.get(
        op, 1800 * MiB if host else 6 * GiB)
    nbytes = size(32 * MiB if op == "plan" else 1 * MiB, top)
    pages = [p for p in (4 * KiB, 8 * KiB, 16 * KiB, 32 * KiB, 64 * KiB, 256 * KiB, 2 * MiB)
             if p * 16 <= nbytes]
    page = rng.choice(pages)
    first = op == "snapshot" and rng.random() < 0.15
    if first:
        nbytes = min(nbytes, 128 * MiB if host else 1 * GiB)
        page = min(page, nbytes // 16 & ~(4 * KiB - 1))
        page = 1 << (page.bit_length() - 1)
    dirty = -1.0 if first else min(rng.uniform(0.01, 0.5),
                                   160 * MiB / nbytes if host else 1.0)
    return dict(FIELDS, op=op, nbytes=nbytes, page=page, regions=rng.randint(1, 64 if op != "plan"
                                                                            else 8),
                dirty=round(dirty, 4), runs=rng.random() < 0.5,
                update=(op in ("snapshot", "noalloc") and not first and rng.random() < 0.5) or
                       (op == "restore" and rng.random() < 0.5),
                verify=op in ("restore", "lazy") and rng.random() < 0.75, host=host,
                requests=rng.randint(2, 32) if op == "plan" else 0,
                touches=rng.randint(1, 64) if op == "lazy" else 0)


# ------------------------------------------------------------------ inputs


def _page_counts(nbytes, page, n):
    """Pages of n allocations of about nbytes in all, sizes spread over a factor of about a
    hundred, as the shape is part of the case it does not depend on the seed."""
    total = max(n, nbytes // page)
    w = np.exp2(np.random.Generator(np.random.PCG64(n)).uniform(0.0, 7.0, n))
    counts = np.maximum(1, np.floor(w / w.sum() * total)).astype(np.int64)
    counts[np.argmax(counts)] += max(total - counts.sum(), 1 - counts.max())
    return counts


def _dirty_pages(rng, n_pages, n_dirty, runs):
    """Exactly n_dirty page indices, ascending."""
    if not runs:
        return np.sort(rng.choice(n_pages, size=n_dirty, replace=False)).astype(np.int64)
    mark = np.zeros(n_pages, bool)
    while mark.sum() < n_dirty:
        start = int(rng.integers(0, n_pages))
        mark[start:start + min(int(rng.geometric(1 / 32)), n_dirty)] = True
    at = np.flatnonzero(mark)
    return at[:n_dirty].astype(np.int64)


class _Table:
    """A region table in one device arena: current bytes, shadows that differ on the
    chosen pages (1 to 16 words each), and where the application writes."""

    def __init__(self, rng, gen, nbytes, page, n_regions, dirty, runs, first_id=1):
        counts = _page_counts(nbytes, page, n_regions)
        lens = counts * page
        offs = np.concatenate([[0], np.cumsum(lens + 512)[:-1]])
        self.page, self.n_pages = page, int(counts.sum())
        words = int(offs[-1] + lens[-1] + 512) // 8
        self.cur = torch.empty(words, dtype=torch.int64, device="cuda").random_(generator=gen)
        self.shadow = None
        self.n_dirty = self.n_pages
        if dirty >= 0:
            self.shadow = self.cur.clone()
            self.n_dirty = min(self.n_pages, max(1, round(dirty * self.n_pages)))
            d = _dirty_pages(rng, self.n_pages, self.n_dirty, runs)
            owner = np.searchsorted(np.cumsum(counts), d, side="right")
            first = np.concatenate([[0], np.cumsum(counts)[:-1]])
            base = torch.from_numpy((offs[owner] + (d - first[owner]) * page) // 8).cuda()
            at = torch.randint(0, page // 8, (self.n_dirty, 16), device="cuda", generator=gen)
            n = torch.randint(1, 17, (self.n_dirty, 1), device="cuda", generator=gen)
            at = torch.where(torch.arange(16, device="cuda") < n, at, at[:, :1]) + base[:, None]
            flip = torch.randint(1, 1 << 62, (self.n_dirty, 1), device="cuda", generator=gen)
            self.shadow[at] = self.cur[at] ^ flip
            self.written = at[:, 0].contiguous()  # one word of each dirty page
            self.one = torch.ones(self.n_dirty, dtype=torch.int64, device="cuda")
        self.lens, self.offs, self.first_id = lens, offs, first_id

    def tuples(self, cur, shadow):
        c = cur.data_ptr()
        s = shadow.data_ptr() if shadow is not None else 0
        return [(c + int(o), s + int(o) if s else 0, int(n), self.first_id + i)
                for i, (o, n) in enumerate(zip(self.offs, self.lens))]

    def image_bytes(self, n_dirty):
        return C.crum_image_bytes(len(self.lens), self.n_pages, n_dirty, self.page)


def _device(n):
    return torch.empty(n // 8, dtype=torch.int64, device="cuda")


def _pinned(n):
    return torch.empty(n // 8, dtype=torch.int64, pin_memory=True)


class _Context:
    """A library context (and plan) that lives as long as the state that uses it."""

    def __init__(self):
        self.ctx, self.plan = C.crum_ctx_create(0), None

    def __del__(self):
        torch.cuda.synchronize()
        if self.plan is not None:
            self.plan.destroy()
        C.crum_ctx_destroy(self.ctx)


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _plan_requests(case):
    """(bytes, page size) of each request, log-uniform over a factor of 64."""
    g = np.random.Generator(np.random.PCG64(case["requests"]))
    w = np.exp2(g.uniform(0.0, 6.0, case["requests"]))
    sizes = np.maximum(1, np.floor(w / w.sum() * case["nbytes"] / (64 * KiB))) * (64 * KiB)
    return [(int(n), 4 * KiB if g.random() < 0.5 else 64 * KiB) for n in sizes]


def prepare(case, seed):
    s = dict(case)
    rng = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s["owner"] = _Context()
    s["ctx"] = ctx = s["owner"].ctx
    op, page = case["op"], case["page"]
    if op == "plan":
        tables, ask, end, worst = [], [], 0, 0
        for i, (n, p) in enumerate(_plan_requests(case)):
            t = _Table(rng, gen, n, p, min(case["regions"], n // p), case["dirty"], case["runs"],
                       64 * i)
            tables.append(t)
            ask.append((t.tuples(t.cur, t.shadow), p, 0, i))
            end = -(-end // 4096) * 4096 + t.image_bytes(t.n_dirty)
            worst = -(-worst // 4096) * 4096 + t.image_bytes(t.n_pages)
        s["tables"] = tables
        s["staging"] = _device(worst).zero_()
        s["image"] = _pinned(worst).zero_()
        s["status"] = torch.zeros(5 * len(ask), dtype=torch.int64, pin_memory=True)
        s["owner"].plan = C.Plan(ctx, ask, s["staging"].data_ptr(), worst,
                                 s["image"].data_ptr(), worst)
        s["out"] = s["image"][: end // 8]
        return s
    t = _Table(rng, gen, case["nbytes"], page, case["regions"], case["dirty"], case["runs"])
    full, size = t.image_bytes(t.n_pages), t.image_bytes(t.n_dirty)
    s["status"] = torch.zeros(5, dtype=torch.int64, pin_memory=True)
    s["table"] = t
    s["regions"] = C.region_table(t.tuples(t.cur, t.shadow))
    s["flags"] = (C.CRUM_UPDATE_SHADOW if case["update"] else 0) | \
        (C.CRUM_VERIFY if case["verify"] else 0)
    if op in ("snapshot", "noalloc"):
        s["staging"] = _device(full)
        s["image"] = _pinned(full) if case["host"] else None
        s["out"] = (s["image"] if case["host"] else s["staging"])[: size // 8]
        return s
    # a restore: the image of the current bytes, and targets that still hold the old ones
    s["staging"] = _device(size)
    s["image"] = _pinned(size) if case["host"] else None
    rc = C.crum_snapshot(ctx, s["regions"], page, 0, seed & 0xFFFF, s["staging"].data_ptr(), size,
                         s["image"].data_ptr() if case["host"] else 0, size, _stream(),
                         s["status"].data_ptr())
    assert rc == C.CRUM_OK
    torch.cuda.synchronize()
    s["image_bytes"] = size
    s["cur"] = t.shadow.clone()
    s["shadow"] = t.shadow if case["update"] else None
    t.cur = t.shadow = None
    s["regions"] = C.region_table(t.tuples(s["cur"], s["shadow"]))
    if op == "lazy":
        r = rng.integers(0, len(t.lens), case["touches"])
        s["touch"] = [(int(i), int(rng.integers(0, t.lens[i] // page)) * page) for i in r]
    return s


# -------------------------------------------------------------------- a pass


def run(s):
    op, stream = s["op"], _stream()
    if op == "plan":
        rc = s["owner"].plan.launch(stream, s["status"].data_ptr())
        out = [s["out"], s["status"]]
    elif op in ("snapshot", "noalloc"):
        t = s["table"]
        if s["update"]:
            # the application's step since the last snapshot
            t.cur.index_add_(0, t.written, t.one)
        call = C.crum_snapshot if op == "snapshot" else C.crum_snapshot_noalloc
        n = s["staging"].numel() * 8
        rc = call(s["ctx"], s["regions"], s["page"], s["flags"], 1, s["staging"].data_ptr(), n,
                  s["image"].data_ptr() if s["host"] else 0, n if s["host"] else 0, stream,
                  s["status"].data_ptr())
        out = [s["out"], s["status"]] + ([t.shadow] if s["update"] else [])
    elif op == "restore":
        rc = C.crum_restore(s["ctx"], s["regions"], s["image"].data_ptr() if s["host"] else 0,
                            s["image_bytes"], s["flags"], s["staging"].data_ptr(),
                            s["image_bytes"], stream, s["status"].data_ptr())
        out = [s["cur"], s["status"]] + ([s["shadow"]] if s["update"] else [])
    else:
        z = C.Lazy(s["ctx"], s["regions"], s["image"].data_ptr(), s["image_bytes"], s["flags"],
                   2 * MiB, s["staging"].data_ptr(), s["image_bytes"], stream,
                   s["status"].data_ptr())
        for region, offset in s["touch"]:
            z.touch(region, offset, s["page"], stream)
        z.finish(stream, s["status"].data_ptr())
        z.close()
        rc = C.CRUM_OK
        out = [s["cur"], s["status"]]
    if rc != C.CRUM_OK:
        raise RuntimeError(f"{op}: {crum.CODE_NAMES.get(rc, rc)}")
    return out


def work(case):
    """Bytes that a pass reads and writes once: a snapshot reads both copies and writes the
    dirty pages to the image (and the shadow), a restore reads the image and writes its pages."""
    def table(nbytes, page, n):
        pages = int(_page_counts(nbytes, page, n).sum())
        n_dirty = pages if case["dirty"] < 0 else min(pages, max(1, round(case["dirty"] * pages)))
        return pages * page, n_dirty * page

    if case["op"] == "plan":
        each = [table(n, p, min(case["regions"], n // p)) for n, p in _plan_requests(case)]
    else:
        each = [table(case["nbytes"], case["page"], case["regions"])]
    total, packed = (sum(v) for v in zip(*each))
    copies = 2 if case["update"] else 1
    if case["op"] in ("restore", "lazy"):
        return {"bytes": packed * (1 + copies), "flops": 0}
    return {"bytes": total * (1 if case["dirty"] < 0 else 2) + packed * copies, "flops": 0}
