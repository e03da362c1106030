"""Autotuning driver: chooses launch shapes per (op, k, size) in embed/extract
pairs and on cold covers, the large-image workload's in its own sequence, sweeps
the batched kernel, and stores the winners as JSON next to this file.

``load()`` installs a stored table into the library (called on import of
paper_0912_0947_amd.api).  Buckets that were not tuned take the entry of the
nearest tuned bucket of the same (op, k).

Usage on a GPU: ``python -m paper_0912_0947_amd.tune [--batch]``.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
TABLE = os.path.join(HERE, "tune_gfx950.json")
# One size per bucket from 2 MB on, in its middle or the size of a workload that falls into it.
SIZES = [{22: 6220800, 27: 201326592}.get(b, 3 << (b - 1)) for b in range(21, 31)]
KS = range(1, 9)
# Buffers from here up take streaming (non-temporal) shapes only: one cover
# and its stego no longer fit the 256 MB last-level cache.
STREAM_MIN = 1 << 27
# Runs of blocks per XCD start at 128 blocks: smaller covers keep launch order.
RUNS_MIN = 1 << 21
ROT_SETS = 3
BLOCKS, UNROLLS, CAPS, ORDERS = (256, 512, 1024), (1, 2, 4), (0, 1, 2, 4, 8, 16), (0, 1)


def bucket(n: int) -> int:
    return max(int(n).bit_length() - 1, 0)


def load(handle=None, path: str = TABLE) -> bool:
    """Install a stored tuning table into the library; returns False if there
    is none.  ``handle`` is the loaded liblsb.so (the binding passes it while
    it loads the library)."""
    if not os.path.exists(path):
        return False
    import ctypes

    from ._lib import LaunchCfg, check

    if handle is None:
        from ._lib import lib
        handle = lib()
    with open(path) as f:
        table = json.load(f)
    by_opk = {}
    for e in table.get("entries", []):
        by_opk.setdefault((e["op"], e["k"]), []).append(e)
    for (op, k), entries in by_opk.items():
        tuned = {e["bucket"]: e["cfg"] for e in entries}
        keys = sorted(tuned)
        for b in range(64):
            c = tuned[min(keys, key=lambda t: (abs(t - b), t))]
            cfg = LaunchCfg(c["block"], c["unroll"], c["blocks_per_cu"], c["nontemporal"], c.get("pack", 0),
                            c.get("order", 0))
            if handle.lsb_tune_set(op, k, b, ctypes.byref(cfg)) != 0:
                raise RuntimeError("bad tuning entry %s" % c)
    if "batch" in table:
        c = table["batch"]["cfg"]
        cfg = LaunchCfg(c["block"], c["unroll"], c["blocks_per_cu"], c["nontemporal"], 0)
        if handle.lsb_batch_tune_set(ctypes.byref(cfg), int(table["batch"]["tile_vectors"])) != 0:
            raise RuntimeError("bad batch tuning entry %s" % table["batch"])
        c = table["batch"].get("extract_cfg")
        if c:
            cfg = LaunchCfg(c["block"], c["unroll"], c["blocks_per_cu"], c["nontemporal"], 0)
            if handle.lsb_batch_tune_set_op(1, ctypes.byref(cfg)) != 0:
                raise RuntimeError("bad batch extract tuning entry %s" % c)
    _ = check
    return True


class Timer:
    """Launches of embed and extract over arenas of covers, stegos and
    messages, each timed by events bound to its kernel."""

    def __init__(self, arena: int = 6 << 30):
        import torch

        from . import api, inputs
        from ._lib import lib

        dev = torch.device("cuda:0")
        self.lib, self.arena, self.at = lib(), arena, 0
        self.cover, self.stego = (torch.empty(arena, dtype=torch.uint8, device=dev) for _ in range(2))
        self.msg, self.out = (torch.empty(arena // 4, dtype=torch.uint8, device=dev) for _ in range(2))
        inputs.fill_uniform(self.cover, 13)
        inputs.fill_uniform(self.msg, 23)
        self.state = torch.zeros(2, dtype=torch.int32, device=dev)
        self.ev = [[torch.cuda.Event(enable_timing=True) for _ in range(2)] for _ in range(64)]
        for pair in self.ev:  # create the HIP events (torch records lazily); the library re-records them
            for e in pair:
                e.record()
        torch.cuda.synchronize()
        self.run = {api.OP_EMBED: self._embed, api.OP_EXTRACT: self._extract}

    def use(self, k: int, n: int, at: int = 0) -> None:
        """Covers of n bytes at k, each ``at`` bytes behind an aligned address,
        every stego of the arena a valid one."""
        from . import api

        self.k, self.n, self.cap, self.lead = k, n, min(api.capacity(n, k), 1 << 30), at
        self.step, self.mstep = -(-(at + n) // 256) * 256, -(-self.cap // 256) * 256
        self.slots, self.mslots = self.arena // self.step, self.arena // 4 // self.mstep
        for i in range(self.slots):
            self._embed(i, None)

    def _embed(self, i, ev):
        from . import api

        c, m = i % self.slots * self.step + self.lead, i % self.mslots * self.mstep
        if ev:
            self.lib.lsb_time_next_launch(*ev)
        api.embed(self.cover[c:c + self.n], self.msg[m:m + self.cap], self.k, out=self.stego[c:c + self.n])

    def _extract(self, i, ev):
        from . import api

        c, m = i % self.slots * self.step + self.lead, i % self.mslots * self.mstep
        if ev:
            self.lib.lsb_time_next_launch(*ev)
        api.extract(self.stego[c:c + self.n], self.k, out=self.out[m:m + self.cap], len_status=self.state)

    def hot(self, passes: int):
        """(embed, extract) us of passes that embed into one of three buffer
        sets in turn and at once extract from it."""
        import torch

        for i in range(passes):
            self._embed(i % 3, self.ev[2 * i])
            self._extract(i % 3, self.ev[2 * i + 1])
        torch.cuda.synchronize()
        us = [a.elapsed_time(b) * 1e3 for a, b in self.ev[:2 * passes]]
        return list(zip(us[::2], us[1::2]))

    def cold(self, op: int, launches: int):
        """us of launches on covers that no cache holds: each a seventh of the
        arena behind the one before."""
        import torch

        for i in range(launches):
            self.at += max(1, self.slots // 7)
            self.run[op](self.at, self.ev[i])
        torch.cuda.synchronize()
        return [a.elapsed_time(b) * 1e3 for a, b in self.ev[:launches]]

    def check(self) -> None:
        """The last extract returned its message."""
        assert self.state.cpu().tolist() == [self.cap, 0], (self.k, self.n, self.state.cpu().tolist())


def _install(op: int, k: int, n: int, c: dict) -> None:
    from . import api

    api.tune_set(op, k, bucket(n), c["block"], c["unroll"], c["blocks_per_cu"], c["nontemporal"], c["pack"], c["order"])


def _shapes(nts, orders, packs=(0,)):
    """Candidate shapes, plain ones first: shapes that tie take the first."""
    return [{"block": b, "unroll": u, "blocks_per_cu": c, "nontemporal": nt, "pack": pk, "order": o}
            for pk in packs for c in CAPS for o in orders for u in UNROLLS for b in BLOCKS for nt in nts]


def _choose(best_of, hot, cold):
    """Index of the shape with the lowest cold time among those within 2 % of
    the best hot time; within 1 % of that, the first."""
    near = [i for i in best_of if hot[i] <= 1.02 * min(hot[j] for j in best_of)]
    low = min(cold[i] for i in near)
    return min(i for i in near if cold[i] <= 1.01 * low)


def tune_pair(timer: Timer, k: int, n: int, reps: int = 4, finals: int = 24, log=print):
    """Shapes of embed and extract for (k, n), each chosen in two views.  Hot:
    passes that embed into a stego buffer and extract from it, over three buffer
    sets in turn, with the other operation at its best shape so far; the sum of
    both launches, so a shape that leaves the memory system in a state the next
    kernel pays for, or its output in the caches, is charged or credited for it.
    Cold: single launches on covers that no cache holds, as a loop over an
    archive sees them.  Candidates take turns (slow drift of the device affects
    all alike); the best ``finals`` hot ones are timed again, hot and cold, and
    among those that are as good hot the best cold one is taken (either view
    alone picks shapes that the other finds up to a quarter slower).  Returns
    the two table entries."""
    import statistics

    from . import api

    timer.use(k, n)
    nts = (1,) if n >= STREAM_MIN else (0, 1)
    orders = ORDERS if n >= RUNS_MIN else (0,)
    first = _shapes((nts[-1],), (0,))[0]
    best = {api.OP_EMBED: first, api.OP_EXTRACT: first}
    entries = {}
    for op in (api.OP_EXTRACT, api.OP_EMBED, api.OP_EXTRACT):
        for o in best:
            _install(o, k, n, best[o])
        cands = _shapes(nts, orders, (0, 1) if op == api.OP_EXTRACT and k == 1 else (0,))

        def turns(indices, rounds, passes, view):
            times = {i: [] for i in indices}
            for r in range(rounds + 1):
                for i in indices:
                    _install(op, k, n, cands[i])
                    t = view(passes)
                    if r:  # round 0 warms every shape up
                        times[i] += t
            return times

        hot = turns(range(len(cands)), reps, 1, timer.hot)
        hot = {i: statistics.median(e + x for e, x in ts) for i, ts in hot.items()}
        last = sorted(sorted(hot, key=hot.get)[:finals])
        both = turns(last, reps, 6, timer.hot)
        cold = turns(last, reps, 6, lambda c: timer.cold(op, c))
        hot = {i: statistics.median(e + x for e, x in ts) for i, ts in both.items()}
        cold = {i: statistics.median(ts) for i, ts in cold.items()}
        i = _choose(last, hot, cold)
        best[op] = cands[i]
        _install(op, k, n, best[op])
        entries[op] = {"op": op, "k": k, "bucket": bucket(n), "n": n, "cfg": best[op],
                       "us": round(statistics.median(t[op] for t in both[i]), 2), "cold_us": round(cold[i], 2),
                       "method": "hot and cold"}
    timer.check()
    log("k=%d n=%d -> %s" % (k, n, ["%s %.1f us hot, %.1f cold" % (list(e["cfg"].values()), e["us"], e["cold_us"])
                                    for e in entries.values()]))
    return [entries[0], entries[1]]


def keep_better(timer: Timer, stored, new, rounds: int = 6, log=print):
    """Of two pairs of entries of one (k, n), the new one only if it is better by
    more than measurements differ: both pairs take turns, hot and cold, on
    aligned covers and on covers at byte 54 of a file; the sum of the four views
    has to fall by 2 %, and none may rise by 2 %.  The covers in a file stand
    here because they alone show what streaming loads cost when every line is
    read by two vectors: 50 MB at k=3, extract with such loads 33.3 us a pass
    against 33.4 us aligned, 40.3 against 37.2 us at byte 54."""
    import statistics

    k, n = new[0]["k"], new[0]["n"]
    views = [[], []]
    for at in (0, 54):
        timer.use(k, n, at)
        times = [([], []) for _ in range(2)]
        for r in range(rounds + 1):
            for pair, (hot, cold) in zip((stored, new), times):
                for e in pair:
                    _install(e["op"], k, n, e["cfg"])
                h = [sum(p) for p in timer.hot(8)]
                c = [sum(p) for p in zip(*(timer.cold(e["op"], 8) for e in pair))]
                if r:
                    hot += h
                    cold += c
        for v, both in zip(views, times):
            v += [statistics.median(t) for t in both]
    old, got = views
    better = sum(got) < 0.98 * sum(old) and all(g < 1.02 * o for g, o in zip(got, old))
    log("k=%d n=%d hot, cold, hot and cold in a file: stored %s us, new %s us -> %s" % (
        k, n, *(" ".join("%.2f" % t for t in v) for v in views), "new" if better else "stored"))
    for e in new if better else stored:
        _install(e["op"], k, n, e["cfg"])
    return new if better else stored


def tune_small(timer: Timer, log=print):
    """One shape per operation for every cover below RUNS_MIN and every k.  A
    kernel takes 4 us there by its own events whatever its shape, to within the
    spread of a measurement, so a choice per size by those would be one by
    noise; what differs, by up to a microsecond, is an embed and waited extract
    issued from C (lsb_roundtrip_latency, 14 to 16 us to a hundredth).  Shapes are
    ranked by its sum over sizes and k, the other operation at the first shape.
    Returns the entries of the largest bucket below RUNS_MIN, which the smaller
    ones share."""
    import ctypes
    import statistics

    import torch

    from . import api
    from ._lib import check

    cands = [c for c in _shapes((0, 1), (0,)) if c["blocks_per_cu"] == 0]
    points = [(n, k) for n in (4096, 49152, 196608, 786432, 1572864) for k in (1, 2, 5)]
    med, low = ctypes.c_double(), ctypes.c_double()
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    entries = []
    for op in (api.OP_EMBED, api.OP_EXTRACT):
        total = [0.0] * len(cands)
        for n, k in points:
            _install(1 - op, k, n, cands[0])
            us = [[] for _ in cands]
            for r in range(4):
                for i, c in enumerate(cands):
                    _install(op, k, n, c)
                    check(timer.lib.lsb_roundtrip_latency(
                        timer.cover.data_ptr(), timer.stego.data_ptr(), n, timer.msg.data_ptr(), n * k // 16, k,
                        timer.out.data_ptr(), 300, ctypes.byref(med), ctypes.byref(low), stream))
                    if r:
                        us[i].append(med.value)
            total = [t + statistics.median(u) / len(points) for t, u in zip(total, us)]
        i = total.index(min(total))
        log("op=%d below %d bytes -> %s, waited pass %.2f us (worst shape %.2f)" % (
            op, RUNS_MIN, list(cands[i].values()), total[i], max(total)))
        n = RUNS_MIN - 1
        entries += [{"op": op, "k": k, "bucket": bucket(n), "n": n, "cfg": cands[i], "us": round(total[i], 2),
                     "method": "waited passes below 2 MB"} for k in KS]
    for e in entries:
        _install(e["op"], e["k"], e["n"], e["cfg"])
    return entries


def tune_plain(reps: int = 4, sizes=SIZES, ks=KS, log=print, stored=()):
    """Entries for every k and size; those in ``stored`` (an earlier table's)
    stay where the new ones are not measurably better."""
    timer = Timer()
    entries = tune_small(timer, log=log)
    old = {(e["op"], e["k"], e["n"]): e for e in stored}
    for n in sizes:
        for k in ks:
            new = tune_pair(timer, k, n, reps=reps, log=log)
            had = [old.get((e["op"], k, n)) for e in new]
            entries += keep_better(timer, had, new, log=log) if all(had) else new
    return entries


def tune_batch(log=print, count: int = 4096):
    """Sweep the batched kernel's launch shapes on the uneven 4096-cover
    workload: embed plans and extract plans are timed separately (GPU events
    around each plan run, best of three after a warm-up) and each keeps its
    own shape; the tile size is the one whose two best shapes sum lowest."""
    import torch

    from . import api, batch
    from .workloads import BatchWorkload

    dev = torch.device("cuda:0")
    wl = BatchWorkload(count, api.capacity, seed=401)
    cover, stego, msg, out = wl.allocate(dev)
    status = torch.zeros(count, dtype=torch.int32, device=dev)
    lens = torch.zeros(count, dtype=torch.int32, device=dev)
    stream = torch.cuda.current_stream()

    def gtime(fn, reps=3):
        best = None
        for r in range(reps + 1):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record(stream)
            fn()
            e1.record(stream)
            torch.cuda.synchronize()
            if r:
                ms = e0.elapsed_time(e1)
                best = ms if best is None else min(best, ms)
        return best

    results = []
    by_tv = {}
    # streaming stores only: the arenas (about 35 GB) are far beyond the cache
    for tv in (512, 1024, 2048, 4096):
        for block in (256, 512, 1024):
            for unroll in (1, 2, 4):
                for bpc in (0, 8):
                    batch.tune_set(block, unroll, bpc, 1, tv)
                    pe = batch.Plan(count, api.OP_EMBED, wl.jobs(api.OP_EMBED))
                    px = batch.Plan(count, api.OP_EXTRACT, wl.jobs(api.OP_EXTRACT))
                    te = gtime(lambda: pe.embed_batch(cover, stego, msg, status))
                    tx = gtime(lambda: px.extract_batch(stego, out, lens, status))
                    pe.close()
                    px.close()
                    cfg = {"block": block, "unroll": unroll, "blocks_per_cu": bpc, "nontemporal": 1}
                    results.append({"cfg": cfg, "tile_vectors": tv, "embed_ms": round(te, 3), "extract_ms": round(tx, 3)})
                    log("batch %s tv=%d -> embed %.3f ms, extract %.3f ms" % (cfg, tv, te, tx))
                    e, x = by_tv.setdefault(tv, [None, None])
                    if e is None or te < e[0]:
                        by_tv[tv][0] = (te, cfg)
                    if x is None or tx < x[0]:
                        by_tv[tv][1] = (tx, cfg)
    assert bool((status == 0).all()) and torch.equal(out, msg), "the sweep's last runs lost messages"
    tv = min(by_tv, key=lambda t: by_tv[t][0][0] + by_tv[t][1][0])
    (te, ce), (tx, cx) = by_tv[tv]
    return {"cfg": ce, "extract_cfg": cx, "tile_vectors": tv, "embed_ms": round(te, 3),
            "extract_ms": round(tx, 3)}, results


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--reps", type=int, default=4)
    ap.add_argument("--batch", action="store_true", help="also sweep the batched kernel")
    ap.add_argument("--batch-only", action="store_true",
                    help="sweep the batched kernel only; the stored plain-kernel entries stay")
    ap.add_argument("--small-only", action="store_true", help="re-choose the shapes of covers below 2 MB only")
    ap.add_argument("--below", type=int, default=0,
                    help="re-choose the plain kernels' shapes of covers below this size only")
    ap.add_argument("--sequence-only", action="store_true",
                    help="re-choose the large-image workload's six launch shapes inside their sequence only")
    ap.add_argument("--out", default=TABLE)
    args = ap.parse_args()
    import torch

    log = lambda *a: print(*a, file=sys.stderr, flush=True)  # noqa: E731
    if args.sequence_only:
        with open(TABLE) as f:
            table = json.load(f)
        seq = {(e["op"], e["k"], e["bucket"]): e for e in tune_sequence(log=log)}
        table["entries"] = [seq.get((e["op"], e["k"], e["bucket"]), e) for e in table["entries"]]
        with open(args.out, "w") as f:
            json.dump(table, f, indent=1)
        log("wrote", args.out)
        return
    if args.batch_only:
        with open(TABLE) as f:
            table = json.load(f)
        table["batch"], table["batch_sweep"] = tune_batch(log=log)
        with open(args.out, "w") as f:
            json.dump(table, f, indent=1)
        log("wrote", args.out)
        return
    if args.small_only:
        with open(TABLE) as f:
            table = json.load(f)
        table["entries"] = tune_small(Timer(1 << 28), log=log) + [e for e in table["entries"] if e["n"] >= RUNS_MIN]
        with open(args.out, "w") as f:
            json.dump(table, f, indent=1)
        log("wrote", args.out)
        return
    if args.below:
        with open(TABLE) as f:
            table = json.load(f)
        kept = [e for e in table["entries"] if e["n"] >= args.below]
        table["entries"] = tune_plain(args.reps, [n for n in SIZES if n < args.below], log=log,
                                      stored=table["entries"]) + kept
        with open(args.out, "w") as f:
            json.dump(table, f, indent=1)
        log("wrote", args.out)
        return
    entries = tune_plain(args.reps, log=log)
    # the large-image workload's launches are chosen inside its own sequence
    seq = {(e["op"], e["k"], e["bucket"]): e for e in tune_sequence(log=log)}
    entries = [seq.get((e["op"], e["k"], e["bucket"]), e) for e in entries]
    table = {"arch": "gfx950", "device": torch.cuda.get_device_name(0), "created": time.strftime("%Y-%m-%d %H:%M"),
             "entries": entries}
    if args.batch:
        table["batch"], table["batch_sweep"] = tune_batch(log=log)
    elif os.path.exists(args.out):
        with open(args.out) as f:
            old = json.load(f)
        if "batch" in old:
            table["batch"] = old["batch"]
    with open(args.out, "w") as f:
        json.dump(table, f, indent=1)
    log("wrote", args.out)


if __name__ == "__main__":
    main()
