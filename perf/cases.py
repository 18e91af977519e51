"""Timed cases of the validity-status checker: what a program using libvcheck has it do.

A case is a plain dict: its family (which public entry point it calls), its sizes and its
options.  The listed cases are the sizes the framework is used at; draw() spreads over
the ranges around them: from a few hundred events to the largest trace, one to millions
of variables, odd sizes, given initial statuses, explicit bodies, fewer memory spaces.

Every family goes through the binding in paper_1910_11110_amd.vcheck:

call        a small trace held on the host: load, check, read every result, free
plain       a trace resident on the device, checked; the results stay there
components  access-mode declarations translated into effects and checked
overlap     a trace over overlapping arrays
dynamic     a trace that creates and destroys partial vectors
spaces      a trace over k memory spaces
declared    the well-declaredness check of component programs with explicit bodies
programs    structured programs (While / If), results read to the host
batched     many traces of uneven length checked in one batch
served      streams of chunks through the server, from host memory and back

A program that checks a trace wants to know whether it is clean, so each pass reads the
number of violations and the first one back (which waits for the check); the per-event
statuses, final statuses and violation list are used where they lie on the device.
"""
from __future__ import annotations

import ctypes as C
import math
import time

import numpy as np
import torch

from paper_1910_11110_amd import gen
from paper_1910_11110_amd import vcheck as V

CHUNK = 1 << 16  # events per served chunk

_shared = None


def _context():
    """One stream and one context for the whole process, as a program keeps them."""
    global _shared
    if _shared is None:
        stream = torch.cuda.Stream()
        _shared = (stream, V.Context(0, stream))
    return _shared


def listed():
    return [
        # one small trace from start to end: the latency of the calls themselves
        {"name": "call-10k-64", "family": "call", "n": 10_000, "n_ids": 64, "init": False},
        # an ordinary trace, at sizes that are no multiple of anything
        {"name": "plain-1M-50k", "family": "plain", "n": 1_000_003, "n_ids": 50_021, "init": True},
        # the largest trace over few variables, and over many
        {"name": "plain-2^28-64", "family": "plain", "n": 1 << 28, "n_ids": 64, "init": False},
        {"name": "plain-2^26-2^20", "family": "plain", "n": 1 << 26, "n_ids": 1 << 20, "init": False},
        # the headline workload: declarations of 2^23 components translated and checked
        {"name": "components-2^23", "family": "components", "n_comp": 1 << 23, "n_vars": 1 << 20, "bodies": False,
         "read": False},
        {"name": "overlap-2^24-2^16", "family": "overlap", "n": 1 << 24, "n_ids": 1 << 16},
        {"name": "dynamic-2^23-2^16", "family": "dynamic", "n": 1 << 23, "n_vectors": 1 << 10,
         "n_pvectors": (1 << 16) - (1 << 10)},
        {"name": "spaces-k4-2^26-2^20", "family": "spaces", "n": 1 << 26, "n_ids": 1 << 20, "k": 4, "read": False},
        {"name": "declared-2^18-2^16", "family": "declared", "n_comp": 1 << 18, "n_vars": 1 << 16, "arrays": True,
         "extend": True},
        {"name": "programs-2^18-16", "family": "programs", "n_prog": 1 << 18, "n_vars": 16, "fuel": 4096},
        # mixed traces as they come, a fifth of them over arrays
        {"name": "batched-1024", "family": "batched", "n_traces": 1024, "shape": 1},
        # a burst of streams through the server, copies from and to the host included
        {"name": "served-64", "family": "served", "n_streams": 64, "shape": 1},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    f = rng.choice(["call", "plain", "plain", "components", "overlap", "dynamic", "spaces", "declared", "programs",
                    "batched", "served"])
    if f == "call":
        return {"family": f, "n": _log_int(rng, 100, 1 << 20), "n_ids": _log_int(rng, 1, 1 << 16),
                "init": rng.random() < 0.5}
    if f == "plain":
        few = rng.random() < 0.4
        return {"family": f, "n": _log_int(rng, 1 << 14, (1 << 27) if few else (1 << 25)),
                "n_ids": _log_int(rng, 1, 64) if few else _log_int(rng, 65, 1 << 23), "init": rng.random() < 0.5}
    if f == "components":
        n_comp = _log_int(rng, 1 << 10, 1 << 22)
        return {"family": f, "n_comp": n_comp, "n_vars": _log_int(rng, 16, 1 << 20), "bodies": rng.random() < 0.4,
                "read": n_comp < (1 << 16)}
    if f == "overlap":
        return {"family": f, "n": _log_int(rng, 1 << 14, 1 << 23), "n_ids": _log_int(rng, 64, 1 << 16)}
    if f == "dynamic":
        nv = _log_int(rng, 4, 1 << 10)
        n = _log_int(rng, 1 << 15, 1 << 22)
        return {"family": f, "n": n, "n_vectors": nv,
                "n_pvectors": min(n // 4, nv * rng.randint(1, 48) + rng.randint(0, 9))}
    if f == "spaces":
        n = _log_int(rng, 1 << 14, 1 << 25)
        return {"family": f, "n": n, "n_ids": _log_int(rng, 8, 1 << 22), "k": rng.choice([2, 3, 4]),
                "read": n < (1 << 20)}
    if f == "declared":
        arrays = rng.random() < 0.7
        return {"family": f, "n_comp": _log_int(rng, 1 << 8, 1 << 17), "n_vars": _log_int(rng, 16, 1 << 16),
                "arrays": arrays, "extend": arrays and rng.random() < 0.5}
    if f == "programs":
        return {"family": f, "n_prog": _log_int(rng, 64, 1 << 17), "n_vars": rng.randint(1, 64),
                "fuel": _log_int(rng, 64, 8192)}
    if f == "batched":
        return {"family": f, "n_traces": _log_int(rng, 2, 512), "shape": rng.randrange(1 << 20)}
    return {"family": f, "n_streams": _log_int(rng, 1, 64), "shape": rng.randrange(1 << 20)}


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
def _rng(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _ints(g, lo, hi, n):
    return torch.randint(lo, hi, (n,), generator=g, device="cuda", dtype=torch.int32)


def _plain_events(g, n, n_ids):
    """Variable uniform, op uniform over r, w, Push, Pull, Noop, side fair."""
    e = _ints(g, 0, 5, n) << 24
    e |= _ints(g, 0, 2, n) << 27
    e |= _ints(g, 0, n_ids, n)
    return e


def _init(g, n_ids, hi=4):
    return torch.randint(1, hi, (n_ids,), generator=g, device="cuda", dtype=torch.int32).to(torch.uint8)


def _space_events(g, n, n_ids, k):
    op = _ints(g, 0, 4, n)
    e = op << 24
    a = _ints(g, 0, k, n)
    e |= torch.where(op == 3, 0, a) << 26
    b = _ints(g, 0, k, n)
    e |= torch.where(op == 2, b, 0) << 28
    e |= _ints(g, 0, n_ids, n)
    return e


def _components(g, n_comp, n_vars, kmax=8, s=1.1):
    """1 to kmax distinct Zipf(s) variables a component, as many of each, R/W/RW in shares of
    0.5/0.3/0.2 (so the sizes follow from the case), one side a component: component
    offsets (int64) and declaration words (int32)."""
    kmax = min(kmax, n_vars)
    cdf = torch.arange(1, n_vars + 1, device="cuda", dtype=torch.float64).pow_(-s).cumsum(0)
    cdf /= cdf[-1].clone()

    def zipf(n):
        u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
        return torch.searchsorted(cdf, u, right=True).clamp_(max=n_vars - 1).to(torch.int32)

    k = torch.randperm(n_comp, generator=g, device="cuda", dtype=torch.int32) % kmax + 1
    ids = zipf(n_comp * kmax).view(n_comp, kmax)
    for j in range(1, kmax):  # a repeated variable is drawn again until distinct
        rows = torch.nonzero(k > j).flatten()
        while rows.numel():
            rows = rows[(ids[rows, :j] == ids[rows, j:j + 1]).any(1)]
            if rows.numel():
                ids[rows, j] = zipf(rows.numel())
    keep = torch.arange(kmax, device="cuda")[None, :] < k[:, None]
    var = ids[keep]
    u = torch.randperm(var.numel(), generator=g, device="cuda", dtype=torch.int32) % 10
    mode = (u >= 5).to(torch.int32) + (u >= 8).to(torch.int32)
    side = torch.repeat_interleave(_ints(g, 0, 2, n_comp), k)
    off = torch.zeros(n_comp + 1, device="cuda", dtype=torch.int64)
    torch.cumsum(k, 0, out=off[1:])
    return off, var | (mode << 24) | (side << 27)


def _bodies(off, decls):
    """Explicit bodies that do what the declarations allow: R reads, W writes, RW reads and
    then writes, on the declaration's side."""
    mode, keep = (decls >> 24) & 3, decls & 0x08FFFFFF
    cnt = 1 + (mode == 2).to(torch.int64)
    end = torch.cumsum(cnt, 0)
    body = torch.empty(int(end[-1]), device="cuda", dtype=torch.int32)
    body[end - cnt] = keep | ((mode == 1).to(torch.int32) << 24)
    rw = mode == 2
    body[(end - 1)[rw]] = keep[rw] | (1 << 24)
    start = torch.zeros(end.numel() + 1, device="cuda", dtype=torch.int64)
    start[1:] = end
    return start[off], body


def _shapes(case):
    return gen.trace_shapes(case.get("n_traces", case.get("n_streams")), case["shape"])


class _OnDevice:
    def __init__(self, trace, ptr, n, kind):
        self.trace = trace  # owns the memory: it lives as long as a view does
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": kind, "data": (ptr, False), "version": 3}


def _view(trace, ptr, n, kind="|u1"):
    """The n values at a device address of the trace's, as a tensor (which keeps the trace)."""
    if not n or not ptr:
        return torch.empty(0, device="cuda", dtype=torch.uint8 if kind == "|u1" else torch.int32)
    return torch.as_tensor(_OnDevice(trace, ptr, n, kind), device="cuda")


# ------------------------------------------------------------------------------------------
# what a program has in hand before the call
# ------------------------------------------------------------------------------------------
def prepare(case, seed):
    f = case["family"]
    stream, ctx = _context()
    s = {"case": case, "ctx": ctx, "stream": stream, "views": None}
    with torch.cuda.stream(stream):
        g = _rng(seed)
        if f == "call":
            s["events"] = _plain_events(g, case["n"], case["n_ids"]).cpu().numpy().view(np.uint32)
            s["init"] = _init(g, case["n_ids"]).cpu().numpy() if case["init"] else None
            s["violations"] = np.zeros(case["n"], np.int32)
        elif f == "plain":
            ev = _plain_events(g, case["n"], case["n_ids"])
            s["trace"] = V.Trace.load(ctx, ev, case["n_ids"], _init(g, case["n_ids"]) if case["init"] else None)
        elif f == "components":
            off, decls = _components(g, case["n_comp"], case["n_vars"])
            boff, body = _bodies(off, decls) if case["bodies"] else (None, None)
            stream.synchronize()
            s["trace"] = V.translate(ctx, off, decls, case["n_vars"], boff, body, check=True)
        elif f == "overlap":
            lo, hi = gen.intervals(case["n_ids"], seed, space=max(1 << 13, 256 * case["n_ids"]))
            s["trace"] = V.Trace.load(ctx, _plain_events(g, case["n"], case["n_ids"]), case["n_ids"])
            s["trace"].set_arrays(lo, hi)
        elif f == "dynamic":
            d = gen.dynamic_trace(case["n"], case["n_vectors"], case["n_pvectors"], seed,
                                  space=case["n_vectors"] << 14)
            s["trace"] = V.Trace.load(ctx, d.events, d.lo.size, lifetimes=True)
            s["trace"].set_dynamic_arrays(d.lo, d.hi, d.mother)
        elif f == "spaces":
            ev = _space_events(g, case["n"], case["n_ids"], case["k"])
            s["trace"] = V.Trace.load_spaces(ctx, ev, case["n_ids"], case["k"])
        elif f == "declared":
            p = gen.declared_program(case["n_comp"], case["n_vars"], seed, arrays=case["arrays"],
                                     space=max(1 << 8, 64 * case["n_vars"]), max_len=64)
            dev = [None if a is None else torch.from_numpy(a.view(np.int64 if a.dtype == np.uint64 else np.int32)).cuda()
                   for a in (p.comp_off, p.decls, p.body_off, p.body, p.idx)]
            stream.synchronize()
            s["trace"] = V.check_declared(ctx, dev[0], dev[1], case["n_vars"], dev[2], dev[3], dev[4], p.lo, p.hi,
                                          extend=case["extend"])
        elif f == "programs":
            p = gen.structured_programs(case["n_prog"], case["n_vars"], seed, n_templates=512)
            s["programs"] = V.Programs(ctx, p.prog_off, p.words, case["n_vars"], p.choice, p.init, case["fuel"])
        elif f == "batched":
            s["traces"] = []
            for i, sh in enumerate(_shapes(case)):
                t = V.Trace.load(ctx, _plain_events(g, sh.length, sh.n_vars), sh.n_vars)
                if sh.has_arrays:
                    t.set_arrays(*gen.intervals(sh.n_vars, seed + i))
                s["traces"].append(t)
        elif f == "served":
            s["streams"] = []
            for i, sh in enumerate(_shapes(case)):
                ev = _plain_events(g, sh.length, sh.n_vars).cpu().numpy().view(np.uint32)
                lo, hi = gen.intervals(sh.n_vars, seed + i) if sh.has_arrays else (None, None)
                s["streams"].append((ev, sh.n_vars, lo, hi))
            s["status"] = np.zeros(sum(e.size for e, *_ in s["streams"]), np.uint8)
            s["server"] = V.Server(V.Context(0), 8 << 30)
        stream.synchronize()
    return s


# ------------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------------
def _results(s, t):
    """The number of violations and the first one, and the results where they lie (the list
    of violations in its whole capacity: zeros follow its end)."""
    total, first = C.c_uint64(), C.c_uint64()
    rc = V.lib().vc_read_violations(t.h, None, 0, C.byref(total), C.byref(first))
    if rc != V.VC_OK:
        raise V.VCError(rc, V.lib().vc_last_error().decode())
    if s["views"] is None:
        n, n_ids = t.info()
        st, fin, viol = t.device_results()
        s["views"] = (_view(t, st, n), _view(t, fin, n_ids) if s["case"]["family"] != "declared" else None,
                      _view(t, viol, n, "<i4"))
        with torch.cuda.stream(s["stream"]):
            s["views"][2][total.value:] = 0
    status, final, viol = s["views"]
    return {"status": status, "final": final, "violations": viol, "total": total.value, "first": first.value}


def _serve(s):
    srv = s["server"]
    opened, at = [], 0
    for ev, n_ids, lo, hi in s["streams"]:
        st = srv.open(n_ids, lo, hi)
        for a in range(0, ev.size, CHUNK):
            b = min(a + CHUNK, ev.size)
            srv.submit(st, ev[a:b], s["status"][at + a:at + b])
        opened.append(st)
        at += ev.size
    left = sum(-(-ev.size // CHUNK) for ev, *_ in s["streams"])
    done = {}
    while left:
        cs = srv.poll()
        for c in cs:
            if c.status != V.VC_OK:
                raise RuntimeError(f"chunk {c.chunk} failed with {c.status}")
            done[(c.stream, c.first_event)] = (c.n_violations, c.first_violation)
        left -= len(cs)
        if not cs:
            time.sleep(0.0001)
    finals = [srv.close_stream(st, x[1]) for st, x in zip(opened, s["streams"])]
    order = {st: i for i, st in enumerate(opened)}
    chunks = [done[k] for k in sorted(done, key=lambda k: (order[k[0]], k[1]))]
    return {"status": s["status"], "final": np.concatenate(finals), "chunks": np.array(chunks, np.uint64).view(np.int64)}


def run(s):
    f = s["case"]["family"]
    if f == "call":
        t = V.Trace.load(s["ctx"], s["events"], s["case"]["n_ids"], s["init"])
        t.check()
        v = t.violations()
        s["violations"][:v.total] = v.indices
        out = {"status": t.status(), "final": t.final(), "violations": s["violations"], "total": v.total,
               "first": v.first}
        t.free()
        return out
    if f == "programs":
        s["programs"].run()
        return [x.view(np.int64) if x.dtype == np.uint64 else x for x in s["programs"].read()]
    if f == "served":
        return _serve(s)
    if f == "batched":
        V.batch_check(s["ctx"], s["traces"])
        if s["views"] is None:
            s["views"] = []
            for t in s["traces"]:
                (n, n_ids), (st, fin, _) = t.info(), t.device_results()
                s["views"].append((_view(t, st, n), _view(t, fin, n_ids)))
        with torch.cuda.stream(s["stream"]):  # the context's stream: after the batch
            return {"status": torch.cat([a for a, _ in s["views"]]), "final": torch.cat([b for _, b in s["views"]])}
    t = s["trace"]
    if f == "components":
        t.rerun()
    else:
        t.check()
    out = _results(s, t)
    if s["case"].get("read"):  # a program of ordinary size takes the whole result to the host
        if f == "components":
            out["events"] = t.events().view(np.int32)
        else:
            out["status16"] = t.status16().view(np.int16)
    return out


# ------------------------------------------------------------------------------------------
# what one pass cannot do without: every input read once, every output written once
# (about 0.15 of the events of a plain trace are violations)
# ------------------------------------------------------------------------------------------
def _plain_bytes(n, n_ids):
    return 4 * n + n + 0.6 * n + n_ids


def work(case):
    f = case["family"]
    if f in ("call", "plain"):
        b = _plain_bytes(case["n"], case["n_ids"])
    elif f == "components":
        kmax = min(8, case["n_vars"])
        decls = case["n_comp"] * (kmax + 1) / 2
        b = 8 * case["n_comp"] + 4 * decls + 5 * 3.1 * decls + 2 * case["n_vars"]
        if case["bodies"]:
            b += 8 * case["n_comp"] + 4 * 1.2 * decls
    elif f == "overlap":
        b = _plain_bytes(case["n"], case["n_ids"]) + 8 * case["n_ids"]
    elif f == "dynamic":
        ids = case["n_vectors"] + case["n_pvectors"]
        b = _plain_bytes(case["n"], ids) + 12 * ids
    elif f == "spaces":
        b = 4 * case["n"] + 2 * case["n"] + 1.4 * case["n"] + case["n_ids"]
    elif f == "declared":
        decls = 2.5 * case["n_comp"]
        body = decls * 0.8 * (14 if case["arrays"] else 1)
        b = 16 * case["n_comp"] + 4 * decls + (8 if case["arrays"] else 4) * body + case["n_comp"]
        b += 8 * case["n_vars"] if case["arrays"] else 0
    elif f == "programs":
        b = case["n_prog"] * (4 * 60 + 8 + 8 + 33 + 2 * case["n_vars"])
    else:
        b = sum(_plain_bytes(sh.length, sh.n_vars) for sh in _shapes(case))
    return {"bytes": float(b), "flops": 0.0}


def exact(case, seed):
    """Every output is a whole number (statuses, flags, indices, counts): equal or wrong,
    so there is no value in 64 bits to be near to."""
    return None
