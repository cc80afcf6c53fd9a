"""The work that programs have this library do, case by case: the calls of
paper_2411_01964_amd.esq and .scan over the sizes, positions and options that
the tests, the benchmark and the server use, from windows of a few thousand n
to the paper's own chunks below 2^50.

A case is a dict of plain values:
  call     "verify" (verify_range), "scan" (scan.scan), "sieve"
           (sieve_segment), "batch" (verify_batch), "prepared" (PreparedBatch)
  at_log2  the intervals end below 2^at_log2, at a place drawn from the seed
  n        odd numbers per interval (verify, sieve) or per chunk (scan)
  and the options of the call.
"""
import math
import random

import numpy as np
import torch

from paper_2411_01964_amd import esq, scan, workloads

MAX_HI = (1 << 50) + (1 << 32)

# 32-bit operations per odd n that a bit-parallel search needs: an AND and a
# popcount per step and 32-n word, 2.928 steps expected per 64-n word.
OPS_PER_N = 4 * 2.928 / 64


def listed():
    return [
        # a window around one n, asked for by hand or by the smallest requests
        # of the served stream (2^12 n): all latency
        {"name": "window_per_n", "call": "verify", "at_log2": 50, "n": 5003, "per_n": True},
        # a short interval from a loop that may not allocate, aggregates only
        {"name": "short_noalloc", "call": "verify", "at_log2": 40, "n": 65537, "noalloc": True},
        # as many n as lie below 2^22 (the smallest workload of the benchmark), per-n output
        {"name": "per_n_2pow21", "call": "verify", "at_log2": 23, "n": (1 << 21) - 1, "per_n": True},
        # an ordinary ragged interval, aggregates only
        {"name": "ordinary_100M", "call": "verify", "at_log2": 46, "n": 100000007},
        # one contiguous interval of 2^31 odd n below 2^40: the benchmark's second workload
        {"name": "long_2pow31", "call": "verify", "at_log2": 40, "n": 1 << 31},
        # the paper's run over consecutive intervals, the benchmark's headline
        # interval of 2^33 odd n as the chunk, next to the bound 2^50
        {"name": "scan_4x2pow33", "call": "scan", "at_log2": 50, "n": 1 << 33, "chunks": 4},
        # least k of every n of a long interval, 2 GiB of bytes to memory
        {"name": "per_n_2pow31", "call": "verify", "at_log2": 50, "n": 1 << 31, "per_n": True},
        # a bounded search that lists the n it leaves (Algorithm 2's k_max and report)
        {"name": "kmax_exceptions", "call": "verify", "at_log2": 44, "n": (1 << 24) + 77, "kmax": 4,
         "exceptions_cap": 4096},
        # what the server admits at once: requests of uneven length, per-n output
        {"name": "batch_per_n_24", "call": "batch", "at_log2": 50, "count": 24, "len_log2": 24, "per_n": True},
        # the benchmark's batch workload: uneven intervals, planned once, replayed as a graph
        {"name": "prepared_1024", "call": "prepared", "at_log2": 50, "count": 1024, "len_log2": 28},
        # squarefree flags of a short stretch at an odd place
        {"name": "sieve_1M", "call": "sieve", "at_log2": 40, "n": (1 << 20) + 13},
        # squarefree flags of the headline interval, 1 GiB of bits to memory
        {"name": "sieve_2pow33", "call": "sieve", "at_log2": 50, "n": 1 << 33},
    ]


def _size(rng, a, b):
    """A size log-uniform in [2^a, 2^b], odd three times out of four."""
    n = int(2.0 ** rng.uniform(a, b))
    return n | 1 if rng.random() < 0.75 else n


def draw(rng):
    call = rng.choice(["verify", "verify", "verify", "verify", "scan", "sieve", "sieve", "batch", "prepared"])
    if call == "verify":
        per_n = rng.random() < 0.5
        n = _size(rng, 10, 30 if per_n else 33)
        c = {"call": call, "at_log2": rng.randint(max(23, n.bit_length() + 2), 50), "n": n}
        if per_n:
            c["per_n"] = True
        if rng.random() < 0.25:
            c["kmax"] = rng.randint(3, 6)
            if n < 1 << 26:
                c["exceptions_cap"] = rng.choice([16, 1000, 4096])
        elif rng.random() < 0.25:
            c["noalloc"] = True
        return c
    if call == "scan":
        n = _size(rng, 20, 33)
        return {"call": call, "at_log2": rng.randint(n.bit_length() + 4, 50), "n": n, "chunks": rng.randint(2, 4)}
    if call == "sieve":
        n = _size(rng, 12, 33)
        return {"call": call, "at_log2": rng.randint(max(23, n.bit_length() + 2), 50), "n": n}
    if call == "batch":
        return {"call": call, "at_log2": rng.randint(40, 50), "count": rng.randint(2, 30),
                "len_log2": rng.randint(16, 26), "per_n": rng.random() < 0.5}
    return {"call": call, "at_log2": rng.randint(40, 50), "count": rng.randint(33, 1024), "len_log2": rng.randint(20, 28)}


def _intervals(case, seed):
    """The intervals [lo, hi) of a case: their places from the seed, their
    lengths (so the shapes of the outputs) from the case."""
    rng = random.Random(seed)
    top = 1 << case["at_log2"]
    if "count" in case:
        shortest = 12 if case["call"] == "batch" else 16
        lo, hi = workloads.batch_intervals(seed=case["count"], count=case["count"],
                                           log2_len=(shortest, case["len_log2"]))
        starts = [rng.randrange(top >> 2, top - (2 << case["len_log2"])) | 1 for _ in lo]
        return [(s, s + b - a) for s, a, b in zip(starts, lo, hi)]
    span = 2 * case["n"] * case.get("chunks", 1)
    lo = rng.randrange(top // 2 - span // 2, top - span) | 1
    return [(lo, lo + span)]


def prepare(case, seed):
    esq.init(0, MAX_HI)
    ivs = _intervals(case, seed)
    state = {"case": case, "ivs": ivs}
    if case["call"] == "sieve":
        state["out"] = torch.empty((case["n"] + 63) // 64, dtype=torch.int64, device="cuda")
    elif case["call"] == "prepared":
        state["batch"] = esq.PreparedBatch([a for a, _ in ivs], [b for _, b in ivs])
        state["batch"].records.zero_()  # only the first n_records of an interval are written
    return state


def _numbers(results, exceptions_cap=0):
    """The aggregates of a list of results as arrays, the records and the
    listed exceptions in rows of the capacity that they were asked with."""
    out = {k: np.array([r[k] for r in results], dtype=np.int64)
           for k in ("n0", "n_odd", "hist", "ksum", "kmax_seen", "n_exceptions", "status")}
    out["records"] = np.zeros((len(results), esq.ESQ_RECORDS_CAP, 2), dtype=np.int64)
    out["exceptions"] = np.zeros((len(results), exceptions_cap), dtype=np.int64)
    for i, r in enumerate(results):
        out["records"][i, :len(r["records"])] = r["records"]
        if exceptions_cap:
            out["exceptions"][i, :len(r["exceptions"])] = r["exceptions"]
    return out


def run(state):
    case, ivs = state["case"], state["ivs"]
    lo, hi = ivs[0]
    if case["call"] == "sieve":
        return esq.sieve_segment(lo, hi, out=state["out"])
    if case["call"] == "prepared":
        b = state["batch"]
        b.launch(graph=True)
        return {"summaries": b.summaries, "records": b.records}
    if case["call"] == "scan":
        return _numbers([scan.scan(lo, hi, chunk=2 * case["n"])])
    if case["call"] == "batch":
        rs = esq.verify_batch([a for a, _ in ivs], [b for _, b in ivs],
                              per_n=[True] * len(ivs) if case["per_n"] else None)
        out = _numbers(rs)
        if case["per_n"]:
            out["per_n"] = [r["per_n"] for r in rs]
        return out
    r = esq.verify_range(lo, hi, kmax=case.get("kmax", 0), per_n=case.get("per_n", False),
                         exceptions_cap=case.get("exceptions_cap", 0), noalloc=case.get("noalloc", False))
    out = _numbers([r], case.get("exceptions_cap", 0))
    if case.get("per_n"):
        out["per_n"] = r["per_n"]
    return out


def work(case):
    """Bytes that have to reach memory, and the search's 32-bit operations (one
    per odd number and 32-bit word for the sieve alone)."""
    if "count" in case:
        n, calls = sum((b - a) // 2 for a, b in _intervals(case, 0)), case["count"]
    else:
        n, calls = case["n"] * case.get("chunks", 1), case.get("chunks", 1)
    if case["call"] == "sieve":
        return {"bytes": (n + 63) // 64 * 8, "flops": n / 32}
    return {"bytes": (n if case.get("per_n") else 0) + calls * (esq.SUMMARY_BYTES + esq.RECORD_BYTES),
            "flops": OPS_PER_N * n}


# ------------------------------------------------- the same numbers in plain numpy

def _squarefree(m0, count, primes):
    """Squarefree flags of the odd m0, m0 + 2, ... (count of them, m0 > 0)."""
    flags = np.ones(count, dtype=bool)
    q = primes.astype(np.int64) ** 2
    q = q[q <= m0 + 2 * (count - 1)]
    # first odd multiple of q at or above m0
    first = (-(-m0 // q)) | 1
    at = (first * q - m0) // 2
    few = at + q >= count
    flags[at[few & (at < count)]] = False
    for a, s in zip(at[~few].tolist(), q[~few].tolist()):
        flags[a::s] = False
    return flags


def _primes(limit):
    odd = np.ones(limit // 2 + 1, dtype=bool)  # odd[i]: 2i + 1
    odd[0] = False
    for p in range(3, math.isqrt(limit) + 1, 2):
        if odd[p // 2]:
            odd[p * p // 2::p] = False
    p = 2 * np.nonzero(odd)[0] + 1
    return p[p <= limit]


def _verify(lo, hi, kmax, primes):
    n0 = max(lo, 3) | 1
    count = (hi - n0 + 1) // 2
    n = n0 + 2 * np.arange(count, dtype=np.int64)
    least = np.zeros(count, dtype=np.int64)
    left = np.arange(count)
    for k in range(1, (kmax or 20) + 1):
        if not left.size:
            break
        m = n[left] - (1 << k)
        keep = m > 0
        if left.size > 8:
            a = max(1, n0 - (1 << k)) | 1
            f = _squarefree(a, (int(n[-1]) - (1 << k) - a) // 2 + 1, primes)
            ok = np.zeros(left.size, dtype=bool)
            ok[keep] = f[(m[keep] - a) // 2]
        else:
            q = primes.astype(np.int64) ** 2
            ok = np.array([x > 0 and not (x % q[q <= x] == 0).any() for x in m.tolist()], dtype=bool)
        least[left[ok]] = k
        left = left[~ok]
    depth = np.where(least == 0, 1 << 30, least)
    best = np.maximum.accumulate(depth)
    new = np.nonzero(np.concatenate([[True], best[1:] > best[:-1]]))[0]
    return {"n0": n0, "n_odd": count, "hist": np.bincount(least, minlength=65).tolist(), "ksum": int(least.sum()),
            "kmax_seen": int(least.max()), "n_exceptions": int(left.size), "status": 0,
            "records": [(int(n[i]), int(least[i])) for i in new], "exceptions": n[left], "per_n": least}


def exact(case, seed):
    if case["call"] not in ("verify", "sieve") or case["n"] > 1 << 22:
        return None
    (lo, hi), = _intervals(case, seed)
    primes = _primes(math.isqrt(hi) + 1)
    if case["call"] == "sieve":
        m0 = lo | 1
        bits = np.zeros((case["n"] + 63) // 64 * 64, dtype=np.uint8)
        bits[:case["n"]] = _squarefree(m0, case["n"], primes)
        return m0, case["n"], np.packbits(bits, bitorder="little").view(np.int64)
    r = _verify(lo, hi, case.get("kmax", 0), primes)
    r["exceptions"] = r["exceptions"][:case.get("exceptions_cap", 0)]
    out = _numbers([r], case.get("exceptions_cap", 0))
    if case.get("per_n"):
        out["per_n"] = r["per_n"].astype(np.uint8)
    return out
