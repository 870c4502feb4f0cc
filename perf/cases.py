"""Performance cases of the RANLUX++ library: what a user's program has it do,
through the package's public calls, from single small draws to gigabytes.

A case is a dict of plain values; its `kind` names the call:

  draw    n records of one luxury level p draw `count` values of type `out`
          each (rlx.generate_*).  `seed_each` re-seeds the records first, as
          the repository's benchmark step does.  `start`: how many values the
          records have drawn before (0: fresh from the seed), `ragged`: every
          record its own number below `start`, so positions inside a step
          differ.  `keep`: the program keeps its output tensor.
  levels  the same for records of several luxury levels in one call.
  skip    n records jump ahead, each by its own number of generator steps
          (log-uniform over 64 bits) or all by one number.
  seed    n records are seeded, from given 64-bit ids or an id range.
  batch   a kept Plan over n requests with uneven counts and mixed levels;
          `replan` updates it with the pass's requests first, as a server
          does for every batch.

Uniform values, integers and records are exact; normals are computed.
"""
import functools

import numpy as np
import torch

import paper_2106_02504_amd as rlx

LEVELS = (24, 218, 404, 794, 2048)
STEP_OPS = 2 * 73 * 73          # a 576-bit product by a constant on 8-bit digits
MULMOD_OPS = 2 * 72 * 72        # a 576-bit product of two variables
RECORD = 80                     # bytes of a stream record

OUT_TYPES = {"f64": torch.float64, "u64": torch.int64, "f32": torch.float32, "normal": torch.float64}
CALLS = {"f64": rlx.generate_f64, "u64": rlx.generate_u64, "f32": rlx.generate_f32,
         "normal": rlx.generate_normal_f64}


def listed():
    return [
        # a host loop that fetches a few numbers for a few streams at a time:
        # latency of one call
        dict(name="small_call", kind="draw", n=64, count=100, p=2048, out="f64", start=0, ragged=False,
             seed_each=False, keep=False),
        # one generator filling one long array: the repository's single-stream
        # workload
        dict(name="single_stream", kind="draw", n=1, count=1 << 20, p=2048, out="f64", start=0, ragged=False,
             seed_each=False, keep=True),
        # one stream per particle or path, two steps' worth of numbers at a
        # time: the many-thread use with few draws per call
        dict(name="few_draws", kind="draw", n=1 << 19, count=24, p=2048, out="f64", start=0, ragged=False,
             seed_each=False, keep=True),
        # a simulation's worth of streams in mid-sequence, odd counts, raw
        # 48-bit integers
        dict(name="ragged_u64", kind="draw", n=5000, count=1001, p=404, out="u64", start=12000, ragged=True,
             seed_each=False, keep=True),
        # the repository's headline workload: seeding and 2^28 doubles
        dict(name="many_streams", kind="draw", n=65536, count=4096, p=2048, out="f64", start=0, ragged=False,
             seed_each=True, keep=True),
        # standard normals for a Monte Carlo batch
        dict(name="normals", kind="draw", n=16384, count=1000, p=2048, out="normal", start=0, ragged=False,
             seed_each=False, keep=True),
        # single-precision numbers for a network's noise or dropout masks
        dict(name="f32", kind="draw", n=32768, count=2048, p=794, out="f32", start=0, ragged=False,
             seed_each=False, keep=True),
        # streams of several luxury levels side by side, in no order
        dict(name="mixed_levels", kind="levels", n=8192, count=1000, p=0, out="f64", start=1200, ragged=False,
             seed_each=False, keep=True),
        # jumping streams apart: the repository's skip workload
        dict(name="skip_ahead", kind="skip", n=1 << 20, p=2048, per_record=True),
        # seeding from 64-bit ids such as event or hash numbers
        dict(name="seed_ids", kind="seed", n=1 << 18, p=2048, ids=True),
        # the repository's batch workload through a kept plan
        dict(name="batch", kind="batch", n=8192, max_draws=1 << 20, replan=False),
        # a server's small batch: plan, upload and draw
        dict(name="serve_batch", kind="batch", n=256, max_draws=1 << 16, replan=True),
    ]


def _log(rng, lo, hi):
    """An integer log-uniform in [lo, hi]."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _total(rng, n, lo, hi, most):
    """A count log-uniform in [lo, hi] with n * count <= most."""
    return _log(rng, lo, max(lo, min(hi, most // n)))


def draw(rng):
    kind = rng.choice(("small", "single", "few", "many", "many", "normal", "levels", "skip", "seed", "batch",
                       "serve"))
    p = rng.choice(LEVELS)
    if kind == "skip":
        return dict(kind="skip", n=_log(rng, 1 << 10, 1 << 20), p=p, per_record=rng.random() < 0.6)
    if kind == "seed":
        return dict(kind="seed", n=_log(rng, 1 << 10, 1 << 20), p=p, ids=rng.random() < 0.6)
    if kind == "batch":
        return dict(kind="batch", n=_log(rng, 256, 8192), max_draws=1 << rng.randint(14, 20), replan=False)
    if kind == "serve":
        return dict(kind="batch", n=_log(rng, 8, 1024), max_draws=1 << rng.randint(10, 18), replan=True)
    out = rng.choice(("f64", "f64", "u64", "f32", "normal"))
    most = 1 << 26
    if kind == "small":
        n = _log(rng, 1, 1024)
        count = _total(rng, n, 2, 4096, 1 << 18)
    elif kind == "single":
        n = _log(rng, 1, 64)
        count = _total(rng, n, 1 << 14, 1 << 22, most)
    elif kind == "few":
        n = _log(rng, 1 << 15, 1 << 20)
        count = _total(rng, n, 2, 250, 1 << 25)
    elif kind == "normal":
        out = "normal"
        n = _log(rng, 1 << 10, 1 << 16)
        count = _total(rng, n, 250, 4096, most)
    else:  # many, levels
        n = _log(rng, 1 << 10, 1 << 16)
        count = _total(rng, n, 250, 4096, most)
    if out == "f32":
        count += count & 1
    start = rng.choice((0, 0, _log(rng, 1, 100000)))
    case = dict(kind="draw", n=n, count=count, p=p, out=out, start=start,
                ragged=start > 0 and rng.random() < 0.5, seed_each=False, keep=kind != "small")
    if kind == "levels":
        case.update(kind="levels", p=0)
    elif kind == "many" and start == 0:
        case["seed_each"] = rng.random() < 0.5
    return case


def _inputs(case, seed):
    """Host arrays that fix the case's inputs: made from the seed alone."""
    rng = np.random.Generator(np.random.PCG64([seed, case["n"]]))
    n, kind = case["n"], case["kind"]
    d = {"id0": int(rng.integers(0, 1 << 40))}
    if kind in ("draw", "levels"):
        d["drawn"] = (rng.integers(0, case["start"] + 1, size=n) if case["ragged"]
                      else np.full(n, case["start"])).astype(np.int64)
        d["level"] = (rng.integers(0, len(LEVELS), size=n) if kind == "levels"
                      else np.full(n, LEVELS.index(case["p"])))
    elif kind == "skip":
        bits = rng.integers(0, 64, size=n if case["per_record"] else 1)
        low = rng.integers(0, 1 << 63, size=bits.size, dtype=np.uint64) << np.uint64(1)
        d["steps"] = (low | np.uint64(1 << 63)) >> bits.astype(np.uint64)
    elif kind == "seed":
        d["ids"] = rng.integers(0, np.iinfo(np.uint64).max, size=n, dtype=np.uint64, endpoint=True)
    else:
        # log-uniform sizes: the same ones for every seed, in another order
        lg = np.log2(case["max_draws"])
        sizes = np.floor(np.exp2(lg * (np.arange(n) + 0.5) / n)).astype(np.int64)
        d["count"] = rng.permutation(sizes)
        d["level"] = rng.integers(0, len(LEVELS), size=n)
        d["start"] = rng.integers(0, 1 << 20, size=n) if case["replan"] else np.zeros(n, dtype=np.int64)
    return d


def _records(id0, level):
    """Records of ids id0, id0 + 1, ..., record i at luxury level level[i]."""
    states = rlx.new_states(level.size)
    for k, p in enumerate(LEVELS):
        at = np.flatnonzero(level == k)
        if at.size:
            ids = torch.from_numpy((id0 + at).astype(np.int64)).cuda()
            states[torch.from_numpy(at).cuda()] = rlx.init_streams(rlx.new_states(at.size), p, ids=ids)
    return states


def prepare(case, seed):
    d, kind, n = _inputs(case, seed), case["kind"], case["n"]
    s = {"case": case}
    if kind in ("draw", "levels"):
        s["id0"] = d["id0"]
        s["states"] = _records(d["id0"], d["level"])
        if case["start"]:
            rlx.skip_values(s["states"], torch.from_numpy(d["drawn"]).cuda(),
                            rlx.P_RECORD if kind == "levels" else case["p"])
        s["out"] = (torch.empty((n, case["count"]), dtype=OUT_TYPES[case["out"]], device="cuda")
                    if case["keep"] else None)
    elif kind == "skip":
        s["states"] = rlx.init_streams(rlx.new_states(n), case["p"], id0=d["id0"])
        s["steps"] = (torch.from_numpy(d["steps"].view(np.int64)).cuda() if case["per_record"]
                      else int(d["steps"][0]))
    elif kind == "seed":
        rlx.prepare(case["p"])
        s["states"] = rlx.new_states(n)
        s["id0"] = d["id0"]
        s["ids"] = torch.from_numpy(d["ids"].view(np.int64)).cuda() if case["ids"] else None
    else:
        s["states"] = _records(d["id0"], d["level"])
        s["requests"] = rlx.requests_array(np.arange(n), d["start"], d["count"], np.array(LEVELS)[d["level"]])
        s["plan"] = rlx.Plan(s["requests"], lanes=64, seg_blocks=4096)
        s["out"] = torch.empty(int(d["count"].sum()), dtype=torch.float64, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind in ("draw", "levels"):
        p = rlx.P_RECORD if kind == "levels" else case["p"]
        if case["seed_each"]:
            rlx.init_streams(s["states"], p, id0=s["id0"])
        return CALLS[case["out"]](s["states"], case["count"], p, out=s["out"]), s["states"]
    if kind == "skip":
        return rlx.skip(s["states"], s["steps"], case["p"])
    if kind == "seed":
        return rlx.init_streams(s["states"], case["p"], ids=s["ids"], id0=0 if case["ids"] else s["id0"])
    if case["replan"]:
        s["plan"].update(s["requests"])
    return s["plan"].generate_f64(s["states"], s["out"])


def work(case):
    """Inputs read and outputs written once; the products by a constant that
    the numbers need (one per 12 values), or for jumps and seeds one product
    of two variables per non-zero 16-bit digit."""
    kind, n = case["kind"], case["n"]
    if kind in ("draw", "levels"):
        size = 4 if case["out"] == "f32" else 8
        steps = n * case["count"] / (24 if case["out"] == "f32" else 12)
        return {"bytes": n * case["count"] * size + (RECORD if case["seed_each"] else 2 * RECORD) * n,
                "flops": steps * STEP_OPS}
    if kind == "skip":
        return {"bytes": (2 * RECORD + (8 if case["per_record"] else 0)) * n,
                "flops": n * MULMOD_OPS * (2.5 if case["per_record"] else 1)}
    if kind == "seed":
        return {"bytes": (RECORD + (8 if case["ids"] else 0)) * n, "flops": n * MULMOD_OPS * (3 if case["ids"] else 2)}
    mean = float((case["max_draws"] - 1) / np.log(case["max_draws"]))
    return {"bytes": n * (mean * 8 + RECORD + 48), "flops": n * mean / 12 * STEP_OPS}


# ---------------------------------------------------------------------------
# the same results in plain Python integers and numpy

M = 2**576 - 2**240 + 1
A = M - (M - 1) // 2**24        # one subtract-with-borrow step as a multiplier


@functools.lru_cache(None)
def _power(e):
    return pow(A, e, M)


def _state(ident, level, drawn=0):
    """(X, pos, p) of the stream of seed `ident` after `drawn` values."""
    p = LEVELS[level]
    return pow(A, p * ((ident << 96) + drawn // 12), M), drawn % 12, p


def _fields(x, pos, p, count):
    """`count` 48-bit fields from the state on, as uint64, and (X, pos) after."""
    mult = _power(p)
    blob = bytearray()
    for _ in range((pos + count + 11) // 12):
        blob += ((x << 576) // M).to_bytes(72, "little")
        last, x = x, x * mult % M
    if (pos + count) % 12:
        x = last
    b = np.frombuffer(bytes(blob), dtype=np.uint8).reshape(-1, 6)
    v = np.zeros((b.shape[0], 8), dtype=np.uint8)
    v[:, :6] = b
    return v.view("<u8").reshape(-1), x, (pos + count) % 12


def _values(v, pos, count, out):
    """Output values at positions pos .. pos + count of a row of fields."""
    if out == "u64":
        return v[pos:pos + count].astype(np.int64)
    if out == "f64":
        return v[pos:pos + count] * 2.0**-48
    if out == "f32":
        both = np.stack((v & np.uint64(0xFFFFFF), v >> np.uint64(24)), axis=1).reshape(-1)
        return both[2 * pos:2 * (pos + count)] * 2.0**-24
    u1, t = v[0::2] * 2.0**-48, v[1::2] * 2.0**-46
    r = np.sqrt(-2.0 * np.log1p(-u1))
    j = np.rint(t)                                   # whole quarter turns
    phi = (t - j) * (np.pi / 2)
    q = j.astype(np.int64) % 4
    c, s = np.cos(phi), np.sin(phi)
    co = np.choose(q, (c, -s, -c, s))
    si = np.choose(q, (s, c, -s, -c))
    return np.stack((r * co, r * si), axis=1).reshape(-1)[pos:pos + count]


def _record_rows(states):
    return np.frombuffer(b"".join(x.to_bytes(72, "little") + (pos | p << 32).to_bytes(8, "little")
                                  for x, pos, p in states), dtype="<i8").reshape(-1, 10)


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    d = _inputs(case, seed)
    if kind in ("draw", "levels"):
        per = case["count"] // 2 if case["out"] == "f32" else case["count"]
        if n * (per + 12) > 40_000_000 or n > (1 << 19):
            return None
        rows, after = [], []
        for i in range(n):
            if i and kind == "draw":    # consecutive ids are 2^96 steps apart
                seeded = seeded * apart % M
                p, pos = case["p"], int(d["drawn"][i]) % 12
                x = seeded * _power(p * (int(d["drawn"][i]) // 12)) % M
            else:
                x, pos, p = _state(d["id0"] + i, int(d["level"][i]), int(d["drawn"][i]))
                seeded, apart = _state(d["id0"] + i, int(d["level"][i]))[0], _power(p << 96)
            v, x, end = _fields(x, pos, p, per)
            rows.append(_values(v, pos, per, case["out"]))
            after.append((x, end, p))
        return np.stack(rows), _record_rows(after)
    if n > 40_000:
        return None
    level = LEVELS.index(case["p"]) if kind in ("skip", "seed") else None
    if kind == "skip":
        steps = np.broadcast_to(d["steps"], (n,))
        return _record_rows([_state(d["id0"] + i, level, 12 * int(steps[i])) for i in range(n)])
    if kind == "seed":
        return _record_rows([_state(int(d["ids"][i]) if case["ids"] else d["id0"] + i, level) for i in range(n)])
    if int(d["count"].sum()) + 12 * n > 30_000_000:
        return None
    parts = []
    for i in range(n):
        first, count = int(d["start"][i]), int(d["count"][i])
        x, pos, p = _state(d["id0"] + i, int(d["level"][i]), first)
        parts.append(_values(_fields(x, pos, p, count)[0], pos, count, "f64"))
    return np.concatenate(parts)
