"""The work that programs have this library do, as cases that can be timed.

A case is a dict of plain values.  `listed` gives the fixed ones, `draw` more of
the same ranges, `prepare` what a program holds before the call (operands on the
GPU, a batch descriptor, a server), `run` one pass through the public entry
points, `work` the bytes and operations a pass cannot do without, and `exact`
the same results from plain 64-bit integer arithmetic in torch.

Kinds of work:
  single     one circular convolution (conv_circular)
  batch      convolutions of one length, back to back (conv_batched)
  uneven     convolutions of many power-of-two lengths in one call (conv_batched)
  transform  a batch of rows forward and a batch of spectra back
             (ntt_forward, ntt_inverse)
  crt        exact integer convolutions by two primes (conv_crt)
  deconv     exact deconvolution of rows (deconvolve)
  conv2d     one two-dimensional convolution (conv2d)
  served     a burst of host requests of mixed lengths through the library's
             own scheduler (NativeConvServer)
"""
import math

import numpy as np
import torch

import paper_1005_1497_amd as nt
from paper_1005_1497_amd import serve

# Primes and the longest transform of each (32-bit words): the Rader primes of
# the paper's Table 1 and the Euler-form prime 7 * 2^20 + 1; for 64-bit words
# the 45-bit Rader prime of the served workload.
RADER = {13631489: 19, 319489: 12, 2424833: 10}
EULER = {7340033: 20}
WIDE = {31065037602817: 18}
M_MAIN, M_EULER, M_WIDE = 13631489, 7340033, 31065037602817


def listed():
    return [
        # the smallest call a program makes: one short convolution, latency only
        {"name": "single_2^10", "kind": "single", "m": M_MAIN, "n": 10},
        # the longest transform of the main prime, one at a time
        {"name": "single_2^19", "kind": "single", "m": M_MAIN, "n": 19},
        # many short sequences, an odd count (digital filters over short blocks)
        {"name": "batch_2^7", "kind": "batch", "m": M_MAIN, "n": 7, "count": 100003},
        # the longest length that one workgroup holds in local memory
        {"name": "batch_2^12", "kind": "batch", "m": M_MAIN, "n": 12, "count": 5000},
        # a middling batch of middling length, Euler-form prime
        {"name": "batch_2^14", "kind": "batch", "m": M_EULER, "n": 14, "count": 777},
        # the benchmark's own batch
        {"name": "batch_2^16", "kind": "batch", "m": M_MAIN, "n": 16, "count": 4096},
        # the benchmark's uneven batch: lengths 2^6 .. 2^19 in one call
        {"name": "uneven_2^6..2^19", "kind": "uneven", "m": M_MAIN, "lo": 6, "hi": 19, "count": 10000},
        # spectra for a program that works in the transform domain: both ways
        {"name": "transform_2^16", "kind": "transform", "m": M_MAIN, "n": 16, "count": 300},
        # exact integer convolutions of 15-bit samples
        {"name": "crt_2^15", "kind": "crt", "n": 15, "count": 600, "bits": 15},
        # undoing a filter, rows of a moderate length
        {"name": "deconv_2^13", "kind": "deconv", "m": M_MAIN, "n": 13, "count": 1000},
        # an image-sized two-dimensional convolution, not square
        {"name": "conv2d_1024x4096", "kind": "conv2d", "m": M_MAIN, "rows": 10, "cols": 12},
        # the served workload: 64-bit words, mixed lengths, operands on the host
        {"name": "served_2^8..2^18", "kind": "served", "m": M_WIDE, "lo": 8, "hi": 18, "count": 48},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "batch", "batch", "batch", "uneven", "transform", "crt", "deconv", "conv2d", "wide",
                       "served"])
    m = rng.choice([M_MAIN, M_MAIN, M_EULER, 319489, 2424833])
    top = RADER[m] if m in RADER else EULER[m]
    if kind == "single":
        return {"kind": kind, "m": m, "n": rng.randint(6, top)}
    if kind == "uneven":
        hi = rng.randint(12, 19)
        lo = rng.randint(4, hi - 4)
        # mean length is about 2^(hi + 1) / (hi - lo + 1)
        most = max(8, min(10000, (1 << 28) * (hi - lo + 1) >> (hi + 1)))
        return {"kind": kind, "m": M_MAIN, "lo": lo, "hi": hi, "count": _log(rng, 6, most)}
    if kind == "served":
        lo = rng.randint(6, 12)
        return {"kind": kind, "m": M_WIDE, "lo": lo, "hi": rng.randint(lo + 2, 18), "count": rng.randint(4, 60)}
    if kind == "conv2d":
        rows = rng.randint(5, min(13, top))
        return {"kind": kind, "m": m, "rows": rows, "cols": rng.randint(5, min(13, top))}
    total = _log(rng, 1 << 14, 1 << 27)   # elements of an operand
    if kind == "wide":
        n = rng.randint(6, WIDE[M_WIDE])
        return {"kind": "batch", "m": M_WIDE, "n": n, "count": max(1, min(200000, (total >> 1) >> n))}
    if kind == "crt":
        n = rng.randint(6, 19)
        return {"kind": kind, "n": n, "count": max(1, min(200000, total >> n)), "bits": min(23, (46 - n) // 2)}
    n = rng.randint(4, top)
    count = max(1, min(300000, total >> n))
    if kind == "deconv":
        return {"kind": kind, "m": m, "n": n, "count": max(1, count // 4)}
    return {"kind": kind, "m": m, "n": n, "count": count}


def _flags(m):
    return nt.FLAG_EULER if m in EULER else 0


def _uniform(gen, hi, shape, wide=False):
    return torch.randint(0, hi, shape, generator=gen, device="cuda", dtype=torch.int64 if wide else torch.int32)


def _lengths(case, seed):
    """log2 lengths of a mixed batch: the lengths a queue holds are drawn once
    per program, the operands per call."""
    del seed
    rng = np.random.default_rng(case["count"] * 64 + case["hi"])
    return rng.integers(case["lo"], case["hi"] + 1, size=case["count"])


def _offsets(log2n):
    sizes = np.left_shift(np.int64(1), log2n.astype(np.int64))
    return np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64), int(sizes.sum())


def prepare(case, seed):
    kind = case["kind"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    if kind == "served":
        rng = np.random.default_rng(int(seed))
        logs = _lengths(case, seed)
        ops = [[rng.integers(0, case["m"], size=1 << int(n), dtype=np.uint64) for _ in range(2)] for n in logs]
        out = [np.empty(1 << int(n), dtype=np.uint64) for n in logs]
        srv = serve.NativeConvServer(case["m"], 22, streams=8, max_inflight=8, host_arenas=True)
        return {"kind": kind, "srv": srv, "ops": ops, "out": out}
    s = {"kind": kind}
    if kind == "crt":
        shape = (case["count"], 1 << case["n"])
        s["f"], s["g"] = (_uniform(gen, 1 << case["bits"], shape) for _ in range(2))
        s["out"] = torch.empty(shape, dtype=torch.int64, device="cuda")
        return s
    m = s["m"] = case["m"]
    s["flags"] = _flags(m)
    wide = m in WIDE
    if kind == "conv2d":
        shape = (1 << case["rows"], 1 << case["cols"])
    elif kind == "single":
        shape = (1 << case["n"],)
    elif kind == "uneven":
        logs = _lengths(case, seed)
        offs, total = _offsets(logs)
        shape = (total,)
        s["desc"] = nt.BatchDesc(logs, offs)
    elif kind == "batch":
        shape = (case["count"] << case["n"],)
        s["desc"] = nt.BatchDesc(np.full(case["count"], case["n"]),
                                 np.arange(case["count"], dtype=np.int64) << case["n"])
    else:
        shape = (case["count"], 1 << case["n"])
    if kind in ("batch", "uneven"):
        s["order"] = nt.max_log2n(m) if m in EULER else nt.modulus_order(m)
        s["root"] = nt.euler_root(m, s["order"]) if m in EULER else 2
    s["f"] = _uniform(gen, m, shape, wide)
    if kind == "deconv":
        # a filter that can be undone: no coefficient of its spectrum is zero
        s["f"] = nt.ntt_inverse(torch.randint(1, m, shape, generator=gen, device="cuda", dtype=torch.int32), m,
                                flags=s["flags"])
    s["g"] = _uniform(gen, m, shape, wide)
    s["out"] = torch.empty_like(s["f"])
    if kind == "transform":
        s["back"] = torch.empty_like(s["f"])
    return s


def run(s):
    kind = s["kind"]
    if kind == "served":
        srv = s["srv"]
        tickets = [srv.submit(f, g) for f, g in s["ops"]]
        return [srv.result(t, out=o) for t, o in zip(tickets, s["out"])]
    if kind == "crt":
        return nt.conv_crt(s["f"], s["g"], out=s["out"])
    m, flags = s["m"], s["flags"]
    if kind == "single":
        return nt.conv_circular(s["f"], s["g"], m, out=s["out"], flags=flags)
    if kind in ("batch", "uneven"):
        return nt.conv_batched(s["f"], s["g"], s["desc"], m, root=s["root"], root_log2order=s["order"], out=s["out"],
                               flags=flags)
    if kind == "transform":
        return (nt.ntt_forward(s["f"], m, out=s["out"], flags=flags),
                nt.ntt_inverse(s["g"], m, out=s["back"], flags=flags))
    if kind == "deconv":
        return nt.deconvolve(s["f"], s["g"], m, out=s["out"], flags=flags)
    return nt.conv2d(s["f"], s["g"], m, out=s["out"], flags=flags)


def _conv_ops(n):
    """Additions and multiplications modulo m of one convolution of length 2^n
    by three radix-2 transforms and a product."""
    N = 1 << n
    return 3 * (N // 2) * n * 3 + 2 * N


def work(case):
    kind = case["kind"]
    if kind in ("uneven", "served"):
        logs = _lengths(case, 0)
        wb = 8 if case["m"] in WIDE else 4
        return {"bytes": 3 * wb * int(np.left_shift(np.int64(1), logs.astype(np.int64)).sum()),
                "flops": int(sum(_conv_ops(int(n)) for n in logs))}
    if kind == "conv2d":
        n = case["rows"] + case["cols"]
        return {"bytes": 12 << n, "flops": _conv_ops(n)}
    n, count = case["n"], case.get("count", 1)
    if kind == "crt":
        return {"bytes": 16 * count << n, "flops": 2 * count * _conv_ops(n)}
    if kind == "transform":
        return {"bytes": 16 * count << n, "flops": 2 * count * 3 * ((1 << n) // 2) * n}
    wb = 8 if case["m"] in WIDE else 4
    return {"bytes": 3 * wb * count << n, "flops": count * _conv_ops(n)}


# ------------------------------------------------------------- exact results
# Textbook radix-2 transforms in 64-bit integers.  Products of two residues
# above 2^31 are taken in 15-bit pieces, so that nothing exceeds 2^62.

def _mul(a, b, m):
    if m < 1 << 31:
        return a * b % m
    r = a * (b >> 30) % m
    r = ((r << 15) + a * ((b >> 15) & 0x7FFF) % m) % m
    return ((r << 15) + a * (b & 0x7FFF) % m) % m


def _root(m, n):
    """A root of exact order 2^n modulo the prime m, for convolutions (any will do)."""
    z = 2
    while pow(z, (m - 1) // 2, m) != m - 1:
        z += 1
    return pow(z, (m - 1) >> n, m)


def _powers(w, count, m, device):
    p = torch.ones(1, dtype=torch.int64, device=device)
    while p.numel() < count:
        p = torch.cat([p, _mul(p, torch.full_like(p, pow(w, p.numel(), m)), m)])
    return p[:count]


def _ntt(x, w, m):
    """sum_t x(t) w^(u t) mod m along the last dimension (decimation in time)."""
    N = x.shape[-1]
    if N == 1:
        return x % m
    lead = x.shape[:-1]
    # Stockham passes: a has shape (lead, N / span, span)
    a = (x % m).reshape(*lead, N, 1)
    span = 1
    while span < N:
        half = a.shape[-2] // 2
        e, o = a[..., :half, :], a[..., half:, :]
        tw = _powers(pow(w, N // (2 * span), m), span, m, x.device)
        o = _mul(o, tw, m)
        a = torch.cat([(e + o) % m, (e - o) % m], dim=-1)
        span *= 2
    return a.reshape(*lead, N)


def _inverse(X, w, m):
    N = X.shape[-1]
    y = _ntt(X, pow(w, -1, m), m)
    return _mul(y, torch.full_like(y, pow(N, -1, m)), m)


def _conv(f, g, m):
    N = f.shape[-1]
    w = _root(m, N.bit_length() - 1)
    return _inverse(_mul(_ntt(f, w, m), _ntt(g, w, m), m), w, m)


def _power(x, e, m):
    r = torch.ones_like(x)
    while e:
        if e & 1:
            r = _mul(r, x, m)
        x = _mul(x, x, m)
        e >>= 1
    return r


def _rows(fn, n, *operands):
    """fn over the rows of length 2^n of each operand, a share at a time."""
    rows = [t.reshape(-1, 1 << n) for t in operands]
    share = max(1, (1 << 26) >> n)
    return torch.cat([fn(*(t[i:i + share].to(torch.int64) for t in rows)) for i in range(0, rows[0].shape[0], share)])


def exact(case, seed):
    kind = case["kind"]
    s = prepare(case, seed)
    if kind == "served":
        s["srv"].close()
        return [_conv(*(torch.from_numpy(x.astype(np.int64)).cuda() for x in p), case["m"]).cpu().numpy().astype(np.uint64)
                for p in s["ops"]]
    f, g = s["f"], s["g"]
    if kind == "uneven":
        logs, out = _lengths(case, seed), s["out"]
        offs, _ = _offsets(logs)
        for n in sorted(set(int(v) for v in logs)):
            at = torch.from_numpy(offs[logs == n]).cuda()
            idx = (at[:, None] + torch.arange(1 << n, device="cuda")[None, :]).reshape(-1)
            out[idx] = _rows(lambda a, b: _conv(a, b, case["m"]), n, f[idx], g[idx]).reshape(-1).to(out.dtype)
            del idx
        return out
    if kind == "crt":
        m1, m2 = M_MAIN, M_EULER

        def integers(a, b):
            h1, h2 = _conv(a, b, m1), _conv(a, b, m2)
            return h1 + m1 * _mul((h2 - h1) % m2, torch.full_like(h1, pow(m1, -1, m2)), m2)
        return _rows(integers, case["n"], f, g).reshape(f.shape)
    m = case["m"]
    if kind == "conv2d":
        wr, wc = _root(m, case["rows"]), _root(m, case["cols"])
        F, G = (_ntt(_ntt(t.to(torch.int64), wc, m).T.contiguous(), wr, m) for t in (f, g))
        return _inverse(_inverse(_mul(F, G, m), wr, m).T.contiguous(), wc, m).to(f.dtype)
    n = case["n"]
    if kind == "transform":
        w = nt.euler_root(m, n) if m in EULER else nt.default_root(m, n)
        return (_rows(lambda a: _ntt(a, w, m), n, f).reshape(f.shape).to(f.dtype),
                _rows(lambda a: _inverse(a, w, m), n, g).reshape(f.shape).to(f.dtype))
    if kind == "deconv":
        w = _root(m, n)

        def quotient(a, h):
            return _inverse(_mul(_ntt(h, w, m), _power(_ntt(a, w, m), m - 2, m), m), w, m)
        return _rows(quotient, n, f, g).reshape(f.shape).to(f.dtype)
    return _rows(lambda a, b: _conv(a, b, m), n, f, g).reshape(f.shape).to(f.dtype)
