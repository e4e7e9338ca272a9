"""A CPU model of two shortcuts of the transform kernel (csrc/parametric.h)
against the plain evaluation they stand for, bit for bit: whole periods of a
schedule taken at once (`repeats` and the shift of all clocks), and blocks as
one addition of whole ulps -- against a slot-by-slot walk that adds every cost.
(tests/test_send_scan_model.py: a slot's Sends as scans.)

It calls neither the library nor the oracle; the GPU parity tests check the
kernel itself."""
import math
import random
import struct

import pytest


def bits(v):
    return struct.unpack("<q", struct.pack("<d", v))[0]


def double(b):
    return struct.unpack("<d", struct.pack("<q", b))[0]


def repeats(pair, bwd, nf, nb, K, mr, back):
    step = 1 if pair else 2
    n = 1 << 30
    if pair or not bwd:
        k0 = nf - step * (1 + back)
        n = K - nf
        if k0 < mr:
            n = min(n, mr - nf)
    if pair or bwd:
        k0 = nb - step * (1 + back)
        if k0 < 1:
            return 0
        n = min(n, K - nb)
        if k0 < mr:
            n = min(n, mr - nb)
    return int(n / step)


def pipeline(schedule, P, K, mr, cost, send, skip):
    """Final clocks of P stages and the number of slots walked.  cost(s, bwd,
    size class, accumulating): a block's op costs; send[size class]."""
    train = schedule != "infer"
    length = (2 if train else 1) * K
    wu = [min(P - 1 - s, K) if schedule == "1f1b" else K for s in range(P)]
    clk, nf, nb = [0.0] * P, [0] * P, [0] * P
    c0, prev_d, prev, odd, slots = None, -1, None, False, 0

    def block(t, ops, e_ok=True):
        if skip and t > 0.0 and not math.isinf(t):
            # whole ulps of the binade, if none is a half and the sum stays in it
            e = math.frexp(t)[1] - 1
            tot, tie = 0, False
            for c in ops:
                u = math.ldexp(c, 52 - e)
                tot += round(u)
                tie = tie or abs(u - round(u)) == 0.5
            nxt = bits(t) + tot
            if not tie and nxt >> 52 == bits(t) >> 52:
                return double(nxt)
        for c in ops:
            t += c
        return t

    while True:
        ready = {}
        for s in range(P):
            bwd = nf[s] == K or nf[s] - nb[s] > wu[s]
            k = nb[s] if bwd else nf[s]
            avail = (nf[s] if s == P - 1 else nb[s + 1]) if bwd else (1 << 30 if s == 0 else nf[s - 1])
            if nf[s] + nb[s] < length and avail > k:
                ready[s] = (bwd, k)
        if not ready:
            return clk, slots
        slots += 1
        for s, (bwd, k) in ready.items():
            clk[s] = block(clk[s], cost(s, bwd, k < mr, k > 0))
            if bwd:
                nb[s] += 1
            else:
                nf[s] += 1
        for s in sorted(ready):
            bwd, k = ready[s]
            o = s - 1 if bwd else s + 1
            if 0 <= o < P:
                clk[s] = clk[o] = max(clk[s], clk[o]) + send[k < mr]
        dirs = {s: b for s, (b, _) in ready.items()}
        if odd and skip:
            b = [bits(c) for c in clk]
            both = len(dirs) == P and prev is not None and len(prev) == P
            pat = both and (all(dirs[s] != prev[s] for s in range(P)) if schedule == "1f1b" else
                            all(dirs[s] == prev[s] == dirs[0] for s in range(P)))
            d = [b[s] - c0[s] for s in range(P)] if c0 else None
            ok = pat and d and len(set(d)) == 1 and len({x >> 52 for x in b + c0}) == 1 and 0 < b[0] >> 52 < 0x7ff
            if ok:
                back = d[0] & 1
                q = min(repeats(schedule == "1f1b", dirs[s], nf[s], nb[s], K, mr, back) for s in range(P))
                if back and prev_d != d[0]:
                    q = 0
                if d[0] > 0:
                    room = min((((x >> 52) + 1) << 52) - 1 - x for x in b)
                    q = min(q, room // d[0])
                if back:
                    q &= ~1
                if q > 0:
                    clk = [double(x + q * d[0]) for x in b]
                    for s in range(P):
                        nf[s] += q if schedule == "1f1b" else (0 if dirs[s] else 2 * q)
                        nb[s] += q if schedule == "1f1b" else (2 * q if dirs[s] else 0)
            prev_d = d[0] if ok else -1
        if odd:
            c0 = [bits(c) for c in clk]
        odd, prev = not odd, dirs


@pytest.mark.parametrize("schedule", ["1f1b", "gpipe", "infer"])
def test_whole_periods_equal_the_walk(schedule):
    rng = random.Random(schedule)
    walked = skipped = 0
    for trial in range(120):
        P = rng.choice([1, 2, 3, 5, 8])
        K = rng.choice([1, 2, 7, 40, 97, 160])
        mr = rng.randrange(K)
        kind = trial % 3
        unit = 2.0 ** rng.randint(-14, -8)

        def draw():
            if kind == 0:    # ordinary costs
                return rng.uniform(0.2, 5.0) * 1e-4
            if kind == 1:    # short dyadic fractions: half-way roundings
                return rng.randint(0, 7) * unit
            return rng.choice([0.0, unit, rng.uniform(0, 1e-15), rng.uniform(0, 1.0)])

        table = {}

        def cost(s, bwd, mc, acc):
            role = 0 if s == 0 else (1 if s == P - 1 else 2)
            key = (role, bwd, mc, bwd and acc)
            if key not in table:
                table[key] = [draw() for _ in range(rng.randint(1, 6))]
            return table[key]

        send = {True: draw(), False: draw()}
        want, n0 = pipeline(schedule, P, K, mr, cost, send, False)
        got, n1 = pipeline(schedule, P, K, mr, cost, send, True)
        assert got == want, (trial, P, K, mr)
        walked += n0
        skipped += n0 - n1
    assert skipped > walked // 4
