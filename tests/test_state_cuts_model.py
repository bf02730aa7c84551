"""The hybrid plan's state cuts restated on the CPU, at small sizes: guessed lanes, compared and repaired,
give the serial scan's states wherever they are taken to stand; and the slice count found beside them is
that of the speculative plan (hostmodel.spec_plan) they stand for, halts and misaligned buffers
included."""
import random

import pytest

import hostmodel
import workloads
from workloads import tokensets as T

P = pytest.importorskip("paper_2608_03473_amd")


class Serial:
    """The serial scan without fallbacks: at[p] = (row, token start) before byte p, the token starts,
    the byte that sent it to SINK (dead), whether a fallback was met first (fell)."""

    def __init__(self, m, w):
        self.at, self.starts, self.dead, self.fell = [(0, 0)], set(), None, False
        st, tok = 0, 0
        for p, b in enumerate(w):
            st, tok, e = step(m, st, tok, b, p)
            if e:
                self.starts.add(p)
            if st in (m.sink, m.fail):
                self.fell = st != m.sink
                self.dead = p
                break
            self.at.append((st, tok))
        if self.dead is None and w and st and not m.info[st >> 8] & hostmodel.INFO_ACC and not m.mono:
            self.fell = True


def step(m, st, tok, b, p):
    x = int(m.T[st + (b ^ ((st >> 8) & 31))])
    return (x & hostmodel.ROWMASK) >> 2, p if x & hostmodel.EMIT else tok, bool(x & hostmodel.EMIT)


def lanes_stand(m, w, mis, W, wpl, own, warm):
    """k_hstate and state_stands: whether the cuts stand, and per own lane the state it was walked from."""
    n = len(w)
    nwin = -(-(n + mis) // W)
    nl = -(-nwin // wpl)
    pos = lambda i: min(n, max(0, i * W - mis))  # noqa: E731
    dead = lambda st: st in (m.sink, m.fail)  # noqa: E731

    def walk(st, tok, a, b):
        for p in range(a, b):
            st, tok, _ = step(m, st, tok, w[p], p)
        return st, tok

    blocks = []
    for b in range(-(-nl // own)):
        ks = [k for k in range(b * own - warm, min(nl, (b + 1) * own)) if k >= 0]
        frm, end = {}, {}
        for k in ks:
            st, tok = 0, pos(k * wpl - 4) if k else 0
            for i in range(k * wpl - 4, k * wpl if k else -4):  # a guess: a dead end starts afresh
                st, tok = walk(st, tok, pos(i), pos(i + 1))
                if dead(st):
                    st, tok = 0, pos(i + 1)
            frm[k] = st, tok
            end[k] = walk(*frm[k], pos(k * wpl), pos((k + 1) * wpl))
        for _ in range(len(ks) + 1):
            new = {k: end[k - 1] for k in ks if k - 1 in end and not dead(end[k - 1][0]) and end[k - 1] != frm[k]}
            if not new:
                break
            for k in new:
                frm[k] = new[k]
                end[k] = walk(*frm[k], pos(k * wpl), pos((k + 1) * wpl))
        assert not new
        mine = [k for k in ks if k >= b * own]
        halt = next((k for k in mine if end[k][0] == m.sink or (
            pos((k + 1) * wpl) == n and m.mono and end[k][0] and not dead(end[k][0])
            and not m.info[end[k][0] >> 8] & hostmodel.INFO_ACC)), None)
        fell = any(not m.mono and (end[k][0] == m.fail or (pos((k + 1) * wpl) == n and end[k][0] and not dead(
            end[k][0]) and not m.info[end[k][0] >> 8] & hostmodel.INFO_ACC)) for k in mine if halt is None or k < halt)
        blocks.append((frm, end, mine, halt, fell))
    first = next((h for *_, h, _ in blocks if h is not None), None)
    for b, (frm, end, mine, halt, fell) in enumerate(blocks):
        if first is not None and mine[0] > first:
            break
        if fell or (b and frm[mine[0]] != blocks[b - 1][1][mine[0] - 1]):
            return False, first, {}
    return True, first, {k: bl[0][k] for bl in blocks for k in bl[2] if first is None or k <= first}


def slice_count(m, w, S, X, s, mis, W):
    """k_hscan and check_cuts, for a scan whose state cuts stand."""
    n = len(w)
    nc = -(-n // S)
    e0 = (nc - 1) * S + X
    halts = s.dead is not None
    if halts and (e0 >= n or s.dead < e0):
        return 1
    count = nc - 1 if halts else nc
    for k in range(1, nc):
        c, end, bend = k * S, min(k * S + X, n), min((k + 1) * S + X, n)
        w0 = (end - 1 + mis) // W * W - mis
        st, p, tok, lacc, same = 0, c, c, c, False
        mine = {c}
        while not same and tok < end and p < bend:
            st, tok, e = step(m, st, tok, w[p], p)
            if e:
                mine.add(tok)
            p += 1
            if not m.mono and int(m.info[st >> 8]) & hostmodel.INFO_ACC:
                lacc = p
            if st in (m.sink, m.fail):
                p = tok = lacc if st == m.fail and not m.mono and lacc > tok else tok + 1
                lacc, st = p, 0
                mine.add(p)
            elif p <= w0 and (p + mis) % W == 0:
                same = s.at[p] == (st, tok)
        same = same or any(w0 <= x < end and x in s.starts for x in mine)
        if k + 1 == nc:
            count = min(count, 1 if halts and same else nc - 1 if not same else count)
        elif not same:
            return 1
    return count


@pytest.mark.parametrize("name,mode", [("clike_b", 0), ("clike_b", 1), ("clike_d", 0), ("json", 0)])
def test_states_and_slice_counts(name, mode):
    m = hostmodel.Model(P.Lexer.compile(T.as_tuples(T.NAMED[name])), mode)
    rng = random.Random(name + str(mode))
    stood = counts = 0
    for it in range(400):
        n = rng.randint(70, 700)
        w = bytearray((workloads.json(n, it)[:n] if name == "json" else workloads.clike(n, it, bcomment=name == "clike_b")).tobytes())
        for _ in range(rng.randint(0, 2)):
            a, k = rng.randrange(n), rng.randint(1, 90)
            body = [b"\x01", b'"' + b"x" * k + b'"', b"/*" + bytes(rng.choices(b'ab "\n-*', k=k)) + b"*/", b"\n" * k, b'"' + b"x" * k + b"\n"]
            new = rng.choice(body)
            w[a: a + len(new)] = new
        if rng.random() < 0.3:
            w += rng.choice([b'"ab', b"/*a", b"12.", b"\n" * 40])
        w = bytes(w)
        W, X = 16, 48
        mis, S = rng.randrange(W), rng.choice([48, 56, 64, 80])
        s = Serial(m, w)
        ok, first, states = lanes_stand(m, w, mis, W, 4, rng.randint(1, 5), rng.randint(1, 4))
        if s.fell:
            assert not ok
            continue
        if not ok:
            continue
        stood += 1
        for k, (st, tok) in states.items():  # up to the first halted lane, its start included
            assert s.at[min(len(w), max(0, k * 4 * W - mis))] == (st, tok)
        assert (first is None) == (s.dead is None and not (
            m.mono and s.at[-1][0] and not m.info[s.at[-1][0] >> 8] & hostmodel.INFO_ACC))
        if -(-len(w) // S) < 2:
            continue
        cuts = hostmodel.spec_plan(m, w, S, X)
        want = 1 if cuts is None else sum(a < b for a, b in zip(cuts, cuts[1:] + [len(w)]))
        assert slice_count(m, w, S, X, s, mis, W) == want, (it, len(w), S, mis)
        counts += want > 1
    assert stood > 60 and counts > 20
