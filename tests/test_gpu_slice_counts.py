"""The slice count of a refused set's scan, against the plan's definition (hostmodel.spec_plan): the
state cuts write the tokens, but the count reported is that of the speculative plan's cuts."""
import numpy as np
import pytest

import hostmodel
import oracle
import workloads
from workloads import tokensets as T

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2608_03473_amd")

S, X = 4096, 2048
_SETS = {}


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def check(name, buf, mode, pads=(0,), lane=S):
    if name not in _SETS:
        defs = T.as_tuples(T.NAMED[name])
        _SETS[name] = P.Lexer.compile(defs), oracle.OracleSet(defs)
    lx, oc = _SETS[name]
    w = np.array(buf, dtype=np.uint8, copy=True)
    cuts = hostmodel.spec_plan(hostmodel.Model(lx, mode), w.tobytes(), lane, X)
    want = 1 if cuts is None else sum(a < b for a, b in zip(cuts, cuts[1:] + [w.size]))
    k, l, con = oc.lex(w.tobytes(), discard=bool(mode & 1))
    for pad in pads:
        big = torch.zeros(w.size + pad, dtype=torch.uint8, device="cuda")
        big[pad:] = torch.from_numpy(w).cuda()
        for emit in (P.LEX_EMIT_DEFAULT, P.LEX_EMIT_LANE):
            o = P.RunOpts(lane_bytes=lane, emit=emit)
            assert lx.plan(w.size, mode, o)["hybrid"] == 1
            r = lx.run(big[pad:], mode=mode, opts=o)
            assert (r.status, r.error_offset, r.ntokens) == (0, con, len(k))
            np.testing.assert_array_equal(r.kinds.cpu().numpy(), k)
            np.testing.assert_array_equal(r.lens.cpu().numpy().view(np.uint32), l)
            assert r.nslices == want, (name, w.size, pad, emit)
    return want


@pytest.mark.parametrize("name,mode,tail", [("clike_d", 0, b'"ab'), ("clike_d", 0, b"\x01"), ("json", 0, b'"ab'),
                                            ("clike_b", 0, b"/* a b"), ("clike_b", 1, b'"ab')])
def test_halt_at_the_end(name, mode, tail):
    """An unterminated last token halts the scan without a restart in any speculative lane."""
    for n in (8192, 12_300, 40_000):
        w = workloads.json(n, n) if name == "json" else workloads.clike(n, n, bcomment=name == "clike_b")
        w = np.concatenate([w[: n - len(tail)], np.frombuffer(tail, np.uint8)])
        print(f"[case] {name} mode={mode} n={n} tail={tail}", flush=True)
        want = check(name, w, mode, pads=(0, 5))
        if name == "clike_d" and tail == b'"ab':
            assert want > 1


def test_halt_past_the_last_window():
    """A string over the last lane's sync window that halts after it: no lane restarts past its cut,
    so the plan keeps its other cuts; one that halts inside the window falls back."""
    base = np.frombuffer(b"if (a1 <= 20) b = c + 7;\n\tdd = 'e';\n".replace(b"'", b" ") * 300, np.uint8)  # no halt of its own
    for at, size in ((8192 - 100, 2300), (8192 - 100, 2100), (8192 - 100, 700), (8192 + 300, 2300), (4000, 6600)):
        w = np.concatenate([base[:at], np.frombuffer(b'\n"' + b"x" * size + b"\n", np.uint8)])
        w = np.concatenate([w, base[: 12_000 - w.size]])
        print(f"[case] string of {size} at {at}", flush=True)
        want = check("clike_d", w, 0, pads=(0, 1, 63))
        if (at, size) == (8192 - 100, 2300):
            assert want == 2


@pytest.mark.parametrize("lane", [S, S + 16, S + 48])
@pytest.mark.parametrize("d", [1960, 1985, 2000, 2020, 2046, 2047, 2048, 2049])
def test_first_common_start_late_in_the_window(d, lane):
    """A comment over a lane's start that ends d bytes past it: the walks meet there, in the sync window's
    last 64 bytes, between two window starts when the buffer is not aligned."""
    rng = np.random.default_rng(d)
    for body in (b"ab ", b'a" b\n', None):
        at = 2 * lane + d
        n = at - (2 * lane - 30) - 4
        inside = rng.choice(np.frombuffer(b'abc019 +-"\n\n\\', np.uint8), n) if body is None else np.frombuffer(body * n, np.uint8)[:n]
        w = np.concatenate([workloads.clike(2 * lane - 31, d, bcomment=True), np.frombuffer(b"\n/*", np.uint8), inside,
                            np.frombuffer(b"*/\n", np.uint8), workloads.clike(3 * lane, d + 1, bcomment=True)])
        print(f"[case] comment to {d}, lane {lane}", flush=True)
        want = check("clike_b", w, d & 1, pads=(0, 1, 5, 37, 63), lane=lane)
        if body == b"ab ":
            assert (want > 1) == (d < X)


@pytest.mark.parametrize("n", [8192 + 1, 8192 + 63, 8192 + 64, 8192 + 100, 8192 + 2048, 8192 + 2049, 8192 + 4000])
def test_short_last_lane(n):
    w = workloads.clike(n, n, bcomment=True)
    for tail in (b"", b"/* a */", b"abcdefghij" * 9):
        v = np.concatenate([w[: n - len(tail)], np.frombuffer(tail, np.uint8)])
        print(f"[case] n={n} tail of {len(tail)}", flush=True)
        check("clike_b", v, 1, pads=(0, 1, 63))
