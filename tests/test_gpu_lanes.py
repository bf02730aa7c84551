"""The count walk's packed lanes, its stretches' edges and halted scans, against the oracle.

Where they can go wrong: certified bytes far sparser or denser than the lanes (most lanes empty,
a workgroup without any, a last slice that ends past its workgroup), slices ending around the
64- and 128-byte stretches, scans that halt at every place of a window, a lane and a 256-lane
group, and the slice count, which is the number of lanes whose nominal range holds a certified
byte (lane 0 always).  The outputs are whole numbers and must be equal.
"""
import numpy as np
import pytest

import oracle
import workloads
from workloads import tokensets as T

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2608_03473_amd")

_SETS = {}


def lexers(name, framed=False):
    if (name, framed) not in _SETS:
        defs = T.as_tuples(T.NAMED[name])
        lx = P.Lexer.compile_framed(defs, 0x1E) if framed else P.Lexer.compile(defs)
        oc = oracle.OracleSet(defs, reserved=0x1E) if framed else oracle.OracleSet(defs)
        _SETS[name, framed] = lx, oc
    return _SETS[name, framed]


def check(name, buf, mode, lane=0, path=0, pad=0, framed=False, offsets=False, block=0, label=""):
    lx, oc = lexers(name, framed)
    o = P.RunOpts(lane_bytes=lane, path=path, block_threads=block)
    plan = lx.plan(len(buf), mode, o)
    print(f"[case] {name} mode={mode} n={len(buf)} lane={plan['lane_bytes']} path={plan['path']} pad={pad} {label}", flush=True)
    big = torch.zeros(len(buf) + pad, dtype=torch.uint8, device="cuda")
    big[pad:] = torch.from_numpy(np.array(buf, copy=True)).cuda()
    k, l, f, con = oc.lex(bytes(buf), discard=bool(mode & 1), offsets=True)
    r = lx.run(big[pad:], mode=mode, offsets=offsets, opts=o)
    assert (r.status, r.error_offset, r.ntokens) == (0, con, len(k))
    np.testing.assert_array_equal(r.kinds.cpu().numpy(), k)
    np.testing.assert_array_equal(r.lens.cpu().numpy().view(np.uint32), l)
    if offsets:
        np.testing.assert_array_equal(r.offsets.cpu().numpy().astype(np.uint64), f)
    cert = np.zeros(256, bool)
    cert[list(lx.cert(mode))] = True
    hit = cert[np.asarray(buf)]
    lb = plan["lane_bytes"]
    want = 1 + sum(bool(hit[x: x + lb].any()) for x in range(lb, len(buf), lb)) if len(buf) else 0
    if not plan["hybrid"]:
        assert r.nslices == want
    return r


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def lines(n, width, seed):
    """C-like text whose line feeds stand about `width` bytes apart."""
    w = workloads.clike(n, seed).copy()
    w[w == 10] = 32
    w[w == ord('"')] = ord("x")
    w[w == ord("/")] = ord("+")  # no comments: they would run to the line's end
    rng = np.random.default_rng(seed)
    at = np.cumsum(rng.integers(max(1, width // 2), width * 3 // 2 + 1, max(2, 2 * n // width)))
    w[at[at < n]] = 10
    return w


@pytest.mark.parametrize("lane", [16, 64, 128, 512, 1024])
@pytest.mark.parametrize("width", [3, 40, 70, 700, 20000])
def test_sparse_and_dense_cuts(width, lane):
    w = lines(150_001, width, width + lane)
    for path in (1, 2, 3):
        check("clike_l", w, P.LEX_MODE_EXACT, lane, path, pad=5 * path, offsets=path == 2)
    check("clike_d", w, P.LEX_MODE_DISCARD, lane, 3, pad=1)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 4095, 16384, 16385, 20000])
def test_one_and_two_groups(n):
    """One 256-lane group (no look-back) and just past it, at the default lane."""
    w = workloads.clike(n, n)
    j = workloads.json(max(n, 32), n)[:n]
    for pad in (0, 1, 63):
        check("clike_l", w, P.LEX_MODE_EXACT, pad=pad, offsets=True)
        check("clike_d", w, P.LEX_MODE_DISCARD, pad=pad)
        check("json", j, P.LEX_MODE_DISCARD, pad=pad)


@pytest.mark.parametrize("name,mode", [("clike_l", 0), ("clike_d", 1), ("json", 1)])
@pytest.mark.parametrize("lane", [64, 512])
def test_halts_everywhere(name, mode, lane):
    """A byte that starts no token, over the places of a window, a lane and a group."""
    n = 300 * lane + 77
    base = workloads.json(n, 7) if name == "json" else workloads.clike(n, 7)
    places = [0, 1, 63, 64, 65, lane - 1, lane, 129, 200 * lane + 31, 256 * lane - 1, 256 * lane, 256 * lane + 5, n - 1]
    for i, x in enumerate(places):
        w = base.copy()
        w[x] = 0x01
        for path in (2, 3):
            check(name, w, mode, lane, path, pad=(0, 3, 64)[i % 3], offsets=i % 2 == 0, label=f"at {x}")
    # unterminated at the end, and a halt in every line
    w = base.copy()
    w[-5:] = np.frombuffer(b'\n"ab\\', np.uint8)
    check(name, w, mode, lane, 3, label="unterminated")
    check(name, np.where(base == 10, 1, base).astype(np.uint8), mode, lane, 0, label="every line")


@pytest.mark.parametrize("block", [256, 1024])
@pytest.mark.parametrize("lane", [64, 128, 1024])
def test_framed_records_packed(lane, block):
    w = workloads.clike(400_003, 3, bcomment=True, frame=8)
    for mode in (P.LEX_MODE_EXACT, P.LEX_MODE_DISCARD):
        check("clike_b", w, mode, lane, 2, pad=7, framed=True, block=block)
