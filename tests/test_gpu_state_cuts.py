"""The hybrid plan's state cuts against the oracle: sizes around the lanes' and workgroups' edges
(the lane is 4, 8 or 16 windows, a workgroup 240 lanes), buffers at any alignment, tokens that
outlast the warm-up, a workgroup's lanes or the plan's sync window, halts at every kind of place
and longest-match fallbacks (the second route).  Whole numbers, equal, the slice count included:
the plan's cuts 4 KiB apart, one slice when some boundary finds none or the scan halts."""
import numpy as np
import pytest

import oracle
import workloads
from workloads import tokensets as T

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2608_03473_amd")

_SETS = {}


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def check(name, buf, mode, pad=0, offsets=False, slices=None, label=""):
    if name not in _SETS:
        defs = T.as_tuples(T.NAMED[name])
        _SETS[name] = P.Lexer.compile(defs), oracle.OracleSet(defs)
    lx, oc = _SETS[name]
    assert lx.plan(len(buf), mode)["hybrid"] == 1
    print(f"[case] {name} mode={mode} n={len(buf)} pad={pad} {label}", flush=True)
    big = torch.zeros(len(buf) + pad, dtype=torch.uint8, device="cuda")
    big[pad:] = torch.from_numpy(np.array(buf, copy=True)).cuda()
    k, l, f, con = oc.lex(bytes(buf), discard=bool(mode & 1), offsets=True)
    r = lx.run(big[pad:], mode=mode, offsets=offsets)
    assert (r.status, r.error_offset, r.ntokens) == (0, con, len(k))
    np.testing.assert_array_equal(r.kinds.cpu().numpy(), k)
    np.testing.assert_array_equal(r.lens.cpu().numpy().view(np.uint32), l)
    if offsets:
        np.testing.assert_array_equal(r.offsets.cpu().numpy().astype(np.uint64), f)
    if slices is not None:
        assert r.nslices == slices
    return r


def text(n, seed):
    return workloads.clike(n, seed, bcomment=True)


@pytest.mark.parametrize("n", [4097, 4159, 4160, 8192, 8193, 61440, 61441, 61440 + 4096, 122881, 400_003])
def test_edges(n):
    for pad in (0, 1, 63, 64):
        for mode in (P.LEX_MODE_EXACT, P.LEX_MODE_DISCARD):
            r = check("clike_b", text(n, n), mode, pad, offsets=pad == 1)
            assert r.nslices in (-(-n // 4096), -(-n // 4096) - 1)
        check("clike_d", workloads.clike(n, n), P.LEX_MODE_EXACT, pad)  # monotone
        check("json", workloads.json(n, n), P.LEX_MODE_EXACT, pad)


@pytest.mark.parametrize("at", [300, 4096 - 20, 61440 - 1000, 61440 - 100, 150_000])
@pytest.mark.parametrize("size", [200, 1500, 5000, 70_000])
def test_long_tokens(at, size):
    """A comment over lanes and workgroups: one slice when no start is common within 2 KiB of a cut."""
    body = np.frombuffer(b"/* " + b'x y" ' * (size // 5) + b" */\n", np.uint8)
    w = np.concatenate([text(at, 6), body, text(100_000, 8)])
    for mode in (P.LEX_MODE_EXACT, P.LEX_MODE_DISCARD):
        r = check("clike_b", w, mode, pad=9)
        if any(at + 2 <= c and c + 2048 < at + body.size - 4 for c in range(4096, w.size, 4096)):
            assert r.nslices == 1


@pytest.mark.parametrize("name,mode", [("clike_b", 0), ("clike_b", 1), ("clike_d", 0), ("json", 0)])
def test_halts_and_fallbacks(name, mode):
    n = 140_000
    base = text(n, 3) if name == "clike_b" else workloads.clike(n, 3) if name == "clike_d" else workloads.json(n, 3)
    for i, x in enumerate([0, 1, 255, 256, 4096, 61439, 61440, 61500, 99_999, n - 1]):
        w = base.copy()
        w[x: x + 3] = 0x01
        check(name, w, mode, pad=(0, 5)[i % 2], offsets=i % 3 == 0, label=f"halt at {x}")
    # an unterminated comment or string at the end, and a number cut short in the middle
    for tail in (b"/* a b", b'"ab', b"12."):
        w = base.copy()
        w[-len(tail):] = np.frombuffer(tail, np.uint8)
        check(name, w, mode, label=str(tail))
    if name == "clike_b":
        w = np.concatenate([base[:70_000], np.frombuffer(b"\n/* open", np.uint8)])
        check(name, w, mode, label="fallback at the end")


def test_long_tokens_before_every_workgroup():
    """Comments over the start of every workgroup's warm-up lanes, whose guesses there are wrong: none of
    what they walk may reach the checkpoints of the workgroup that owns those lanes (more
    workgroups than the chip holds at once, so that they run at different times)."""
    n = 24 << 20
    w = text(n, 17).copy()
    for at in range(61440 - 4096 - 700, n - 4096, 61440):
        w[at: at + 3] = np.frombuffer(b"\n/*", np.uint8)
        w[at + 3: at + 1400] = ord("x")
        w[at + 900: at + 1400: 50] = 10
        w[at + 1400: at + 1403] = np.frombuffer(b"*/\n", np.uint8)
    for mode in (P.LEX_MODE_EXACT, P.LEX_MODE_DISCARD):
        check("clike_b", w, mode, label="long comments")
