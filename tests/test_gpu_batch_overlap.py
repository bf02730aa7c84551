"""Documents that share bytes, against the oracle: a table may ask for more 64-window tiles than the
bytes hold, and the batch then records no checkpoints and takes the lane emit for every document."""
import numpy as np
import pytest

import hostmodel
import oracle
import workloads
from workloads import tokensets as T

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2608_03473_amd")

INST = [("clike_l", P.LEX_MODE_EXACT), ("clike_d", P.LEX_MODE_DISCARD), ("clike_b", P.LEX_MODE_DISCARD)]


@pytest.fixture(scope="module")
def setup():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    defs = [T.as_tuples(T.NAMED[n]) for n, _ in INST]
    lx = [P.Lexer.compile(d) for d in defs]
    return lx, [oracle.OracleSet(d) for d in defs], P.Batch([(l, m) for l, (_, m) in zip(lx, INST)])


def slices(lx, inst, w, flags, lane):
    """The plan's slices of a document without a halt (S = X = 2 KiB for a split refused one)."""
    if not w.size or flags & 1:
        return int(w.size > 0)
    cert = np.zeros(256, bool)
    cert[list(lx[inst].cert(INST[inst][1]))] = True
    if not cert.any():
        if w.size <= max(2048, lane):
            return 1
        cuts = hostmodel.spec_plan(hostmodel.Model(lx[inst], INST[inst][1]), bytes(w), 2048, 2048)
        return 1 if cuts is None else sum(a < b for a, b in zip(cuts, cuts[1:] + [w.size]))
    hit = cert[w]
    return 1 + sum(bool(hit[x: x + lane].any()) for x in range(lane, w.size, lane))


def check(setup, data, recs, lane=0, offsets=False):
    lx, oc, batch = setup
    docs = np.array(recs, dtype=P.DOC_DTYPE)
    opts = P.RunOpts(lane_bytes=lane) if lane else None
    print(f"[case] {docs.size} documents over {data.size} bytes, lane {lane}, offsets {offsets}", flush=True)
    r = batch.run(torch.from_numpy(data).cuda(), docs, offsets=offsets, opts=opts, cap=int(docs["length"].sum()) + 16)
    assert r.status == 0
    kinds, lens = r.kinds.cpu().numpy(), r.lens.cpu().numpy().view(np.uint32)
    offs = r.offsets.cpu().numpy().astype(np.uint64) if offsets else None
    pos, want = 0, {}
    for doc, x in zip(docs, r.docs):
        a, n, inst, fl = (int(doc[f]) for f in ("offset", "length", "inst", "flags"))
        key = a, n, inst, fl
        if key not in want:
            w = data[a: a + n]
            want[key] = oc[inst].lex(w.tobytes(), discard=bool(INST[inst][1] & 1), offsets=True) + (w,)
            if want[key][3] == n:
                want[key] += (slices(lx, inst, w, fl, lane or 1024),)
        k, l, o, con = want[key][:4]
        assert (x["tok_offset"], x["ntokens"], x["error_offset"]) == (pos, len(k), con), key
        if len(want[key]) > 5:
            assert x["nslices"] == want[key][5], key
        np.testing.assert_array_equal(kinds[pos: pos + len(k)], k)
        np.testing.assert_array_equal(lens[pos: pos + len(k)], l)
        if offsets:
            np.testing.assert_array_equal(offs[pos: pos + len(k)], o)
        pos += len(k)
    assert pos == r.ntokens


@pytest.mark.parametrize("offsets", [False, True])
@pytest.mark.parametrize("stray", [False, True])
def test_more_tiles_than_the_bytes_hold(setup, stray, offsets):
    """One lane each (serial, or of a refused set under a long lane), a split refused document among
    serial ones, and few long lanes: lanes within the workspace, tiles beyond it."""
    n = 60_000
    data = workloads.clike(n, 3, bcomment=True).copy()
    plain = workloads.clike(n, 4).copy()
    if stray:
        data[41_007] = plain[41_007] = 1
    check(setup, plain, [(0, n, 0, 1)] * 8 + [(7, n - 7, 1, 1), (1, n // 2, 1, 1)], offsets=offsets)
    check(setup, data, [(i, n - i, 2, 0) for i in range(6)], lane=65536, offsets=offsets)
    check(setup, data, [(0, n, 2, 0)] + [(0, n, 2, 1)] * 7, offsets=offsets)
    check(setup, plain, [(0, n, 0, 0), (3, n - 3, 1, 0), (0, n, 1, 0)], lane=16384, offsets=offsets)


@pytest.mark.parametrize("ndocs", [40, 300])
def test_short_documents_over_the_same_bytes(setup, ndocs):
    """More finely walked lanes than the workspace's: the batch is walked in its plan's lanes, one to a
    document here.  More of the plan's lanes than the bytes hold stops it."""
    data = workloads.clike(1000, 9).copy()
    data[700] = 1
    check(setup, data, [(0, 1000, d % 2, 0) for d in range(ndocs)], offsets=True)
    check(setup, data, [(d % 7, 1000 - d % 11 - 7, d % 3, d % 2) for d in range(ndocs)])
    n = 60_000
    big = torch.from_numpy(workloads.clike(n, 4)).cuda()
    for lane in (0, 1024):
        r = setup[2].run(big, np.array([(0, n, 0, 0)] * 3, dtype=P.DOC_DTYPE), cap=3 * n,
                         opts=P.RunOpts(lane_bytes=lane) if lane else None)
        assert r.status == P.LEX_EINVAL and (r.docs["status"] == P.LEX_EINVAL).all()
