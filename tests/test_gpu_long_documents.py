"""Documents of many walked lanes in batches at their default lane, whose pass takes two, four or eight
lanes to a thread, and small scans on the separate routes, counted by one workgroup that writes the
result: against the oracle, halts and the plan's slice counts included."""
import numpy as np
import pytest

import oracle
import workloads
from workloads import tokensets as T

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2608_03473_amd")

INST = [("clike_l", P.LEX_MODE_EXACT), ("clike_d", P.LEX_MODE_DISCARD), ("json", P.LEX_MODE_DISCARD)]


@pytest.fixture(scope="module")
def lexers():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    defs = [T.as_tuples(T.NAMED[n]) for n, _ in INST]
    return [P.Lexer.compile(d) for d in defs], [oracle.OracleSet(d) for d in defs]


def slices(lx, mode, w, con, lane=1024):
    cert = np.zeros(256, bool)
    cert[list(lx.cert(mode))] = True
    hit = cert[w]
    starts = [0] + [j + int(np.argmax(hit[j: j + lane])) for j in range(lane, w.size, lane) if hit[j: j + lane].any()]
    return sum(s <= con for s in starts) if con < w.size else len(starts)


@pytest.mark.parametrize("nbytes", [3 << 20, 12 << 20, 24 << 20])  # walked lanes of 128, 256 and 512 bytes
@pytest.mark.parametrize("ndocs", [14, 80])
def test_long_documents(lexers, nbytes, ndocs):
    lx, oc = lexers
    ratio = {3 << 20: 8, 12 << 20: 4, 24 << 20: 2}[nbytes]
    lane = 1024 // ratio
    sizes = [lane * x + dx for x, dx in ((511, 0), (511, 1), (512, 0), (513, 7), (64 * ratio * 9, 0), (64 * ratio * 9, 1),
                                         (64 * ratio * 8 + ratio, 3), (700, 99))] + [100, 0, 1023, 1025, 9000]
    sizes += [50] * (ndocs - 1 - len(sizes))
    sizes.append(nbytes - sum(sizes))
    docs, parts, at = np.zeros(len(sizes), P.DOC_DTYPE), [], 0
    for d, n in enumerate(sizes):
        inst = d % 3
        w = (workloads.json(max(n, 32), d)[:n] if inst == 2 else workloads.clike(n, d)).copy()
        if n > 5000 and d % 2:  # a halt in the first, a middle or the last step, and empty lanes after it
            x = (n // 3, n - 1, 70 * lane + 5, n - n // 7)[d // 2 % 4]
            w[x] = 1
            w[x + 1: x + 1 + 3 * lane] = ord("a")
        docs[d] = (at, n, inst, 0)
        parts.append(w)
        at += n
    data = torch.from_numpy(np.concatenate(parts)).cuda()
    b = P.Batch([(lx[k], INST[k][1]) for k in range(3)])
    print(f"[case] {len(sizes)} documents, {at} bytes, ratio {ratio}", flush=True)
    r = b.run(data, docs)
    assert r.status == 0
    kinds, lens, pos = r.kinds.cpu().numpy(), r.lens.cpu().numpy().view(np.uint32), 0
    for d, w in enumerate(parts):
        inst = d % 3
        k, l, con = oc[inst].lex(w.tobytes(), discard=bool(INST[inst][1] & 1))
        x = r.docs[d]
        assert (x["tok_offset"], x["ntokens"], x["error_offset"]) == (pos, len(k), con), d
        np.testing.assert_array_equal(kinds[pos: pos + len(k)], k, err_msg=str(d))
        np.testing.assert_array_equal(lens[pos: pos + len(k)], l, err_msg=str(d))
        if w.size:
            assert x["nslices"] == slices(lx[inst], INST[inst][1], w, con), d
        pos += len(k)
    assert pos == r.ntokens


@pytest.mark.parametrize("n", [0, 1, 64, 2333, 16384])
@pytest.mark.parametrize("path,emit", [(1, 0), (2, 0), (2, P.LEX_EMIT_LANE), (1, P.LEX_EMIT_LANE)])
def test_one_workgroup(lexers, n, path, emit):
    lx, oc = lexers
    for inst in (0, 2):
        mode = INST[inst][1]
        base = workloads.json(max(n, 32), n)[:n] if inst == 2 else workloads.clike(n, n)
        for x in sorted({None, 0, n // 2, n - 1} - {-1}, key=lambda v: -1 if v is None else v):
            w = base.copy()
            if x is not None and n:
                w[x] = 1
            o = P.RunOpts(path=path, emit=emit)
            print(f"[case] {INST[inst][0]} n={n} path={path} emit={emit} halt at {x}", flush=True)
            k, l, con = oc[inst].lex(w.tobytes(), discard=bool(mode & 1))
            r = lx[inst].run(torch.from_numpy(w).cuda(), mode=mode, opts=o)
            assert (r.status, r.error_offset, r.ntokens) == (0, con, len(k))
            np.testing.assert_array_equal(r.kinds.cpu().numpy(), k)
            np.testing.assert_array_equal(r.lens.cpu().numpy().view(np.uint32), l)
            lane = lx[inst].plan(n, mode, o)["lane_bytes"]
            assert r.nslices == (slices(lx[inst], mode, w, n, lane) if n else 0)
            if len(k) > 1:
                r = lx[inst].run(torch.from_numpy(w).cuda(), mode=mode, opts=o, cap=len(k) - 1)
                assert (r.status, r.ntokens) == (P.LEX_EOVERFLOW, len(k))
