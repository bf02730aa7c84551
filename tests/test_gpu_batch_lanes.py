"""Batches at their default lane, whose documents are walked in finer lanes than their slices are
counted by: every document against the oracle, its slice count against the plan's definition, and
halted documents (written by the windowed emit up to their halt), at the document counts where
planning and results move from one workgroup to several."""
import numpy as np
import pytest

import oracle
import workloads
from workloads import tokensets as T

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2608_03473_amd")

INST = [("clike_l", P.LEX_MODE_EXACT), ("clike_d", P.LEX_MODE_DISCARD), ("json", P.LEX_MODE_DISCARD),
        ("clike_b", P.LEX_MODE_DISCARD)]


@pytest.fixture(scope="module")
def lexers():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    defs = [T.as_tuples(T.NAMED[n]) for n, _ in INST]
    return [P.Lexer.compile(d) for d in defs], [oracle.OracleSet(d) for d in defs]


def text(inst, n, seed):
    if inst == 2:
        return workloads.json(max(n, 32), seed)[:n]
    return workloads.clike(n, seed, bcomment=inst == 3)


@pytest.mark.parametrize("ninst", [3, 4])
@pytest.mark.parametrize("ndocs,median", [(1, 40000), (16, 3000), (64, 700), (65, 700), (300, 9000)])
def test_default_lane(lexers, ninst, ndocs, median):
    lx, oc = lexers
    rng = np.random.default_rng(ndocs * 7 + ninst)
    sizes = np.minimum((median * np.exp(rng.standard_normal(ndocs))).astype(np.int64), 60000)
    sizes[0] = min(sizes[0], 4097) if ndocs > 1 else sizes[0]
    if ndocs > 3:
        sizes[1:4] = 0, 1, 1024
    docs = np.zeros(ndocs, P.DOC_DTYPE)
    parts, at = [], 0
    for d in range(ndocs):
        inst = d % ninst
        w = text(inst, int(sizes[d]), d).copy()
        if d % 5 == 4 and w.size:  # malformed: at its start, its end or inside
            w[(0, w.size - 1, w.size // 3, w.size * 2 // 3)[d // 5 % 4]] = 0x01
        docs[d] = (at, w.size, inst, 1 if d % 17 == 16 else 0)
        parts.append(w)
        at += w.size
    data = torch.from_numpy(np.concatenate(parts) if at else np.zeros(1, np.uint8)).cuda()
    b = P.Batch([(lx[k], INST[k][1]) for k in range(ninst)])
    print(f"[case] ndocs={ndocs} ninst={ninst} bytes={at}", flush=True)
    for offsets in (False, True):
        r = b.run(data[:at], docs, offsets=offsets)
        assert r.status == 0
        kinds, lens = r.kinds.cpu().numpy(), r.lens.cpu().numpy().view(np.uint32)
        offs = r.offsets.cpu().numpy() if offsets else None
        pos = 0
        for d in range(ndocs):
            inst = int(docs[d]["inst"])
            k, l, o, con = oc[inst].lex(parts[d].tobytes(), discard=bool(INST[inst][1] & 1), offsets=True)
            x = r.docs[d]
            assert (x["tok_offset"], x["ntokens"], x["error_offset"]) == (pos, len(k), con), d
            np.testing.assert_array_equal(kinds[pos: pos + len(k)], k)
            np.testing.assert_array_equal(lens[pos: pos + len(k)], l)
            if offsets:
                np.testing.assert_array_equal(offs[pos: pos + len(k)].astype(np.uint64), o)
            pos += len(k)
            n = parts[d].size
            if docs[d]["flags"]:
                assert x["nslices"] == (n > 0)
            elif inst < 3:  # slices of 1 KiB plan lanes, up to the halted one's
                cert = np.zeros(256, bool)
                cert[list(lx[inst].cert(INST[inst][1]))] = True
                hit = cert[parts[d]]
                starts = [0] + [j + int(np.argmax(hit[j: j + 1024])) for j in range(1024, n, 1024) if hit[j: j + 1024].any()]
                want = sum(s <= con for s in starts) if con < n else len(starts)
                assert x["nslices"] == (want if n else 0), (d, n, con)
        assert pos == r.ntokens
