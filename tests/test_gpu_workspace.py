"""A workspace sized for a larger scan or batch serves every smaller one."""
import numpy as np
import pytest

import workloads
from workloads import tokensets as T

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_2608_03473_amd")


@pytest.fixture(scope="module", autouse=True)
def _needs_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def compiled(name):
    return P.Lexer.compile(T.as_tuples(T.NAMED[name]))


def test_batch_workspace_grows_with_the_bytes():
    batch = P.Batch([(compiled("clike_l"), P.LEX_MODE_EXACT)])
    sizes = sorted(b + d for b in (128, 4096, 1 << 20, 8 << 20, 16 << 20, 32 << 20, 64 << 20)
                   for d in (-1, 0, 1, 127, 128, 129, 1 << 19) if b + d > 0)
    for nd in (1, 16, 5000):
        need = [batch.workspace_size(nd, n) for n in sizes]
        assert need == sorted(need), nd
    # a batch of 8 MiB in the workspace of one of 9 MiB
    n, nd = 8 << 20, 16
    data = torch.from_numpy(workloads.clike(n, 2)).cuda()
    docs = np.zeros(nd, P.DOC_DTYPE)
    docs["length"] = n // nd
    docs["offset"] = np.arange(nd) * (n // nd)
    want = batch.run(data, docs)
    dev = torch.from_numpy(docs.view(np.uint8).copy()).cuda()
    kinds, lens = torch.zeros(n, dtype=torch.uint8, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    res, total = torch.zeros(nd * 32, dtype=torch.uint8, device="cuda"), torch.zeros(3, dtype=torch.int64, device="cuda")
    ws = torch.empty(batch.workspace_size(nd, 9 << 20), dtype=torch.uint8, device="cuda")
    print("[case] 8 MiB batch in a 9 MiB workspace", flush=True)
    batch.run_into(data, n, dev, nd, kinds, lens, None, n, res, total, ws)
    k = int(total.cpu()[0])
    assert k == want.ntokens
    assert torch.equal(kinds[:k], want.kinds) and torch.equal(lens[:k], want.lens)
    np.testing.assert_array_equal(res.cpu().numpy().view(P.DOC_RESULT_DTYPE), want.docs)
