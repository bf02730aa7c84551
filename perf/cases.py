"""The scans that users of the lexer run, from one small file to a resident corpus.

A case is one call of a public entry point (``Lexer.run_into``, ``Lexer.run_static_into``,
``Batch.run_into``) on text shaped like the corpora of the benchmark: C-like source, pretty-printed
JSON, record-framed source and batches of documents with log-normal sizes.  The token sets are the
ones the tests and the benchmark use.
"""
import math
import random

import numpy as np
import torch

import paper_2608_03473_amd as P

IDENT = (r"[A-Za-z_][A-Za-z0-9_]*", 0, False)
INT = (r"[0-9]+", 0, False)
OP = (r"\+|-|\*|/|%|=|==|!=|<|<=|>|>=|&&|\|\||!|\(|\)|\{|\}|\[|\]|;|,|\.", 0, False)
STR = (r'"([^"\\\n]|\\[^\n])*"', 0, False)
CLIKE_L = [IDENT, INT, OP, STR, (r"[ \t]+", 0, False), (r"\n", 0, False), (r"//[^\n]*", 0, False)]
CLIKE_D = [IDENT, INT, OP, STR, (r"[ \t\n]+", 0, True), (r"//[^\n]*", 0, True)]
CLIKE_B = CLIKE_D + [(r"/\*([^*]|\*+[^*/])*\*+/", 0, True)]
JSON = [
    (r'"([^"\\\x00-\x1F]|\\["\\/bfnrt]|\\u[0-9A-Fa-f]{4})*"', 0, False),
    (r"-?(0|[1-9][0-9]*)(\.[0-9]+)?([eE][+-]?[0-9]+)?", 0, False),
    (r"true", 0, False),
    (r"false", 0, False),
    (r"null", 0, False),
    (r"[{}\[\]:,]", 0, False),
    (r"[ \t\n\r]+", 0, True),
]

# name: (definitions, mode, text, tokens written per input byte)
SETS = {
    "clike_l": (CLIKE_L, P.LEX_MODE_EXACT, "clike", 0.264),
    "clike_d": (CLIKE_D, P.LEX_MODE_DISCARD, "clike", 0.119),
    "json": (JSON, P.LEX_MODE_DISCARD, "json", 0.127),
    "framed": (CLIKE_B, P.LEX_MODE_EXACT, "records", 0.207),  # framed at 0x1E (compile_framed)
    "refused": (CLIKE_B, P.LEX_MODE_EXACT, "blocks", 0.206),  # certifies no byte: the hybrid plan
    "clike_b": (CLIKE_B, P.LEX_MODE_DISCARD, "blocks", 0.096),
}
# sets of a serving batch, and of a corpus of documents (a twentieth of it refused)
SERVING, CORPUS = ("clike_l", "clike_d", "json"), ("clike_l", "clike_d", "clike_b")

OPS = ["+", "-", "*", "/", "%", "=", "==", "!=", "<", "<=", ">", ">=", "&&", "||", "!", "(", ")", "{", "}", "[", "]",
       ";", ",", "."]
ALPHA = "ABCDEFGHIJKLMNOPQRSTUVWXYZabcdefghijklmnopqrstuvwxyz_"
ALNUM = ALPHA + "0123456789"
PRINT = [chr(c) for c in range(0x20, 0x7F)]
STRCH = [c for c in PRINT if c not in '"\\']


def listed():
    return [
        # one small file: launches and latency
        dict(name="file_3k", kind="scan", set="clike_l", n=3001, call="into", offsets=False, stray=False),
        # a request of a tight loop on the library's own scratch, start offsets wanted
        dict(name="json_64k_static", kind="scan", set="json", n=65537, call="static", offsets=True, stray=False),
        # the small configuration of the benchmark
        dict(name="clike_l_1m", kind="scan", set="clike_l", n=1 << 20, call="into", offsets=False, stray=False),
        # an ordinary source tree, whitespace and comments dropped, a ragged size
        dict(name="clike_d_16m", kind="scan", set="clike_d", n=16_777_259, call="into", offsets=False, stray=False),
        # a set without certified bytes: speculative cuts
        dict(name="refused_32m", kind="scan", set="refused", n=32 << 20, call="into", offsets=False, stray=False),
        # malformed text: the scan halts at a stray byte past the middle
        dict(name="stray_64m", kind="scan", set="clike_l", n=64 << 20, call="into", offsets=False, stray=True),
        # records framed by a reserved byte
        dict(name="framed_64m", kind="scan", set="framed", n=(64 << 20) + 13, call="into", offsets=False, stray=False),
        # an editor's index: start offsets beside kinds and lengths
        dict(name="clike_l_100m_offsets", kind="scan", set="clike_l", n=100_000_003, call="into", offsets=True,
             stray=False),
        # the JSON configuration of the benchmark
        dict(name="json_256m", kind="scan", set="json", n=256 << 20, call="into", offsets=False, stray=False),
        # the headline configuration of the benchmark
        dict(name="clike_l_512m", kind="scan", set="clike_l", n=512 << 20, call="into", offsets=False, stray=False),
        # one batch of a serving slot
        dict(name="batch_16", kind="batch", sets="serving", docs=16, median=8192, sigma=1.5, offsets=False),
        # a corpus of documents in one batch, some of them of a refused set
        dict(name="batch_16k", kind="batch", sets="corpus", docs=16384, median=16384, sigma=1.5, offsets=False),
    ]


def draw(rng):
    if rng.random() < 0.3:
        return dict(kind="batch", sets=rng.choice(["serving", "corpus"]), docs=int(2 ** rng.uniform(0, 13)),
                    median=rng.choice([2048, 8192, 16384]), sigma=1.5, offsets=rng.random() < 0.2)
    name = rng.choice(["clike_l", "clike_l", "clike_d", "json", "framed", "refused"])
    offsets = rng.random() < 0.25
    n = int(2 ** rng.uniform(10, 25 if name == "refused" else 27))
    if rng.random() < 0.25:
        n = max(1024, n >> 12 << 12)
    call = rng.choice(["static", "into"]) if n <= 4 << 20 else "into"
    return dict(kind="scan", set=name, n=n, call=call, offsets=offsets, stray=name in ("clike_l", "clike_d") and rng.random() < 0.15)


# ------------------------------------------------------------------------------------- text
def _geo(r, mean):
    return max(1, math.ceil(math.log(1.0 - r.random()) / math.log(1.0 - 1.0 / mean)))


def _poisson(r, mean):
    k, p, lim = -1, 1.0, math.exp(-mean)
    while p > lim:
        k += 1
        p *= r.random()
    return k


def _clike_line(r, blocks):
    out = []
    for t in range(_poisson(r, 8.0)):
        if t:
            out.append("".join(" " if r.random() < 0.9 else "\t" for _ in range(r.randint(1, 4))))
        u = r.random() * (0.90 if blocks else 0.85)
        if u < 0.35:
            out.append(r.choice(ALPHA) + "".join(r.choices(ALNUM, k=_geo(r, 6.0) - 1)))
        elif u < 0.50:
            out.append("".join(r.choices("0123456789", k=_geo(r, 3.0))))
        elif u < 0.75:
            out.append(r.choice(OPS))
        elif u < 0.80:
            out.append('"' + "".join(r.choice(STRCH) if r.random() < 0.9 else "\\" + r.choice('ntr0"\\')
                                     for _ in range(_geo(r, 9.0) - 1)) + '"')
        elif u < 0.85:
            out.append("//" + "".join(r.choices(PRINT, k=_geo(r, 21.0) - 1)))
            break
        else:
            body, prev = [], "*"
            for _ in range(_geo(r, 41.0) - 1):
                c = "\n" if r.random() < 0.05 else r.choice(PRINT)
                if prev == "*" and c == "/":
                    c = " "
                body.append(c)
                prev = c
            out.append("/*" + "".join(body) + "*/")
    return "".join(out) + "\n"


def _json_value(r, depth):
    u = r.random()
    if u >= 0.8 and depth >= 6:
        u = r.random() * 0.8
    if u < 0.4:
        s = "".join(r.choice(STRCH) if r.random() < 0.95 else
                    (r.choice(['\\"', "\\\\", "\\/", "\\b", "\\f", "\\n", "\\r", "\\t"]) if r.random() < 8 / 9 else
                     "\\u" + "".join(r.choices("0123456789abcdefABCDEF", k=4))) for _ in range(_geo(r, 13.0) - 1))
        return '"' + s + '"'
    if u < 0.7:
        s = "-" if r.random() < 0.3 else ""
        s += "0" if r.random() < 0.1 else str(r.randint(1, 9)) + "".join(r.choices("0123456789", k=r.randint(0, 5)))
        if r.random() < 0.4:
            s += "." + "".join(r.choices("0123456789", k=r.randint(1, 6)))
        if r.random() < 0.1:
            s += r.choice("eE") + r.choice(["+", "-", ""]) + "".join(r.choices("0123456789", k=r.randint(1, 3)))
        return s
    if u < 0.8:
        return r.choice(["true", "false", "null"])
    return _json_container(r, depth)


def _json_container(r, depth):
    obj = r.random() < 0.5
    pad = " " * (2 * (depth + 1))
    items = []
    for _ in range(r.randint(1, 8)):
        key = '"' + "".join(r.choices(ALPHA[:52], k=r.randint(3, 12))) + '": ' if obj else ""
        items.append(pad + key + _json_value(r, depth + 1))
    return ("{\n" if obj else "[\n") + ",\n".join(items) + "\n" + " " * (2 * depth) + ("}" if obj else "]")


class _Pool:
    """Pieces of text (lines, records, JSON values), drawn from the seed; a corpus is a random
    sequence of them, put together on the GPU."""

    def __init__(self, texts, seed, pieces):
        made, self.first = [], {}
        for k, text in enumerate(texts):
            r = random.Random(seed * 16 + k)
            self.first[text] = len(made)
            for _ in range(pieces):
                if text == "json":
                    made.append(_json_container(r, 0) + "\n")
                elif text == "records":
                    made.append("\x1e" + "".join(_clike_line(r, True) for _ in range(8)))
                else:
                    made.append(_clike_line(r, text == "blocks"))
        made = [m.encode("latin-1") for m in made]
        self.pieces = pieces
        self.lens = np.array([len(m) for m in made], np.int64)
        self.starts = np.cumsum(self.lens) - self.lens
        self.bytes = torch.from_numpy(np.frombuffer(b"".join(made), np.uint8).copy()).cuda()

    def mean(self, text):
        f = self.first[text]
        return float(self.lens[f: f + self.pieces].mean())

    def fill(self, out, picks, at):
        """Writes piece picks[i] at out[at[i]] (out: a uint8 device tensor)."""
        step = max(1, int((1 << 24) / self.lens.mean()))  # about 16 MiB at a time, to bound the indexes
        for a in range(0, picks.size, step):
            p, to = picks[a: a + step], at[a: a + step]
            lens, total = self.lens[p], int(self.lens[p].sum())
            begin = np.cumsum(lens) - lens
            move = torch.from_numpy(np.stack([self.starts[p] - begin, to - begin], 1)).cuda()
            i = torch.arange(total, device="cuda")
            k = torch.repeat_interleave(move, torch.from_numpy(lens).cuda(), dim=0, output_size=total)
            out[i + k[:, 1]] = self.bytes[i + k[:, 0]]


def _text(text, n, seed, stray):
    pool = _Pool([text], seed, 1500 if n > 1 << 20 else 300)
    rng = np.random.default_rng(seed)
    picks = rng.integers(0, pool.pieces, int(n / pool.mean(text) * 1.05) + 64)
    ends = np.cumsum(pool.lens[picks])
    while ends[-1] < n:
        picks = np.concatenate([picks, picks])
        ends = np.cumsum(pool.lens[picks])
    k = int(np.searchsorted(ends, n, side="right"))  # whole pieces only, padded with newlines
    out = torch.full((n,), 0x0A, dtype=torch.uint8, device="cuda")
    if k:
        pool.fill(out, picks[:k], ends[:k] - pool.lens[picks[:k]])
        if stray:  # a byte that starts no token, at a piece's start past the middle
            out[int(ends[min(k - 1, int(k * 0.6))])] = 0x01
    return out


def _documents(case, seed):
    names = SERVING if case["sets"] == "serving" else CORPUS
    texts = sorted({SETS[k][2] for k in names})
    pool = _Pool(texts, seed, 600)
    nd = case["docs"]
    sizes = np.random.default_rng(nd)  # a case's documents have the same sizes whatever the seed
    size = case["median"] * np.exp(case["sigma"] * sizes.standard_normal(nd))
    size = np.clip(size, 64, 4 << 20).astype(np.int64)
    rng = np.random.default_rng(seed)
    inst = rng.choice(3, nd, p=[1 / 3] * 3 if case["sets"] == "serving" else [0.475, 0.475, 0.05])
    mean = np.array([pool.mean(SETS[k][2]) for k in names])
    first = np.array([pool.first[SETS[k][2]] for k in names])
    pieces = (size / mean[inst] * 1.1).astype(np.int64) + 8
    picks = np.repeat(first[inst], pieces) + rng.integers(0, pool.pieces, int(pieces.sum()))
    # each document's pieces from its start on, the whole ones that fit, padded with newlines
    before = np.cumsum(pool.lens[picks]) - pool.lens[picks]
    at = before - np.repeat(before[np.cumsum(pieces) - pieces], pieces)
    fits = at + pool.lens[picks] <= np.repeat(size, pieces)
    docs = np.zeros(nd, P.DOC_DTYPE)
    docs["offset"] = np.cumsum(size) - size
    docs["length"] = size
    docs["inst"] = inst
    at += np.repeat(docs["offset"].astype(np.int64), pieces)
    data = torch.full((int(size.sum()),), 0x0A, dtype=torch.uint8, device="cuda")
    pool.fill(data, picks[fits], at[fits])
    return names, data, docs


# ------------------------------------------------------------------------------------- calls
def _compile(name):
    defs = SETS[name][0]
    return P.Lexer.compile_framed(defs, 0x1E) if name == "framed" else P.Lexer.compile(defs)


def _outputs(s, cap, offsets):
    s["kinds"] = torch.zeros(max(cap, 1), dtype=torch.uint8, device="cuda")
    s["lens"] = torch.zeros(max(cap, 1), dtype=torch.int32, device="cuda")
    s["offs"] = torch.zeros(max(cap, 1), dtype=torch.int64, device="cuda") if offsets else None


def prepare(case, seed):
    s = {"kind": case["kind"], "call": case.get("call"), "offsets": case["offsets"]}
    if case["kind"] == "batch":
        names, s["data"], docs = _documents(case, seed)
        s["batch"] = P.Batch([(_compile(k), SETS[k][1]) for k in names])
        n = s["n"] = s["data"].numel()
        s["docs"] = torch.from_numpy(docs.view(np.uint8).copy()).cuda()
        s["ndocs"] = docs.size
        _outputs(s, n, case["offsets"])
        s["res"] = torch.zeros(docs.size * 4, dtype=torch.int64, device="cuda")
        s["total"] = torch.zeros(3, dtype=torch.int64, device="cuda")
        s["ws"] = torch.empty(s["batch"].workspace_size(docs.size, n), dtype=torch.uint8, device="cuda")
        return s
    s["lexer"] = _compile(case["set"])
    s["mode"] = SETS[case["set"]][1]
    n = s["n"] = case["n"]
    s["data"] = _text(SETS[case["set"]][2], n, seed, case["stray"])
    _outputs(s, n, case["offsets"])
    s["result"] = torch.zeros(3, dtype=torch.int64, device="cuda")
    if case["call"] == "into":
        s["ws"] = torch.empty(s["lexer"].workspace_size(n, s["mode"]), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    if s["kind"] == "batch":
        s["batch"].run_into(s["data"], s["n"], s["docs"], s["ndocs"], s["kinds"], s["lens"], s["offs"], s["n"],
                            s["res"], s["total"], s["ws"])
        return s["kinds"], s["lens"], s["offs"], s["res"], s["total"]
    if s["call"] == "static":
        s["lexer"].run_static_into(s["data"], s["n"], s["mode"], s["kinds"], s["lens"], s["offs"], s["n"],
                                   s["result"])
    else:
        s["lexer"].run_into(s["data"], s["n"], s["mode"], s["kinds"], s["lens"], s["offs"], s["n"], s["result"],
                            s["ws"])
    return s["kinds"], s["lens"], s["offs"], s["result"]


def work(case):
    """Each input byte read once, each token's kind, length (and start offset) written once."""
    per = 13 if case["offsets"] else 5
    if case["kind"] == "batch":
        names = SERVING if case["sets"] == "serving" else CORPUS
        n = case["docs"] * case["median"] * math.exp(case["sigma"] ** 2 / 2) * 0.95
        share = sum(SETS[k][3] for k in names[:2]) / 2 if case["sets"] == "corpus" else sum(SETS[k][3] for k in names) / 3
        return {"bytes": n * (1 + per * share) + 48 * case["docs"], "flops": 0}
    n, share = case["n"], SETS[case["set"]][3]
    return {"bytes": n * (1 + per * share * (0.6 if case["stray"] else 1)) + 24, "flops": 0}
