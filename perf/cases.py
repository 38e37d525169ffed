"""The work that a serving program has this library do, as measurable cases.

Four kinds of pass, each through the package's public entry points:

* ``decode``: ``steps`` steps of ``Handle.apply_mask`` on that step's logits and
  ``Handle.advance`` over the sampled tokens, on a handle compiled beforehand;
  with rows built on demand the row cache is emptied first (``Handle.rebuild``),
  as a new batch of requests finds it;
* ``compile``: ``compile`` of a set (or a forest of per-query sets) against a
  vocabulary built beforehand, then the decode steps on the new handle;
* ``format``: ``compile_format`` of a fixed-format value, then the decode steps;
* ``step``: the benchmark's step: ``Handle.rebuild`` (the masks of every node from
  the resident tables), one ``apply_mask`` and one ``advance``.

The strings are word strings (tool names) or code-like strings (a code list's
lines), the vocabulary 256 byte tokens and substrings of a corpus of the same
kind, as in the benchmark's configurations.  Everything is drawn from the seed but
the tokenizer (the vocabulary) and the pool that code-like strings are picked
from, which a deployment has once.
"""
import functools
import math

import numpy as np
import torch

import paper_2608_12574_amd as tam

T = b'"'  # closes every string
POOL = 74719  # code-like strings that sets are picked from
VMAX = 262144
DTYPES = {"fp32": torch.float32, "bf16": torch.bfloat16}
# representations: a dense table, sparse lists, tail compression, tail
# compression without a table, rows built on demand
FLAGS = {"dense": 0, "lists": tam.FLAG_NO_TABLE, "tail": tam.FLAG_TAIL_LISTS,
         "tail_lists": tam.FLAG_TAIL_LISTS | tam.FLAG_NO_TABLE, "lazy": tam.FLAG_LAZY_ROWS}
D, H = b"0123456789", b"0123456789abcdef"
DATE = [D] * 4 + [b"-"] + [D] * 2 + [b"-"] + [D] * 2
FORMATS = {
    "date": DATE,
    "datetime": DATE + [b"T"] + [D] * 2 + [b":"] + [D] * 2 + [b":"] + [D] * 2,
    "uuid": [H] * 8 + [b"-"] + [H] * 4 + [b"-", b"4"] + [H] * 3 + [b"-", b"89ab"] + [H] * 3 + [b"-"] + [H] * 12,
}


def listed():
    def case(name, kind, text, K, S, V, B, dtype, rep, steps, start):
        return dict(name=name, kind=kind, text=text, K=K, S=S, V=V, B=B, dtype=dtype, rep=rep, steps=steps,
                    start=start)
    return [
        # one request choosing among 100 names: the smallest calls, launches and host time
        case("decode-one", "decode", "words", 100, 1, 32000, 1, "fp32", "dense", 8, "root"),
        # a mid-size batch over a tool list and a vocabulary of odd size, so that
        # the rows of the contiguous logits are not 16-byte aligned
        case("decode-ragged", "decode", "words", 1000, 1, 128255, 64, "fp32", "dense", 8, "uniform"),
        # a full batch decoding from the root of a large name list
        case("decode-words", "decode", "words", 10000, 1, 151936, 256, "bf16", "dense", 16, "root"),
        # a full batch anywhere in a code list, tail compression
        case("decode-codes", "decode", "codes", 10000, 1, 262144, 256, "bf16", "tail", 8, "uniform"),
        # a full batch with a set of its own per request
        case("decode-forest", "decode", "codes", 500, 256, 262144, 256, "bf16", "tail_lists", 16, "root"),
        # the same batch size over one code list, masks only where decoding goes
        case("decode-lazy", "decode", "codes", 10000, 1, 262144, 256, "bf16", "lazy", 16, "root"),
        # one query's set compiled and used at once
        case("compile-query", "compile", "codes", 500, 1, 262144, 1, "bf16", "tail_lists", 4, "root"),
        # a large name list compiled to a full table, then its first steps
        case("compile-words", "compile", "words", 10000, 1, 151936, 256, "bf16", "dense", 4, "root"),
        # the per-query sets of a whole batch compiled together, then the first steps
        case("compile-forest", "compile", "codes", 500, 256, 262144, 256, "bf16", "tail_lists", 4, "root"),
        # a fixed-format value compiled and decoded
        case("format-uuid", "format", "uuid", 0, 1, 262144, 64, "bf16", "dense", 8, "root"),
        # the benchmark's steps: the full table of a code list, and the forest
        case("step-codes", "step", "codes", 10000, 1, 262144, 256, "bf16", "dense", 1, "uniform"),
        case("step-forest", "step", "codes", 500, 256, 262144, 256, "bf16", "tail_lists", 1, "root"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Any kind, text and representation; sizes over the listed cases' ranges, odd ones among them."""
    kind = rng.choice(["decode", "decode", "compile", "compile", "step", "format"])
    text = rng.choice(list(FORMATS)) if kind == "format" else rng.choice(["words", "codes"])
    forest = kind != "format" and rng.random() < 0.35
    S = _log(rng, 2, 256) if forest else 1
    K = 0 if kind == "format" else _log(rng, 20, 500) if forest else _log(rng, 100, 10000)
    V = _log(rng, 32000, VMAX)
    if rng.random() < 0.6:
        V = V // 64 * 64
    B = _log(rng, 1, 256)
    rep = rng.choice(["lists", "tail_lists", "lazy"] if forest else ["dense", "tail", "tail_lists", "lazy"])
    if kind == "format":
        rep = "dense"
    if kind == "step" and rep == "lazy":  # nothing to rebuild but the cache
        rep = "tail_lists"
    steps = 1 if kind == "step" else rng.randint(2, 8)
    return dict(kind=kind, text=text, K=K, S=S, V=V, B=B, dtype=rng.choice(["bf16", "fp32"]), rep=rep, steps=steps,
                start=rng.choice(["root", "uniform"]) if rep != "lazy" else "root")


# ------------------------------------------------------------------ inputs ---

@functools.lru_cache(maxsize=None)
def _lexicon():
    """5,000 lowercase words of 3 to 8 letters, and the Zipf weights of their ranks."""
    rng = np.random.default_rng(1)
    words = {}
    while len(words) < 5000:
        n = int(rng.integers(3, 9))
        words[bytes(rng.integers(97, 123, size=n, dtype=np.uint8))] = None
    return list(words), np.arange(1, 5001, dtype=np.float64) ** -1.1


def _words(rng, K, lo, hi):
    """K distinct strings of lo..hi Zipf words joined by '_', two in five with a verb in front."""
    lex, p = _lexicon()
    L = 200 if K < 500 else 1000 if K < 5000 else 5000
    p = p[:L] / p[:L].sum()
    out = {}
    while len(out) < K:
        n = rng.integers(lo, hi + 1, size=K)
        pick = rng.choice(L, size=(K, hi), p=p)
        verb = rng.integers(0, 8, size=K)
        for i in range(K):
            s = b"_".join([lex[j] for j in pick[i, :n[i]]])
            if verb[i] < 3:
                s = (b"get_", b"list_", b"create_")[verb[i]] + s
            out[s] = None
            if len(out) == K:
                break
    return list(out)


def _codes(rng, n, max_len=64):
    """n code-like lines: a letter, two digits, perhaps '.' and 1 to 4 of [0-9A-Z], ' - ', 3 to 8 Zipf words."""
    lex, p = _lexicon()
    p = p / p.sum()
    AN = b"0123456789ABCDEFGHIJKLMNOPQRSTUVWXYZ"
    lead, dig, dot = rng.integers(0, 26, size=n), rng.integers(0, 100, size=n), rng.random(n) < 0.5
    nf, frag = rng.integers(1, 5, size=n), rng.integers(0, 36, size=(n, 4))
    nw, pick = rng.integers(3, 9, size=n), rng.choice(5000, size=(n, 8), p=p)
    out = []
    for i in range(n):
        s = b"%c%02d" % (65 + lead[i], dig[i])
        if dot[i]:
            s += b"." + bytes(AN[j] for j in frag[i, :nf[i]])
        s += b" - " + b" ".join([lex[j] for j in pick[i, :nw[i]]])
        out.append(s if len(s) <= max_len else s[:s.rindex(b" ", 0, max_len + 1)])
    return out


@functools.lru_cache(maxsize=None)
def _pool():
    rng, out = np.random.default_rng(2), {}
    while len(out) < POOL:
        out.update(dict.fromkeys(_codes(rng, 20000)))
    return list(out)[:POOL]


@functools.lru_cache(maxsize=None)
def _tokens(text):
    """The tokenizer's VMAX tokens: the 256 bytes, for codes 16,384 fragments, then substrings of 2 to 16 bytes."""
    rng = np.random.default_rng(3 if text == "words" else 4)
    seen = dict.fromkeys(bytes([b]) for b in range(256))
    if text == "words":
        lex, p = _lexicon()
        pick = rng.choice(5000, size=1200000, p=p / p.sum())
        sep = rng.integers(0, 2, size=pick.size)
        corpus = b"".join([lex[j] + (b"_", b" ")[s] for j, s in zip(pick.tolist(), sep.tolist())])
    else:
        AN = np.frombuffer(b"0123456789ABCDEFGHIJKLMNOPQRSTUVWXYZ", dtype=np.uint8)
        while len(seen) < 256 + 16384:
            seen[AN[rng.integers(0, 36, size=int(rng.integers(2, 7)))].tobytes()] = None
        corpus = b"\n".join(_codes(rng, 160000))
    while len(seen) < VMAX:
        n = rng.integers(2, 17, size=VMAX)
        at = rng.integers(0, len(corpus) - 16, size=VMAX)
        for a, k in zip(at.tolist(), n.tolist()):
            seen[corpus[a:a + k]] = None
            if len(seen) == VMAX:
                break
    return list(seen)


def _pack(items):
    off = np.zeros(len(items) + 1, dtype=np.int64)
    np.cumsum(np.fromiter(map(len, items), dtype=np.int64, count=len(items)), out=off[1:])
    return np.frombuffer(b"".join(items), dtype=np.uint8), off


@functools.lru_cache(maxsize=None)
def _packed_tokens(text):
    return _pack(_tokens(text))


def _vocab(case):
    blob, off = _packed_tokens("words" if case["text"] == "words" else "codes")
    return tam.Vocab((blob, off[:case["V"] + 1]))


def _strings(case, seed):
    """The sets' strings, set after set, packed, and the sets' offsets (None: one set)."""
    rng = np.random.default_rng([seed, 5])
    K, S = case["K"], case["S"]
    out = []
    for _ in range(S):
        if case["text"] == "words":
            out += _words(rng, K, 2, 3 if K < 500 else 5)
        else:
            pool = _pool()
            out += [pool[i] for i in rng.choice(POOL, size=K, replace=False).tolist()]
    return out, (None if S == 1 else np.arange(S + 1, dtype=np.int64) * K)


# ------------------------------------------------------------------- passes ---

def _compile(st):
    if st["kind"] == "format":
        return tam.compile_format(st["classes"], st["vocab"])
    return tam.compile(st["strings"], st["vocab"], sets=st["sets"], flags=st["flags"])


def prepare(case, seed):
    """The vocabulary, the packed strings, the logits of every step, and the node and token ids a
    decode by argmax over those logits meets (rows begin again at their root when they have ended)."""
    B, V, steps = case["B"], case["V"], case["steps"]
    st = dict(kind=case["kind"], flags=FLAGS[case["rep"]], rep=case["rep"], vocab=_vocab(case))
    if case["kind"] == "format":
        st["classes"] = FORMATS[case["text"]]
    else:
        strings, st["sets"] = _strings(case, seed)
        st["strings"] = _pack(strings)
    g = torch.Generator(device="cuda").manual_seed(seed)
    st["logits"] = torch.empty((steps, B, V), dtype=DTYPES[case["dtype"]], device="cuda")
    for t in range(steps):
        st["logits"][t].normal_(generator=g)
    h = _compile(st)
    roots = torch.as_tensor(h.roots, device="cuda")[torch.arange(B, device="cuda") % h.num_sets].contiguous()
    final = torch.as_tensor(h.is_final, device="cuda").bool()
    st["nodes"], st["tokens"] = [], []
    n = roots
    for t in range(steps):
        if case["start"] == "uniform":
            n = torch.randint(0, h.num_nodes, (B,), dtype=torch.int32, device="cuda", generator=g)
        x = h.apply_mask(n, st["logits"][t].clone())
        v = x.argmax(dim=1).to(torch.int32)
        st["nodes"].append(n)
        st["tokens"].append(v)
        n = h.advance(n, v)
        n = torch.where((n < 0) | final[n.clamp(min=0).long()], roots, n)
    st["handle"] = None
    if case["kind"] in ("decode", "step"):
        st["handle"] = h
    return st


def run(st):
    """One pass; returns the masked logits of every step and the advanced nodes."""
    h = st["handle"]
    if h is None:
        h = _compile(st)
    elif st["kind"] == "step" or st["rep"] == "lazy":
        h.rebuild()
    states = []
    for n, v, x in zip(st["nodes"], st["tokens"], st["logits"]):
        h.apply_mask(n, x)
        states.append(h.advance(n, v))
    return {"logits": st["logits"], "states": states}


def _nodes(case):
    """Trie nodes of the case's sets (of one seed): a root per set and each string's bytes beyond its
    common prefix with the string before it, the closing byte included."""
    if case["kind"] == "format":
        return len(FORMATS[case["text"]]) + 2
    strings, _ = _strings(case, 0)
    total = case["S"]
    for j in range(case["S"]):
        a = np.array(sorted(s + T for s in strings[j * case["K"]:(j + 1) * case["K"]]))
        m = a.view(np.uint8).reshape(len(a), -1)
        lens = np.char.str_len(a)
        lcp = np.cumprod(m[1:] == m[:-1], axis=1).sum(axis=1)
        total += int(lens.sum() - np.minimum(lcp, np.minimum(lens[1:], lens[:-1])).sum())
    return total


def work(case):
    """Per step a mask row read and a row of logits written for each batch row; a dense table is written
    once; for other representations one word per trie node; a compile reads its strings."""
    W = (case["V"] + 63) // 64 * 8
    size = 2 if case["dtype"] == "bf16" else 4
    nbytes = case["steps"] * case["B"] * (W + case["V"] * size + 12)
    if case["kind"] != "decode":
        N = _nodes(case)
        nbytes += N * (W if case["rep"] == "dense" else 4)
        if case["kind"] == "compile":
            nbytes += sum(map(len, _strings(case, 0)[0]))
    return {"bytes": nbytes, "flops": 0}


def tolerance(case):
    """Logits are moved or replaced by -inf, never computed: every bit is fixed by the strings."""
    return "exact"


def exact(case, seed):
    """Nothing is computed in floating point, so there is nothing to hold against 64 bits."""
    return None
