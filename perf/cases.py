"""What a user of the library has it do, as cases that can be timed and compared.

A case is a dict of plain values.  `prepare` makes what a program holds before the call (a
vocabulary handle, automata, compiled tables, logits), `run` makes the calls, `work` says what a
pass cannot do without, and `exact` gives the outputs from plain torch.  The automata stand for the
constraints that the library is used with: one call of a tiny function, a choice of function
signatures, JSON objects of given fields, nested JSON as a push-down grammar, and a random
automaton as the hard case of compilation; logits are those of a language model in scale and size
(normal, standard deviation 2).  All outputs are whole numbers or copies of input bits, so they
are compared exactly.
"""
import math

import numpy as np
import torch

import paper_2407_08103_amd as T

WORDS = ("alpha bravo charlie delta echo foxtrot golf hotel india juliet kilo lima mike november oscar papa "
         "quebec romeo sierra tango uniform victor whiskey xray yankee zulu").split()
LOWER = b"abcdefghijklmnopqrstuvwxyz"
DIGITS = b"0123456789"
IN_STRING = bytes(c for c in range(256) if c not in b'"\\')
PRINTABLE = bytes(range(0x20, 0x7F))
# the bytes that a constraint names: seven in ten bytes of its vocabulary's tokens come from here
ALPHABET = {"call": LOWER + b'(x=")', "functions": LOWER + DIGITS + b'_()=,"-', "schemas": LOWER + DIGITS + b'_"{}:,.+-E \n',
            "grammar": LOWER + DIGITS + b'_ "[]{}:,-'}
# the share of a row's logits that lie in a group of eight with an allowed token among them, over the states that such sequences are in
SHARE = {"call": 0.26, "functions": 0.35, "schemas": 0.38, "grammar": 0.60}


# ----------------------------------------------------------------- the cases
def listed():
    return [
        # one short call checked in a notebook: nothing but latency and launches
        dict(name="step_tiny_f32", path="step", constraint="call", n=1, vocab=512, batch=4, dtype="f32", masked=False),
        # an ordinary decode step of a server: function calls, every sequence somewhere in its text
        dict(name="step_functions_256", path="step", constraint="functions", n=50, vocab=128256, batch=256, dtype="bf16", masked=False),
        # the largest decode step: a constraint of its own for each of 64 groups of sequences
        dict(name="step_schemas_1024", path="step", constraint="schemas", n=64, vocab=128256, batch=1024, dtype="bf16", masked=False),
        # the penalised logits handed on to the caller's own sampler, in fp32
        dict(name="step_masked_f32_64", path="step", constraint="functions", n=50, vocab=128256, batch=64, dtype="f32", masked=True),
        # a draw at a temperature over the whole allowed set
        dict(name="sample_functions_256", path="sample", constraint="functions", n=50, vocab=128256, batch=256, dtype="bf16",
             temperature=1.0, top_k=0),
        # the usual sampler settings of a chat server: a temperature below one and a top-k cut
        dict(name="sample_topk_256", path="sample", constraint="functions", n=50, vocab=128256, batch=256, dtype="bf16",
             temperature=0.7, top_k=50),
        # nested JSON: the push-down step with a stack per sequence
        dict(name="grammar_256", path="grammar", vocab=128256, batch=256, dtype="bf16", temperature=0.0, top_k=0, masked=False),
        # speculative decoding: seven drafted tokens per sequence followed and all eight positions masked, on a packed table
        dict(name="verify_64x7_packed", path="verify", constraint="functions", n=50, vocab=128256, batch=64, k=7, dtype="bf16", packed=True),
        # a request brings a schema of its own: upload, preparation and compilation, from host arrays
        dict(name="new_schema_32000", path="new", constraint="schemas", n=1, vocab=32000),
        # the table of an ordinary large constraint, from an automaton that is already uploaded
        dict(name="compile_functions", path="compile", constraint="functions", n=50, vocab=128256),
        # the largest table: an automaton without any structure, a vocabulary of arbitrary bytes
        dict(name="compile_random_20000", path="compile", constraint="random", n=20000, vocab=256000),
        # a finished table made small for serving: minimised, then packed
        dict(name="finish_functions", path="finish", constraint="functions", n=50, vocab=128256),
    ]


def draw(rng):
    def spread(lo, hi):
        return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))

    path = rng.choice(["step", "step", "sample", "sample", "grammar", "verify", "new", "compile", "compile", "finish"])
    constraint = rng.choice(["functions", "schemas"])
    n = spread(2, 50) if constraint == "functions" else spread(1, 64)
    c = dict(path=path, vocab=spread(512, 128256))
    if path != "grammar":
        c.update(constraint=constraint, n=n)
    if path in ("step", "sample", "grammar", "verify"):
        c.update(dtype=rng.choice(["bf16", "bf16", "f32"]))
    if path == "step":
        c.update(batch=spread(1, 1024), masked=rng.random() < 0.3)
        if rng.random() < 0.1:
            c.update(constraint="call", n=1)
    elif path == "sample":
        c.update(batch=spread(1, 512), temperature=round(rng.uniform(0.3, 1.3), 2), top_k=rng.choice([0, spread(1, 200)]))
    elif path == "grammar":
        drawn = rng.random() < 0.4
        c.update(batch=spread(1, 512), temperature=round(rng.uniform(0.3, 1.3), 2) if drawn else 0.0,
                 top_k=rng.choice([0, spread(1, 200)]) if drawn else 0, masked=rng.random() < 0.2)
    elif path == "verify":
        c.update(batch=spread(1, 128), k=rng.randint(1, 8), packed=rng.random() < 0.5)
    elif path == "compile" and rng.random() < 0.3:
        c.update(constraint="random", n=spread(200, 20000), vocab=spread(512, 256000))
    return c


# ----------------------------------------------------------------- automata
class _Rows:
    """A deterministic automaton that grows state by state."""

    def __init__(self):
        self.rows, self.final = [], []

    def new(self, accept=False):
        self.rows.append(np.full(256, -1, dtype=np.int32))
        self.final.append(accept)
        return len(self.rows) - 1

    def edge(self, sources, symbols, target):
        for s in sources if isinstance(sources, list) else [sources]:
            self.rows[s][list(symbols)] = target
        return target

    def literal(self, s, text):
        for ch in text:
            to = self.rows[s][ch]
            s = int(to) if to >= 0 else self.edge(s, [ch], self.new())
        return s

    def run_of(self, s, first, more, count):
        """One symbol of `first`, then up to count - 1 of `more`; the states in which it may end."""
        ends = []
        for i in range(count):
            s = self.edge(s, more if i else first, self.new())
            ends.append(s)
        return ends

    def number(self, s, digits):
        sign = self.edge(s, b"-", self.new())
        ends = self.run_of(s, DIGITS, DIGITS, digits)
        self.edge(sign, DIGITS, ends[0])
        return ends

    def string(self, s, length):
        s, end = self.edge(s, b'"', self.new()), self.new()
        for _ in range(length):
            self.edge(s, b'"', end)
            s = self.edge(s, IN_STRING, self.new())
        self.edge(s, b'"', end)
        return [end]

    def space(self, states, blank):
        for s in states:
            self.edge(s, b" \n", blank)
        self.edge(blank, b" \n", blank)
        return states + [blank]

    def done(self):
        return np.stack(self.rows), np.array(self.final, dtype=np.uint8), 0


def _call():
    """One call of a one-argument function: [a-z]{1,8}\\(x="[a-z]*"\\)."""
    a = _Rows()
    ends = a.run_of(a.new(), LOWER, LOWER, 8)
    s = a.literal(a.edge(ends, b"(", a.new()), b'x="')
    a.edge(s, LOWER, s)
    a.edge(a.literal(s, b'"'), b")", a.new(accept=True))
    return a.done()


def _name(r, lo, hi):
    return bytes(r.choice(list(LOWER), size=int(r.integers(lo, hi + 1))).astype(np.uint8))


def _functions(r, count):
    """A choice of function signatures name(arg=value,...) with one to six arguments: an integer, a
    string of up to 32 bytes or an identifier of up to 20."""
    a = _Rows()
    root, final, names = a.new(), a.new(accept=True), set()
    while len(names) < count:
        name = _name(r, 4, 10)
        if name in names:
            continue
        names.add(name)
        s = a.literal(root, name + b"(")
        args = int(r.integers(1, 7))
        for i in range(args):
            s = a.literal(s, _name(r, 3, 8) + b"=")
            kind = int(r.integers(0, 3))
            ends = (a.number(s, 9) if kind == 0 else a.string(s, 32) if kind == 1 else
                    a.run_of(s, LOWER + b"_", LOWER + DIGITS + b"_", 20))
            s = a.edge(ends, b",", a.new()) if i < args - 1 else a.edge(ends, b")", final)
    return a.done()


def _schema(r):
    """A JSON object with four to ten given fields in a fixed order and white space between tokens."""
    a = _Rows()
    fields = int(r.integers(4, 11))
    digits, length, frac = int(r.integers(2, 13)), int(r.choice([16, 32, 64, 96])), int(r.integers(1, 9))
    s = a.edge(a.new(), b"{", a.new())
    for i, word in enumerate(r.choice(len(WORDS), size=fields, replace=False)):
        a.space([], s)
        name = WORDS[word] + ("_" + WORDS[int(r.integers(0, len(WORDS)))] if r.random() < 0.5 else "")
        before = a.space([a.literal(s, b'"' + name.encode() + b'"')], a.new())
        s = a.edge(before, b":", a.new())
        a.space([], s)
        kind = i if i < 2 else int(r.integers(0, 5))
        if kind == 0:
            ends = a.number(s, digits)
        elif kind == 1:
            ends = a.string(s, length)
        elif kind == 2:
            ends = [a.literal(s, b"true"), a.literal(s, b"false")]
        elif kind == 3:
            quoted = a.literal(s, b'"')
            ends = [a.literal(a.literal(quoted, WORDS[int(w)].encode()), b'"') for w in r.choice(len(WORDS), size=4, replace=False)]
        else:
            point = a.edge(a.number(s, digits), b".", a.new())
            ends = a.run_of(point, DIGITS, DIGITS, frac)
            power = a.edge(ends, b"eE", a.new())
            sign = a.edge(power, b"+-", a.new())
            last = a.run_of(power, DIGITS, DIGITS, 2)
            a.edge(sign, DIGITS, last[0])
            ends += last
        after = a.space(ends, a.new())
        s = a.edge(after, b"," if i < fields - 1 else b"}", a.new(accept=i == fields - 1))
    return a.done()


def _random(r, n):
    """A random automaton: seven in ten transitions missing."""
    trans = r.integers(0, n, size=(n, 256), dtype=np.int32)
    trans[r.random((n, 256), dtype=np.float32) < 0.7] = -1
    return trans, (r.random(n) < 0.1).astype(np.uint8), 0


def _relabelling(seed):
    """Which letter stands for which under this seed: constraints and vocabularies of two seeds differ by
    this and by the order of the token ids, so their tables have the same number of rows and edges."""
    to = np.arange(256)
    low = np.frombuffer(LOWER, dtype=np.uint8)
    to[low] = np.random.default_rng([seed, 1]).permutation(low)
    return to


def _automata(case, seed):
    """The automata (trans, accept, start) of a case, in the order of their rows in a stacked table."""
    kind = case["constraint"]
    if kind == "random":
        return [_random(np.random.default_rng([seed, 3]), case["n"])]
    r = np.random.default_rng([case["n"], 1])
    made = [_call()] if kind == "call" else [_functions(r, case["n"])] if kind == "functions" else [_schema(r) for _ in range(case["n"])]
    letters = np.argsort(_relabelling(seed))
    return [(np.ascontiguousarray(trans[:, letters]), accept, start) for trans, accept, start in made]


def _grammar():
    """Nested JSON (arrays, objects, strings, integers, true, false, null) as a push-down automaton
    with one stack symbol per open container above the bottom symbol 0: the arguments of CharPDA,
    and its states by what they stand for."""
    bottom, arr, obj = 0, 1, 2
    names = ("begin end first value key_or_close key in_key colon string digits zero minus after "
             "t tr tru f fa fal fals n nu nul").split()
    at = {s: i for i, s in enumerate(names)}
    edges = []

    def add(source, symbols, target, pops=(), pushes=()):
        for ch in symbols:
            edges.append((at[source], ch, pops, at[target], pushes))

    for s in ("begin", "first", "value"):
        add(s, b"[", "first", (), (arr,))
        add(s, b"{", "key_or_close", (), (obj,))
    for s in ("first", "value"):
        add(s, b'"', "string")
        add(s, b"-", "minus")
        for word in ("true", "false", "null"):
            add(s, word[:1].encode(), word[:1])
    for s in ("first", "value", "minus"):
        add(s, b"0", "zero")
        add(s, DIGITS[1:], "digits")
    add("digits", DIGITS, "digits")
    for word in ("true", "false", "null"):
        for i in range(1, len(word)):
            add(word[:i], word[i].encode(), word[:i + 1] if i < len(word) - 1 else "after")
    for s in ("string", "in_key"):
        add(s, LOWER + DIGITS + b"_ ", s)
    add("string", b'"', "after")
    add("in_key", b'"', "colon")
    add("colon", b":", "value")
    add("key_or_close", b'"', "in_key")
    add("key", b'"', "in_key")
    for s in ("after", "digits", "zero"):
        add(s, b",", "value", (arr,), (arr,))
        add(s, b",", "key", (obj,), (obj,))
    for sources, ch, top in ((("first", "after", "digits", "zero"), b"]", arr), (("key_or_close", "after", "digits", "zero"), b"}", obj)):
        for s in sources:
            add(s, ch, "end", (bottom, top), (bottom,))
            for below in (arr, obj):
                add(s, ch, "after", (below, top), (below,))
    edges.sort(key=lambda e: e[0])
    accept = np.zeros(len(names), dtype=np.uint8)
    accept[at["end"]] = 1

    def begins(k):
        return np.cumsum([0] + [len(e[k]) for e in edges])

    def symbols(k):
        return np.array([x for e in edges for x in e[k]], dtype=np.int32)

    src, sym, dst = (np.array([e[k] for e in edges], dtype=np.int32) for k in (0, 1, 3))
    return (len(names), at["begin"], accept, src, sym, dst, begins(2), symbols(2), begins(4), symbols(4)), at


# ----------------------------------------------------------------- vocabularies
def _vocabulary(case, seed):
    """Distinct tokens (bytes, offsets): single bytes, then strings whose lengths follow a Zipf law,
    seven in ten of their bytes from the constraint's alphabet; for the random automaton uniform
    bytes.  Token ids are in no order.  Also the bytes as a matrix, and the lengths."""
    kind, n = case.get("constraint", "grammar"), case["vocab"]
    r = np.random.default_rng([n, 2])
    if kind == "random":
        lo, hi, law, singles, alphabet, share = 1, 32, 1.05, b"", bytes(range(256)), 1.0
    elif kind == "call":
        lo, hi, law, singles, alphabet, share = 2, 8, 0.0, PRINTABLE, PRINTABLE, 1.0
    else:
        lo, hi, law, singles, alphabet, share = 2, 24, 1.1, bytes(range(256)), ALPHABET[kind], 0.7
    alphabet = np.frombuffer(alphabet, dtype=np.uint8)
    other = np.setdiff1d(np.frombuffer(PRINTABLE, dtype=np.uint8), alphabet)
    weights = np.arange(1, hi - lo + 2) ** -law
    mult = r.integers(1, 1 << 62, size=hi + 1).astype(np.uint64)
    text = np.zeros((len(singles), hi), dtype=np.uint8)
    text[:, 0] = np.frombuffer(singles, dtype=np.uint8)
    lens = np.ones(len(singles), dtype=np.int64)
    while True:
        with np.errstate(over="ignore"):
            key = (text * mult[None, :hi]).sum(axis=1, dtype=np.uint64) + lens.astype(np.uint64) * mult[hi]
        keep = np.sort(np.unique(key, return_index=True)[1])[:n]
        text, lens = text[keep], lens[keep]
        if len(lens) == n:
            break
        more = int((n - len(lens)) * 1.5) + 64
        ls = r.choice(np.arange(lo, hi + 1), size=more, p=weights / weights.sum())
        t = alphabet[r.integers(0, len(alphabet), size=(more, hi))]
        if share < 1.0:
            t = np.where(r.random((more, hi), dtype=np.float32) < share, t, other[r.integers(0, len(other), size=(more, hi))])
        t[np.arange(hi)[None, :] >= ls[:, None]] = 0
        text, lens = np.concatenate([text, t]), np.concatenate([lens, ls])
    order = np.random.default_rng([seed, 2]).permutation(n)
    text, lens = text[order], lens[order]
    if kind != "grammar":
        text = _relabelling(seed).astype(np.uint8)[text]
    offsets = np.zeros(n + 1, dtype=np.uint64)
    offsets[1:] = np.cumsum(lens)
    return text[np.arange(hi)[None, :] < lens[:, None]], offsets, text, lens


# ----------------------------------------------------------------- prepare and run
def _generator(seed, what):
    return torch.Generator(device="cuda").manual_seed(seed * 16 + what)


def _logits(case, rows, seed, what=3):
    """[rows, vocabulary] as a language model's head leaves them: rows padded to a multiple of 64 columns."""
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    x = torch.randn((rows, -(-case["vocab"] // 64) * 64), generator=_generator(seed, what), device="cuda")
    return (x * 2.0).to(dtype)


def _states(case, offsets, batch, seed):
    """A state for each sequence: anywhere in the text of its constraint; sequence b has constraint b mod n."""
    r = np.random.default_rng([seed, 4])
    c = np.arange(batch) % (len(offsets) - 1)
    q = offsets[c] + (r.random(batch) * (offsets[c + 1] - offsets[c])).astype(np.int64)
    return torch.from_numpy(q.astype(np.int32)).cuda()


def _int32(*shape):
    return torch.empty(shape, dtype=torch.int32, device="cuda")


def _uploaded(automata):
    """The automaton of all constraints together, and where each one's rows begin."""
    if len(automata) == 1:
        return T.CharDFA(*automata[0]), np.array([0, len(automata[0][0])], dtype=np.int64)
    return T.dfa_union_host(automata)


def prepare(case, seed):
    path = case["path"]
    data, offsets, _, _ = _vocabulary(case, seed)
    s = {"case": case, "vocab": T.Vocab(data, offsets)}
    if path == "grammar":
        args, at = _grammar()
        s["table"] = T.compile_token_pda(s["vocab"], T.CharPDA(*args))
        b, cap = case["batch"], 32
        r = np.random.default_rng([seed, 5])
        depth = r.integers(1, 8, size=b)                              # open containers
        stacks = np.zeros((b, cap), dtype=np.int32)
        stacks[:, 1:] = np.where(np.arange(1, cap)[None, :] <= depth[:, None], r.integers(1, 3, size=(b, cap - 1)), 0)
        in_object = stacks[np.arange(b), depth] == 2
        most = r.random(b)                                            # most of a text lies inside strings
        anywhere = r.choice([at[x] for x in ("value", "colon", "digits", "after", "minus", "fa", "nu")], size=b)
        q = np.where(most < 0.45, at["string"], np.where(most < 0.7, np.where(in_object, at["in_key"], at["string"]), anywhere))
        q = np.where(~in_object & (q == at["colon"]), at["value"], q)
        s["states"] = torch.from_numpy(q.astype(np.int32)).cuda()
        s["before"] = torch.from_numpy(np.concatenate([stacks.reshape(-1), depth.astype(np.int32) + 1]).astype(np.int32)).cuda()
        s["now"] = torch.empty_like(s["before"])                      # stacks and depths, which a step updates
        s["stacks"], s["depths"] = s["now"][:b * cap].view(b, cap), s["now"][b * cap:]
        s["logits"] = _logits(case, b, seed)
        s["tokens"], s["next"] = _int32(b), _int32(b)
        s["masked"] = torch.empty_like(s["logits"]) if case["masked"] else None
        return s
    automata = _automata(case, seed)
    if path == "new":
        s["automata"] = automata
        return s
    s["dfa"], rows = _uploaded(automata)
    if path == "compile":
        return s
    s["table"] = T.compile_token_dfa(s["vocab"], s["dfa"])
    if path == "finish":
        s["accept"] = np.concatenate([a[1] for a in automata])
        s["starts"] = rows[:-1].astype(np.int32)
        return s
    b = case["batch"]
    s["states"] = _states(case, rows, b, seed)
    if path in ("step", "sample"):
        s["logits"] = _logits(case, b, seed)
        s["tokens"], s["next"] = _int32(b), _int32(b)
        s["masked"] = torch.empty_like(s["logits"]) if case.get("masked") else None
        return s
    # verify: the drafts are what a constrained draft model would say, one in five of them replaced
    k = case["k"]
    s["drafts"], s["history"], s["valid"] = _int32(b, k), _int32(b, k + 1), _int32(b)
    q, tok = s["states"].clone(), _int32(b)
    g = _generator(seed, 6)
    for i in range(k):
        T.mask_step(s["table"], _logits(case, b, seed * 8 + i, 7), q, tok, q)
        other = torch.randint(0, case["vocab"], (b,), generator=g, device="cuda", dtype=torch.int32)
        s["drafts"][:, i] = torch.where(torch.rand(b, generator=g, device="cuda") < 0.2, other, tok)
    if case["packed"]:
        s["table"] = T.table_pack(s["table"])
    s["logits"] = _logits(case, b * (k + 1), seed)
    s["tokens"], s["next"] = _int32(b * (k + 1)), _int32(b * (k + 1))
    return s


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "step":
        T.mask_step(s["table"], s["logits"], s["states"], s["tokens"], s["next"], s["masked"])
        return [s["tokens"], s["next"]] + ([s["masked"][:, :case["vocab"]]] if case["masked"] else [])
    if path == "sample":
        T.sample_step(s["table"], s["logits"], s["states"], case["temperature"], 1234, 56, s["tokens"], s["next"], top_k=case["top_k"])
        return [s["tokens"], s["next"]]
    if path == "grammar":
        s["now"].copy_(s["before"])                                    # the step moves the stacks in place
        if case["temperature"] > 0:
            T.pda_sample_step(s["table"], s["logits"], s["states"], s["stacks"], s["depths"], case["temperature"], 1234, 56, s["tokens"],
                              s["next"], s["masked"], top_k=case["top_k"])
        else:
            T.pda_step(s["table"], s["logits"], s["states"], s["stacks"], s["depths"], s["tokens"], s["next"], s["masked"])
        return [s["tokens"], s["next"], s["now"]] + ([s["masked"][:, :case["vocab"]]] if case["masked"] else [])
    if path == "verify":
        T.advance_tokens(s["table"], s["states"], s["drafts"], s["history"], s["valid"])
        T.mask_step(s["table"], s["logits"], s["history"].view(-1), s["tokens"], s["next"])
        return [s["history"], s["valid"], s["tokens"], s["next"]]
    if path == "finish":
        small, accept, state_map = T.table_minimize(s["table"], s["accept"], s["starts"])
        return [accept, state_map] + list(T.table_pack_arrays(T.table_pack(small)))
    dfa = _uploaded(s["automata"])[0] if path == "new" else s["dfa"]
    table = T.compile_token_dfa(s["vocab"], dfa)
    return [table.delta, table.allow]


# ----------------------------------------------------------------- what a pass cannot do without
def work(case):
    v, path = case["vocab"], case["path"]
    size = 2 if case.get("dtype") == "bf16" else 4
    share = SHARE.get(case.get("constraint", "grammar"), 1.0)
    if path in ("step", "sample", "grammar"):
        logits = case["batch"] * v * size
        moved = logits * (2 if case.get("masked") else share) + case["batch"] * v / 8
        return {"bytes": moved, "flops": case["batch"] * v * share}
    if path == "verify":
        rows = case["batch"] * (1 + 0.55 * case["k"])                   # positions behind a refused draft hold no state
        return {"bytes": rows * v * (size * share + 1 / 8), "flops": rows * v * share}
    if case["constraint"] == "random":
        rows, edges = case["n"], case["n"] * 77
    else:
        rows = sum(len(a[0]) for a in _automata(case, 0))
        edges = rows * 64
    table = rows * (v * 4 + v / 8)
    if path == "finish":                                                # the table read once, its edges (a third) and bits written
        return {"bytes": table + rows * v * (4 / 3 + 1 / 8 + 1 / 32), "flops": rows * v}
    return {"bytes": table + edges * 4 + 6 * v, "flops": rows * v}


def tolerance(case):
    # every output is a whole number, or logits copied bit for bit and -inf
    return "exact"


# ----------------------------------------------------------------- the same in plain torch
def _walk(trans, states, text, lens):
    """Where `states` [m] end after each token's bytes: int32 [m, tokens], -1 = nowhere.  A token
    without bytes leads nowhere."""
    n = trans.shape[0]
    full = torch.full((n + 1, 256), n, dtype=torch.int32, device="cuda")
    full[:n] = torch.where(trans >= 0, trans, n)
    cur = torch.where(states >= 0, states, n).to(torch.int32)[:, None].expand(-1, len(lens)).contiguous()
    for i in range(int(lens.max())):
        at = torch.nonzero(lens > i).view(-1)
        part = cur[:, at].long() * 256 + text[at, i][None, :]
        cur[:, at] = full.view(-1)[part]
    cur[:, lens == 0] = n
    return torch.where(cur < n, cur, -1)


def _joined(automata):
    base, parts = 0, []
    for trans, _, _ in automata:
        parts.append(np.where(trans >= 0, trans + base, -1))
        base += len(trans)
    return torch.from_numpy(np.concatenate(parts).astype(np.int32)).cuda()


def _best(case, rows, states, logits):
    """Greedy tokens, next states and penalised logits of table rows [b, vocabulary]."""
    x = torch.where(rows >= 0, logits[:, :case["vocab"]].double(), -math.inf)
    ids = torch.arange(case["vocab"], device="cuda")
    first = torch.where((rows >= 0) & (x == x.max(dim=1, keepdim=True).values), ids, case["vocab"]).min(dim=1).values
    none = first == case["vocab"]
    to = rows.gather(1, torch.where(none, 0, first)[:, None])[:, 0]
    return torch.where(none, -1, first).int(), torch.where(none, states, to).int(), x


def exact(case, seed):
    path = case["path"]
    if path in ("sample", "grammar", "finish") or case["constraint"] == "random" and case["n"] * case["vocab"] > 1 << 30:
        return None
    _, _, text, lens = _vocabulary(case, seed)
    text, lens = torch.from_numpy(text).cuda().long(), torch.from_numpy(lens).cuda()
    automata = _automata(case, seed)
    trans = _joined(automata)
    if path in ("new", "compile"):
        width = 4 * -(-case["vocab"] // 128)
        delta = torch.empty((len(trans), case["vocab"]), dtype=torch.int32, device="cuda")
        for r0 in range(0, len(trans), 256):
            delta[r0:r0 + 256] = _walk(trans, torch.arange(r0, min(r0 + 256, len(trans)), device="cuda"), text, lens)
        bits = torch.zeros((len(trans), width * 32), dtype=torch.bool, device="cuda")
        bits[:, :case["vocab"]] = delta >= 0
        words = (bits.view(len(trans), width, 32).long() << torch.arange(32, device="cuda")).sum(dim=2)
        return [delta, words.int()]
    rows = np.cumsum([0] + [len(a[0]) for a in automata])
    states = _states(case, rows, case["batch"], seed)
    if path == "step":
        best = _best(case, _walk(trans, states, text, lens), states, _logits(case, case["batch"], seed))
        return list(best if case["masked"] else best[:2])
    return None                                                        # verify: its drafts are made with the library
