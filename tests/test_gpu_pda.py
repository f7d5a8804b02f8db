"""GPU parity of push-down constraints (tdfa_compile_token_pda, tdfa_pda_step) against the oracle,
through the C ABI: the set of token edges and, step by step, tokens, states and stacks."""
import numpy as np
import pytest
import torch

from workloads import configs, logits as LG, pda as P, vocab as V

pytestmark = pytest.mark.gpu
F32, BF16 = 0, 1


@pytest.fixture(scope="module")
def T():
    import paper_2407_08103_amd as T
    assert torch.cuda.is_available()
    return T


def _handle(T, pda):
    return T.CharPDA(pda.n_states, pda.start, pda.accept, pda.src, pda.input, pda.dst, pda.pop_begin, pda.pop_syms,
                     pda.push_begin, pda.push_syms)


def _vocab(rng, alphabet: bytes, n_random: int, extra, max_len=7):
    toks = set(extra)
    alpha = np.frombuffer(alphabet, dtype=np.uint8)
    while len(toks) < n_random + len(set(extra)):
        toks.add(bytes(alpha[rng.integers(0, len(alpha), size=int(rng.integers(1, max_len + 1)))]))
    toks = sorted(toks)
    rng.shuffle(toks)
    return toks


def _edge_set(first, token, dst, n_pops, pops, n_push, pushes):
    out = set()
    for q in range(len(first) - 1):
        for e in range(int(first[q]), int(first[q + 1])):
            out.add((q, int(token[e]), tuple(pops[e, :n_pops[e]].tolist()), int(dst[e]), tuple(pushes[e, :n_push[e]].tolist())))
    return out


def _compile_both(T, oracle, pda, toks):
    vocab = V.from_tokens(toks)
    want = oracle.pda_compile(pda, vocab.data, vocab.offsets)
    table = T.compile_token_pda(T.Vocab(vocab.data, vocab.offsets), _handle(T, pda))
    arrs = table.arrays()
    first, token = arrs[0], arrs[1]
    assert table.n_edges == len(want) == int(first[-1])
    assert _edge_set(*arrs) == want.as_set()
    for q in range(pda.n_states):                              # sorted by token inside a state; unused places are -1
        seg = token[int(first[q]):int(first[q + 1])]
        assert (np.diff(seg) >= 0).all()
    assert ((arrs[4] >= 0).sum(axis=1) == arrs[3]).all() and ((arrs[6] >= 0).sum(axis=1) == arrs[5]).all()
    order = np.argsort(want.src, kind="stable")
    want = oracle.TokenEdges(*[getattr(want, k)[order] for k in ("src", "token", "dst", "n_pops", "pops", "n_push", "pushes")])
    return table, want, vocab


CASES = [
    ("anbn", P.anbn, b"ab", 40, [b"a", b"b", b"bb", b"aaab", b""]),
    ("dyck2", P.dyck2, b"()[]", 300, [b"", b"(" * 11, b")" * 11, b"([" * 6 + b"])" * 6]),
    ("int_lists", P.int_lists, b"0123456789[],", 1027, [b"", b"[[[[", b"]]]]", b"],["]),
    ("call_grammar", P.call_grammar, b"foobar(123)456", 500, [b"foo(123)", b"r(4", b"o(1", b""]),
]


@pytest.mark.parametrize("name,make,alphabet,n_random,extra", CASES)
def test_token_edges(T, oracle, name, make, alphabet, n_random, extra):
    rng = np.random.default_rng(len(name) * 31 + n_random)
    toks = _vocab(rng, alphabet, n_random, extra)
    table, want, _ = _compile_both(T, oracle, make(), toks)
    assert table.n_edges > 0


def test_fig7_edges_on_device(T, oracle):
    """The worked example of Figs. 6-7: the hand-derived edges, on the device."""
    table, want, _ = _compile_both(T, oracle, P.anbn(), [b"a", b"b", b"bb", b"aaab"])
    got = _edge_set(*table.arrays())
    assert (2, 2, (1, 1), 2, ()) in got and (0, 3, (), 2, (1, 1)) in got and len(got) == 10


def test_regular_special_case(T, oracle):
    """An automaton that never touches its stack: the token edges are the live entries of delta_T."""
    w = configs.get("c1")
    d = w.dfas[0]
    pda = P.dfa_as_pda(d.trans, d.accept, d.start)
    table = T.compile_token_pda(T.Vocab(w.vocab.data, w.vocab.offsets), _handle(T, pda))
    tab = oracle.compile_walk(d.trans, w.vocab.data, w.vocab.offsets)
    want = {(int(q), int(t), (), int(tab[q, t]), ()) for q, t in zip(*np.nonzero(tab >= 0))}
    assert _edge_set(*table.arrays()) == want


def test_errors(T):
    bad = P.make_pda(3, 0, [2], [(0, P.EPS, (), 1, ()), (0, "a", (), 2, ())])
    with pytest.raises(T.TdfaError) as e:
        _handle(T, bad)
    assert e.value.code == -1 and "not deterministic" in str(e.value)
    loop = P.make_pda(2, 0, [1], [(0, P.EPS, (0,), 0, (0,)), (1, "a", (), 1, ())])
    v = V.from_tokens([b"a", b"b"])
    with pytest.raises(T.TdfaError) as e:
        T.compile_token_pda(T.Vocab(v.data, v.offsets), _handle(T, loop))
    assert e.value.code == -4 and "epsilon" in str(e.value)
    deep = P.make_pda(1, 0, [0], [(0, "a", (), 0, (1, 1, 1, 1, 1))])
    v = V.from_tokens([b"aa", b"aaa"])
    with pytest.raises(T.TdfaError) as e:
        T.compile_token_pda(T.Vocab(v.data, v.offsets), _handle(T, deep))
    assert e.value.code == -4 and "12" in str(e.value)


def _decode(T, oracle, pda, table, want, n_tokens, dtype, batch, steps, cap, seed, sigma=2.0, masked_every=3, odd_stride=False, all_ones_at=()):
    rng = np.random.default_rng(seed)
    states_np = np.full(batch, pda.start, dtype=np.int32)
    stacks_np = np.full((batch, cap), -7, dtype=np.int32)
    stacks_np[:, 0] = P.S0
    depths_np = np.ones(batch, dtype=np.int32)
    states = torch.from_numpy(states_np.copy()).cuda()
    stacks = torch.from_numpy(stacks_np.copy()).cuda()
    depths = torch.from_numpy(depths_np.copy()).cuda()
    tokens = torch.empty(batch, dtype=torch.int32, device="cuda")
    stride = (n_tokens + 7) // 8 * 8 + (1 if odd_stride else 0)     # odd: rows that 16-byte loads cannot take
    n_tok_total = 0
    for s in range(steps):
        x = np.zeros((batch, stride), dtype=np.float32)
        x[:, :n_tokens] = np.round(rng.normal(0, sigma, size=(batch, n_tokens)), 1)       # rounded: ties do occur
        if s == 2:
            x[:, ::3] = np.nan
        lg_np = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        if s in all_ones_at:
            lg_np.view(np.uint32 if dtype == F32 else np.uint16)[:] = 0xFFFFFFFF if dtype == F32 else 0xFFFF
        lg = torch.from_numpy(lg_np).cuda() if dtype == F32 else torch.from_numpy(lg_np.view(np.int16)).cuda().view(torch.bfloat16)
        want_masked = s % masked_every == 0
        out = torch.empty_like(lg) if want_masked else None
        T.pda_step(table, lg, states, stacks, depths, tokens, states, out)
        torch.cuda.synchronize()
        res = oracle.pda_step(pda.n_states, n_tokens, want, lg_np, dtype, states_np, stacks_np, depths_np, row_stride=stride,
                              want_masked=want_masked)
        states_np = res[1]
        assert np.array_equal(tokens.cpu().numpy(), res[0]), f"step {s}: tokens differ"
        assert np.array_equal(states.cpu().numpy(), states_np), f"step {s}: states differ"
        assert np.array_equal(depths.cpu().numpy(), depths_np), f"step {s}: depths differ"
        got_st = stacks.cpu().numpy()
        for b in range(batch):
            assert np.array_equal(got_st[b, :depths_np[b]], stacks_np[b, :depths_np[b]]), f"step {s}: stack of sequence {b} differs"
        if want_masked:
            got = out.cpu().numpy() if dtype == F32 else out.view(torch.int16).cpu().numpy().view(np.uint16)
            ref = res[2] if dtype == F32 else res[2]
            assert np.array_equal(got.view(np.uint32 if dtype == F32 else np.uint16)[:, :n_tokens],
                                  ref.view(np.uint32 if dtype == F32 else np.uint16)[:, :n_tokens]), f"step {s}: masked rows differ"
        n_tok_total += int((res[0] >= 0).sum())
    return n_tok_total


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("name,make,alphabet,n_random,extra", CASES[1:3])
def test_decode_steps(T, oracle, dtype, name, make, alphabet, n_random, extra):
    """Chained steps: tokens, states, stacks and the penalised rows at every step; small stacks, so that some
    sequences end because their stack is full."""
    rng = np.random.default_rng(7)
    toks = _vocab(rng, alphabet, n_random, extra)
    pda = make()
    table, want, vocab = _compile_both(T, oracle, pda, toks)
    n = _decode(T, oracle, pda, table, want, len(toks), dtype, batch=33, steps=30, cap=9, seed=11)
    assert n > 100


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("n_tokens,batch", [(63, 5), (64, 5), (65, 200), (129, 3), (8191, 3), (33000, 4), (33000, 16), (33000, 128), (33000, 129), (33000, 200), (33000, 300),
                                            (51512, 128), (51513, 128)])
def test_traversal_at_the_edges_of_the_directory(T, oracle, dtype, n_tokens, batch):
    """Vocabularies around the 64 tokens of a directory entry, rows that one and that several workgroups share, and the
    row whose token the exact scan decides (step 2: NaN); the step without a penalised row traverses the edge itself."""
    rng = np.random.default_rng(n_tokens + batch)
    ones = [b"(", b")", b"[", b"]"]
    toks = ones + [t for t in _vocab(rng, b"()[]x", n_tokens, [], 7 if n_tokens < 40000 else 9) if t not in ones][:n_tokens - 4]
    assert len(toks) == n_tokens
    rng.shuffle(toks)
    pda = P.dyck2()
    table, want, n = _compile_both(T, oracle, pda, toks)
    _decode(T, oracle, pda, table, want, len(toks), dtype, batch, 4, 24, 7, masked_every=100)


@pytest.mark.parametrize("n_tokens,batch", [(8191, 3), (33000, 4), (33000, 200), (33000, 300)])
def test_rows_of_the_smallest_key(T, oracle, n_tokens, batch):
    """Steps on rows that are the NaN pattern 0xFFFF throughout, whose order key is 0: all wavefronts of a workgroup
    then have the same candidate, and one of them may speak for it; the step after finds the words through which
    workgroups meet as they should be."""
    rng = np.random.default_rng(n_tokens)
    toks = [t for t in _vocab(rng, b"abcdefgh()", n_tokens, [], 7) if t][:n_tokens]
    letters = [(0, chr(c), (), 0, ()) for c in b"abcdefgh"]                # most tokens are letters alone: always allowed
    pda = P.make_pda(1, 0, [0], letters + [(0, "(", (), 0, (1,)), (0, ")", (1,), 0, ())])
    table, want, _ = _compile_both(T, oracle, pda, toks)
    _decode(T, oracle, pda, table, want, len(toks), BF16, batch, 5, 24, 7, masked_every=100, all_ones_at=(1, 2, 4))


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_decode_steps_rows_not_16_byte_aligned(T, oracle, dtype):
    """The same chained steps with a row stride that the step kernel's 16-byte loads cannot take: the step then
    scans the edges of the state."""
    name, make, alphabet, n_random, extra = CASES[2]
    rng = np.random.default_rng(7)
    toks = _vocab(rng, alphabet, n_random, extra)
    pda = make()
    table, want, vocab = _compile_both(T, oracle, pda, toks)
    n = _decode(T, oracle, pda, table, want, len(toks), dtype, batch=33, steps=20, cap=9, seed=12, odd_stride=True)
    assert n > 60


@pytest.mark.parametrize("dtype,with_out", [(F32, True), (BF16, True), (BF16, False), (F32, False)])
def test_decode_special_configurations(T, oracle, dtype, with_out):
    """States that are no state, depths outside the buffer, a stack that is full, flat and NaN logits; with and
    without the penalised rows (16-bit logits without them: the step kernel finds the classes of edges itself)."""
    pda = P.anbn()
    toks = [b"a", b"b", b"bb", b"aaab"]
    table, want, _ = _compile_both(T, oracle, pda, toks)
    cap, R = 8, 1
    cfgs = [(0, [0]), (1, [0]), (1, [0, R]), (2, [0, R]), (2, [0, R, R]), (2, [0]), (4, [0]), (-1, [0]), (7, [0]), (1, [0] + [R] * 7)]
    B = len(cfgs)
    for kind in ("up", "flat", "nan"):
        x = {"up": np.tile(np.arange(8, dtype=np.float32), (B, 1)), "flat": np.zeros((B, 8), np.float32),
             "nan": np.full((B, 8), np.nan, np.float32)}[kind]
        states_np = np.array([c[0] for c in cfgs], dtype=np.int32)
        stacks_np = np.full((B, cap), -7, dtype=np.int32)
        depths_np = np.zeros(B, dtype=np.int32)
        for i, (_, s) in enumerate(cfgs):
            stacks_np[i, :len(s)] = s
            depths_np[i] = len(s)
        depths_np[8] = cap + 3
        states, stacks, depths = (torch.from_numpy(a.copy()).cuda() for a in (states_np, stacks_np, depths_np))
        tokens = torch.full((B,), -9, dtype=torch.int32, device="cuda")
        new = torch.full((B,), -9, dtype=torch.int32, device="cuda")
        lg_np = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        lg = torch.from_numpy(lg_np).cuda() if dtype == F32 else torch.from_numpy(lg_np.view(np.int16)).cuda().view(torch.bfloat16)
        out = torch.empty_like(lg) if with_out else None
        T.pda_step(table, lg, states, stacks, depths, tokens, new, out)
        torch.cuda.synchronize()
        res = oracle.pda_step(pda.n_states, 4, want, lg_np, dtype, states_np, stacks_np, depths_np, row_stride=8, want_masked=with_out)
        assert np.array_equal(tokens.cpu().numpy(), res[0]) and np.array_equal(new.cpu().numpy(), res[1]), kind
        assert np.array_equal(depths.cpu().numpy(), depths_np) and np.array_equal(stacks.cpu().numpy(), stacks_np), kind
        if with_out:
            bits = np.uint32 if dtype == F32 else np.uint16
            got = out.cpu().numpy() if dtype == F32 else out.view(torch.int16).cpu().numpy()
            assert np.array_equal(got.view(bits)[:, :4], res[2].view(bits)[:, :4]), kind
    with pytest.raises(T.TdfaError):
        T.pda_step(table, lg, states, stacks, depths, tokens, new, lg)         # the penalised row may not be the logits


def test_json_grammar_with_c2_vocabulary(T, oracle):
    """A nested JSON grammar against the 32,000-token vocabulary of the JSON workload: all token edges, then 64
    chained steps at batch 64 with bf16 logits, every step checked."""
    w = configs.get("c2")
    pda = P.json_like()
    want = oracle.pda_compile(pda, w.vocab.data, w.vocab.offsets)
    table = T.compile_token_pda(T.Vocab(w.vocab.data, w.vocab.offsets), _handle(T, pda))
    assert _edge_set(*table.arrays()) == want.as_set() and table.n_edges > 5000
    order = np.argsort(want.src, kind="stable")
    want = oracle.TokenEdges(*[getattr(want, k)[order] for k in ("src", "token", "dst", "n_pops", "pops", "n_push", "pushes")])
    assert int(want.n_pops.max()) >= 3 and int(want.n_push.max()) >= 2          # tokens that close or open several containers
    n = _decode(T, oracle, pda, table, want, w.vocab.n_tokens, BF16, batch=64, steps=64, cap=24, seed=3, masked_every=16)
    assert n > 64 * 32


def _decode_sampled(T, oracle, pda, table, want, n_tokens, dtype, batch, steps, cap, seed, temperature, top_k=0, sigma=2.0,
                    masked_every=4):
    """Chained drawn steps: tokens, states, stacks (and the penalised rows now and then) against the oracle at every step."""
    rng = np.random.default_rng(seed)
    states_np = np.full(batch, pda.start, dtype=np.int32)
    stacks_np = np.full((batch, cap), -7, dtype=np.int32)
    stacks_np[:, 0] = P.S0
    depths_np = np.ones(batch, dtype=np.int32)
    states, stacks, depths = (torch.from_numpy(a.copy()).cuda() for a in (states_np, stacks_np, depths_np))
    tokens = torch.empty(batch, dtype=torch.int32, device="cuda")
    stride = (n_tokens + 7) // 8 * 8
    n_tok_total = 0
    for s in range(steps):
        x = np.zeros((batch, stride), dtype=np.float32)
        x[:, :n_tokens] = np.round(rng.normal(0, sigma, size=(batch, n_tokens)), 1)
        if s == 2:
            x[:, ::3] = np.nan
        lg_np = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        lg = torch.from_numpy(lg_np).cuda() if dtype == F32 else torch.from_numpy(lg_np.view(np.int16)).cuda().view(torch.bfloat16)
        want_masked = s % masked_every == 1
        out = torch.empty_like(lg) if want_masked else None
        T.pda_sample_step(table, lg, states, stacks, depths, temperature, 11 + seed, s, tokens, states, out, top_k=top_k)
        torch.cuda.synchronize()
        res = oracle.pda_sample_step(pda.n_states, n_tokens, want, lg_np, dtype, states_np, stacks_np, depths_np, temperature,
                                     11 + seed, s, top_k=top_k, row_stride=stride, want_masked=want_masked)
        states_np = res[1]
        assert np.array_equal(tokens.cpu().numpy(), res[0]), f"step {s}: tokens differ"
        assert np.array_equal(states.cpu().numpy(), states_np), f"step {s}: states differ"
        assert np.array_equal(depths.cpu().numpy(), depths_np), f"step {s}: depths differ"
        got_st = stacks.cpu().numpy()
        for b in range(batch):
            assert np.array_equal(got_st[b, :depths_np[b]], stacks_np[b, :depths_np[b]]), f"step {s}: stack of sequence {b} differs"
        if want_masked:
            bits = np.uint32 if dtype == F32 else np.uint16
            got = out.cpu().numpy() if dtype == F32 else out.view(torch.int16).cpu().numpy()
            assert np.array_equal(got.view(bits)[:, :n_tokens], res[2].view(bits)[:, :n_tokens]), f"step {s}: masked rows differ"
        n_tok_total += int((res[0] >= 0).sum())
    return n_tok_total


@pytest.mark.parametrize("dtype,temperature,top_k", [(BF16, 1.0, 0), (F32, 0.7, 0), (BF16, 1.5, 3)])
@pytest.mark.parametrize("name,make,alphabet,n_random,extra", CASES[1:3])
def test_sampled_decode_steps(T, oracle, dtype, temperature, top_k, name, make, alphabet, n_random, extra):
    """The step of Algorithm 3 with the token drawn: every step of a chained decode against the oracle."""
    rng = np.random.default_rng(7)
    toks = _vocab(rng, alphabet, n_random, extra)
    pda = make()
    table, want, vocab = _compile_both(T, oracle, pda, toks)
    n = _decode_sampled(T, oracle, pda, table, want, len(toks), dtype, batch=33, steps=24, cap=9, seed=5, temperature=temperature,
                        top_k=top_k)
    assert n > 80


def test_sampled_json_grammar_with_c2_vocabulary(T, oracle):
    """Drawn steps under the nested JSON grammar with the 32,000-token vocabulary, batch 64, bf16, every step checked; and
    what the call refuses."""
    w = configs.get("c2")
    pda = P.json_like()
    want = oracle.pda_compile(pda, w.vocab.data, w.vocab.offsets)
    table = T.compile_token_pda(T.Vocab(w.vocab.data, w.vocab.offsets), _handle(T, pda))
    order = np.argsort(want.src, kind="stable")
    want = oracle.TokenEdges(*[getattr(want, k)[order] for k in ("src", "token", "dst", "n_pops", "pops", "n_push", "pushes")])
    n = _decode_sampled(T, oracle, pda, table, want, w.vocab.n_tokens, BF16, batch=64, steps=40, cap=24, seed=3, temperature=1.0,
                        masked_every=16)
    assert n > 64 * 20
    B, V_ = 4, w.vocab.n_tokens
    lg = torch.zeros((B, V_), dtype=torch.bfloat16, device="cuda")
    st = torch.zeros(B, dtype=torch.int32, device="cuda")
    stk = torch.zeros((B, 8), dtype=torch.int32, device="cuda")
    dp = torch.ones(B, dtype=torch.int32, device="cuda")
    tok = torch.empty(B, dtype=torch.int32, device="cuda")
    for bad in (dict(temperature=0.0), dict(temperature=-1.0), dict(temperature=1.0, top_k=-2)):
        with pytest.raises(T.TdfaError):
            T.pda_sample_step(table, lg, st, stk, dp, bad["temperature"], 1, 0, tok, st, top_k=bad.get("top_k", 0))
    odd = torch.zeros((B, V_ + 1), dtype=torch.bfloat16, device="cuda")[:, :V_]
    with pytest.raises(T.TdfaError) as e:                     # rows that 16-byte loads cannot take
        T.pda_sample_step(table, odd, st, stk, dp, 1.0, 1, 0, tok, st)
    assert e.value.code == -4
