"""GPU parity of the token-level optimisation against the oracle, bit for bit (new table, allowed
bits, state map, final states), and decode steps on the optimised table."""
import numpy as np
import pytest
import torch

from workloads import configs, logits as LG, vocab as V
from workloads.regex_dfa import compile_regex
import gpu_util as G

pytestmark = pytest.mark.gpu
DEAD = -1
BF16 = 1


@pytest.fixture(scope="module")
def T():
    import paper_2407_08103_amd as T
    assert torch.cuda.is_available()
    return T


def _upload_table(T, table_np):
    delta = torch.from_numpy(np.ascontiguousarray(table_np)).cuda()
    rw = T.allow_row_words(table_np.shape[1])
    allow = torch.from_numpy(G.bits_from_table(table_np, rw).view(np.int32)).cuda()
    return T.table_wrap(delta, allow)


def _as_torch(T, table):
    """A library-owned table copied into torch buffers (one-table concat = plain copy)."""
    out, _ = T.table_concat([table])
    torch.cuda.synchronize()
    return out


def _check(T, oracle, table, table_np, accept, starts):
    new, acc, mp = T.table_minimize(table, accept, starts)
    want, want_acc, want_mp = oracle.minimize(table_np, accept, starts)
    assert np.array_equal(mp, want_mp)
    assert new.n_rows == want.shape[0] and np.array_equal(acc, want_acc)
    if new.n_rows:
        G.check_rows(_as_torch(T, new), want, np.arange(want.shape[0]))
    return new, want, mp


def test_fig4_example(T, oracle):
    d = compile_regex(r"(foo)+d")
    vocab = V.from_tokens([b"f", b"oo", b"foo", b"for", b"food"])
    table = T.compile_token_dfa(T.Vocab(vocab.data, vocab.offsets), T.CharDFA(d.trans, d.accept, d.start))
    table_np = oracle.compile_walk(d.trans, vocab.data, vocab.offsets)
    new, want, mp = _check(T, oracle, table, table_np, d.accept, [d.start])
    assert mp.tolist() == [0, 1, DEAD, 0, 2] and want.tolist() == [[1, -1, 0, -1, 2], [-1, 0, -1, -1, -1], [-1] * 5]


@pytest.mark.parametrize("seed", range(6))
def test_random_tables(T, oracle, seed):
    rng = np.random.default_rng(100 + seed)
    n, v = int(rng.integers(2, 200)), int(rng.integers(1, 700))
    table_np = rng.integers(0, n, size=(n, v), dtype=np.int32)
    table_np[rng.random((n, v)) < (0.5 + 0.08 * seed)] = DEAD
    # classes to merge: blocks of states that share their row and their flag
    for q in range(n // 2, n):
        table_np[q] = table_np[q % max(1, n // 4)]
    accept = (rng.random(n) < 0.3).astype(np.uint8)
    for q in range(n // 2, n):
        accept[q] = accept[q % max(1, n // 4)]
    starts = rng.integers(0, n, size=int(rng.integers(1, 4))).astype(np.int32)
    _check(T, oracle, _upload_table(T, table_np), table_np, accept, starts)


@pytest.mark.parametrize("n,v", [(50, 63), (50, 511), (50, 513), (50, 4097), (16384, 67), (16385, 67)])
def test_edges_of_the_renaming(T, oracle, n, v):
    """Around the tokens that a wavefront and a workgroup rename at a time, and the number of states up to which the
    map of names is kept in LDS; half of the states copies of others, so that names change."""
    rng = np.random.default_rng(n + v)
    half = n // 2
    table_np = rng.integers(0, n, size=(n, v), dtype=np.int32)
    table_np[rng.random((n, v)) < 0.5] = DEAD
    table_np[half:2 * half] = table_np[:half]
    accept = (rng.random(n) < 0.3).astype(np.uint8)
    accept[half:2 * half] = accept[:half]
    new, want, _ = _check(T, oracle, _upload_table(T, table_np), table_np, accept, [0, n - 1])
    assert 0 < new.n_rows <= n - half


@pytest.mark.parametrize("n,v", [(50, 1), (50, 63), (50, 129), (50, 511), (50, 513), (50, 4095), (50, 4097), (50, 16385), (16384, 67), (16385, 67)])
def test_passes_led_by_the_bits(T, oracle, n, v):
    """A table that the library has written (here by stacking): its passes read only the entries behind a set bit.  Around
    the words that a wavefront reads at a time, the tokens of a piece of a row and the states whose names fit in LDS; rows
    from empty to full, with long runs of tokens that no state allows; half of the rows copies of others."""
    rng = np.random.default_rng(7 * n + v)
    half = n // 2
    table_np = rng.integers(0, n, size=(n, v), dtype=np.int32)
    table_np[rng.random((n, v)) < rng.choice([0.0, 0.5, 0.999], size=n)[:, None]] = DEAD
    table_np[:, v // 3:v // 2] = DEAD
    table_np[half:2 * half] = table_np[:half]
    accept = (rng.random(n) < 0.2).astype(np.uint8)
    accept[half:2 * half] = accept[:half]
    table, _ = T.table_concat([_upload_table(T, table_np)])
    new, want, _ = _check(T, oracle, table, table_np, accept, np.array([0, 1, n // 3], dtype=np.int32))
    packed = T.table_pack(new)
    if new.n_rows:
        targets, begin, _, allow = T.table_pack_arrays(packed)
        assert np.array_equal(targets.cpu().numpy(), want[want != DEAD])
        assert np.array_equal(begin.cpu().numpy(), np.concatenate([[0], np.cumsum((want != DEAD).sum(axis=1))]))
        assert np.array_equal(allow.cpu().numpy().view(np.uint32), G.bits_from_table(want, allow.shape[1]))


@pytest.mark.parametrize("v", [63, 4097, 9000])
@pytest.mark.parametrize("how", ["entries added", "bits cleared, then stacked", "bits set, then stacked", "entries removed"])
def test_result_follows_the_entries(T, oracle, how, v):
    """The allowed bits of a table may have parted from its entries: the caller has edited its own buffers, or wrapped
    ones whose bits forbid more (or less) than the entries before stacking them.  The entries decide, in every pass."""
    n = 60
    rng = np.random.default_rng(v)
    table_np = rng.integers(0, n, size=(n, v), dtype=np.int32)
    table_np[rng.random((n, v)) < rng.choice([0.5, 0.999], size=n)[:, None]] = DEAD
    table_np[n // 2:] = table_np[:n // 2]
    accept = (rng.random(n) < 0.2).astype(np.uint8)
    accept[n // 2:] = accept[:n // 2]
    other = table_np.copy()
    other[rng.random((n, v)) < 0.01] = DEAD                   # with fewer edges, and not the same ones in both halves
    bits_of, entries = (other, table_np) if how in ("entries added", "bits cleared, then stacked") else (table_np, other)
    rw = T.allow_row_words(v)
    bits = torch.from_numpy(G.bits_from_table(bits_of, rw).view(np.int32)).cuda()
    if "stacked" in how:
        table, _ = T.table_concat([T.table_wrap(torch.from_numpy(entries).cuda(), bits)])
    else:
        table, _ = T.table_concat([T.table_wrap(torch.from_numpy(bits_of).cuda(), bits)])
        table.delta.copy_(torch.from_numpy(entries))
        torch.cuda.synchronize()
    _check(T, oracle, table, entries, accept, np.array([0, 1], dtype=np.int32))


def _most_targets(table_np):
    return max(len(np.unique(r[r >= 0])) for r in table_np)


def test_long_chains_merge(T, oracle):
    """Two copies of a counter of 300 states: the copies merge state by state, one refinement round
    per state of the chain (the rounds run on the rows' lists of distinct targets)."""
    L, v = 300, 50
    n = 2 * L + 1
    table_np = np.full((n, v), DEAD, dtype=np.int32)
    table_np[0, 0], table_np[0, 1] = 1, L + 1
    for half in (0, L):
        for i in range(1, L + 1):
            q = half + i
            nxt = q + 1 if i < L else q
            table_np[q, i % v] = nxt
            table_np[q, (3 * i + 7) % v] = nxt if i % 5 else q
    accept = np.zeros(n, np.uint8)
    accept[L], accept[2 * L] = 1, 1
    assert _most_targets(table_np) <= 3072
    new, want, mp = _check(T, oracle, _upload_table(T, table_np), table_np, accept, [0])
    assert new.n_rows == L + 1 and np.array_equal(mp[1:L + 1], mp[L + 1:])


@pytest.mark.parametrize("written_by", ["caller", "library"])
def test_rows_with_many_distinct_targets(T, oracle, written_by):
    """A table whose rows have more distinct targets than the list-building pass keeps per row:
    the call streams the dense rows instead, with the same result."""
    rng = np.random.default_rng(77)
    n, v = 5000, 12000
    table_np = rng.integers(0, n, size=(n, v), dtype=np.int32)
    table_np[rng.random((n, v)) < 0.3] = DEAD
    for q in range(n - 40, n):                       # a few classes to merge
        table_np[q] = table_np[q - 40]
    accept = (rng.random(n) < 0.3).astype(np.uint8)
    accept[n - 40:] = accept[n - 80:n - 40]
    assert _most_targets(table_np) > 3072
    table = _upload_table(T, table_np)
    _check(T, oracle, table if written_by == "caller" else _as_torch(T, table), table_np, accept, [0, 17])


@pytest.mark.parametrize("useful", ["all", "traps", "none final", "few reached"])
@pytest.mark.parametrize("n,v", [(700, 64), (700, 65), (8192, 70), (8193, 200), (20001, 40)])
def test_searches(T, oracle, n, v, useful):
    """Levels of states in shuffled order, each leading to the next: rows that fit the wavefronts in flight and rows that
    do not (both sides of the line), lists around a wavefront's width; states that reach no final state, or are not reached."""
    rng = np.random.default_rng(n + v)
    depth = 30
    per = n // depth
    p = rng.permutation(n).astype(np.int32)
    table_np = np.full((n, v), DEAD, dtype=np.int32)
    for lv in range(depth - 1):
        table_np[p[lv * per:(lv + 1) * per]] = p[(lv + 1) * per + rng.integers(0, per, size=(per, v))]
    table_np[rng.random((n, v)) < 0.3] = DEAD
    accept = np.zeros(n, np.uint8)
    accept[p[(depth - 1) * per:depth * per]] = rng.integers(1, 3, size=per) != 1
    if useful == "traps":                                      # half of the states lead only to one another
        trap = np.unique(rng.integers(0, n, size=n // 2)).astype(np.int32)
        table_np[trap] = trap[rng.integers(0, len(trap), size=(len(trap), v))]
        accept[trap] = 0
    elif useful == "none final":
        accept[:] = 0
    starts = p[:per] if useful != "few reached" else p[:1]
    _check(T, oracle, _upload_table(T, table_np), table_np, accept, starts.astype(np.int32))


def test_lists_longer_than_first_guessed(T, oracle):
    """Rows with about 700 distinct targets each: more list entries in all than the first pass makes room for, so
    the lists are built a second time at their true size."""
    rng = np.random.default_rng(31)
    n, v = 2500, 1200
    table_np = rng.integers(0, n, size=(n, v), dtype=np.int32)
    table_np[rng.random((n, v)) < 0.3] = DEAD
    for q in range(n - 30, n):
        table_np[q] = table_np[q - 30]
    accept = (rng.random(n) < 0.3).astype(np.uint8)
    accept[n - 30:] = accept[n - 60:n - 30]
    per_row = [len(np.unique(r[r >= 0])) for r in table_np]
    assert max(per_row) <= 3072 and sum(per_row) > max(1 << 20, n * 512)
    _check(T, oracle, _upload_table(T, table_np), table_np, accept, [0])


def test_nothing_left(T, oracle):
    table_np = np.array([[1, -1], [0, 1]], dtype=np.int32)
    new, want, mp = _check(T, oracle, _upload_table(T, table_np), table_np, np.zeros(2, np.uint8), [0])
    assert new.n_rows == 0 and mp.tolist() == [DEAD, DEAD]


def test_table_without_tokens(T, oracle):
    vocab, d = T.Vocab(np.zeros(0, np.uint8), np.zeros(1, np.int64)), compile_regex(r"ab")
    table = T.compile_token_dfa(vocab, T.CharDFA(d.trans, d.accept, d.start))
    accept = np.ones(d.n_states, np.uint8)
    new, acc, mp = T.table_minimize(table, accept, [1, 0])
    want, want_acc, want_mp = oracle.minimize(np.zeros((d.n_states, 0), np.int32), accept, np.array([1, 0], np.int32))
    assert np.array_equal(mp, want_mp) and np.array_equal(acc, want_acc) and new.n_rows == want.shape[0]
    assert T.table_pack(new).n_rows == new.n_rows


def test_c2_and_decode(T, oracle):
    w = configs.get("c2")
    d = w.dfas[0]
    table_np = oracle.compile_walk(d.trans, w.vocab.data, w.vocab.offsets, n_threads=8)
    table = T.compile_token_dfa(T.Vocab(w.vocab.data, w.vocab.offsets), T.CharDFA(d.trans, d.accept, d.start))
    new, want, mp = _check(T, oracle, table, table_np, d.accept, [d.start])
    assert 0 < new.n_rows <= d.n_states
    # the same greedy decode on both tables: same tokens, states related by the map
    B, steps, Vn = 32, 40, table_np.shape[1]
    st_a = torch.full((B,), d.start, dtype=torch.int32, device="cuda")
    st_b = torch.full((B,), int(mp[d.start]), dtype=torch.int32, device="cuda")
    tok_a = torch.empty(B, dtype=torch.int32, device="cuda")
    tok_b = torch.empty(B, dtype=torch.int32, device="cuda")
    mp_dev = torch.from_numpy(mp).cuda()
    for s in range(steps):
        lg = torch.from_numpy(LG.gen_logits(configs.logits_seed(2), s, B, Vn, 2.0, "bf16").view(np.int16)).cuda().view(torch.bfloat16)
        T.mask_step(table, lg, st_a, tok_a, st_a)
        T.mask_step(new, lg, st_b, tok_b, st_b)
        torch.cuda.synchronize()
        assert torch.equal(tok_a, tok_b)
        assert torch.equal(mp_dev[st_a.long()], st_b)


def test_stacked_with_several_starts(T, oracle):
    w = configs.get("c5")
    pick = (3, 9, 3)
    vocab = V.from_tokens([bytes(w.vocab.token(t)) for t in range(0, w.vocab.n_tokens, 97)])
    tabs = [oracle.compile_walk(w.dfas[i].trans, vocab.data, vocab.offsets) for i in pick]
    ref, offs = oracle.concat_tables(tabs)
    accept = np.concatenate([w.dfas[i].accept for i in pick]).astype(np.uint8)
    starts = [int(offs[c]) + w.dfas[i].start for c, i in enumerate(pick)]
    _check(T, oracle, _upload_table(T, ref), ref, accept, starts)


def _hold(stream):
    """Work on `stream` that lasts some tens of milliseconds: what is enqueued on it next is still waiting while the host
    goes on.  (Products of 8,192 x 8,192, two floating-point operations for each of 2^39 terms.)"""
    with torch.cuda.stream(stream):
        a = torch.ones((8192, 8192), dtype=torch.bfloat16, device="cuda")
        out = torch.empty_like(a)
        for _ in range(40):
            torch.mm(a, a, out=out)
    return a, out                                             # (kept by the caller until the stream is done)


def test_blocks_of_a_destroyed_table_in_use_on_another_stream(T, oracle):
    """A minimised table is destroyed while steps on another stream wait to read it; the next minimisation finds one
    block that fits its rows, that table's.  The steps see the table as it was: the block is handed out only after a wait,
    so they are done when the call returns.  tdfa_trim gives the memory back."""
    rng = np.random.default_rng(5)
    n, v, steps, batch = 400, 40000, 24, 64
    a_np = rng.integers(0, n, size=(n, v), dtype=np.int32)
    b_np = rng.integers(0, n, size=(n, v), dtype=np.int32)
    accept = np.ones(n, dtype=np.uint8)
    accept[::2] = 0
    a, b = _upload_table(T, a_np), _upload_table(T, b_np)
    x = rng.normal(0, 2, size=(batch, v)).astype(np.float32)
    lg = torch.from_numpy(x).cuda()
    states = rng.integers(0, n, size=batch).astype(np.int32)
    want = states.copy()
    for _ in range(steps):
        _, want = oracle.mask_step(a_np, x, 0, want)
    side = torch.cuda.Stream()
    st = torch.from_numpy(states).cuda()
    tok = torch.empty_like(st)
    T.trim()
    for _ in range(3):
        small, _, mp = T.table_minimize(a, accept, [0])
        assert small.n_rows == n and (mp == np.arange(n)).all()       # nothing merges: the same rows under the same names
        q = st.clone()
        torch.cuda.synchronize()
        held = _hold(side)
        with torch.cuda.stream(side):
            for _ in range(steps):
                T.mask_step(small, lg, q, tok, q)
        small.close()
        assert not side.query()                               # (destroying the table has not waited for the steps)
        other, _, _ = T.table_minimize(b, accept, [0])
        assert side.query()
        del held
        packed = T.table_pack(other)
        torch.cuda.synchronize()
        assert np.array_equal(q.cpu().numpy(), want)
        G.check_rows(_as_torch(T, other), b_np, np.arange(n))
        packed.close()
        other.close()
    torch.cuda.synchronize()
    kept = torch.cuda.mem_get_info()[0]
    T.trim()
    assert torch.cuda.mem_get_info()[0] >= kept + n * v * 4


@pytest.mark.parametrize("minimised", [True, False])
def test_counts_of_a_destroyed_table_in_use_on_another_stream(T, oracle, minimised):
    """A table whose states are counted (one the library minimised, and one it wrote into the caller's buffers) is
    destroyed while steps on another stream wait to read it; then tables with as many states, none of which allows a
    token, are written on the current stream.  Their counts are in place before those steps begin, and must not be
    where the steps read: a state counted as allowing nothing would end its sequence."""
    rng = np.random.default_rng(6)
    n, v, batch, steps = 700, 4001, 64, 6
    tab = rng.integers(0, n, size=(n, v), dtype=np.int32)
    accept = np.ones(n, dtype=np.uint8)
    accept[::2] = 0
    dense, none = _upload_table(T, tab), _upload_table(T, np.full((n, v), -1, dtype=np.int32))
    x = rng.normal(0, 2, size=(batch, (v + 3) // 4 * 4)).astype(np.float32)
    lg = torch.from_numpy(x).cuda()
    states = rng.integers(0, n, size=batch).astype(np.int32)
    want = states.copy()
    for _ in range(steps):
        _, want = oracle.mask_step(tab, x, 0, want, row_stride=x.shape[1])
    q, tok = torch.from_numpy(states).cuda(), torch.empty(batch, dtype=torch.int32, device="cuda")
    outs = [(torch.empty_like(none.delta), torch.empty_like(none.allow)) for _ in range(3)]
    T.mask_step(dense, lg, q, tok, torch.empty_like(q))                 # (the scratch of the steps is there)
    T.trim()                                                  # (no block goes back to the runtime, which waits, below)
    table = T.table_minimize(dense, accept, [0])[0] if minimised else T.table_concat([dense])[0]
    assert table.n_rows == n
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    held = _hold(side)
    with torch.cuda.stream(side):
        for _ in range(steps):
            T.mask_step(table, lg, q, tok, q)
    buffers = table._keep                                     # (the caller's buffers live on; the counts are the library's)
    table.close()
    made = [T.table_concat([none], out=o)[0] for o in outs]
    torch.cuda.current_stream().synchronize()
    assert not side.query()                                   # the steps have not begun or are under way
    torch.cuda.synchronize()
    assert np.array_equal(q.cpu().numpy(), want)
    del held, buffers, made


def test_compile_under_capture_after_a_destroyed_table(T, oracle):
    """A compile call that is being captured finds only counts that a step may still read: it takes other memory."""
    w = configs.get("c1")
    want = oracle.compile_walk(w.dfas[0].trans, w.vocab.data, w.vocab.offsets)
    vocab = T.Vocab(w.vocab.data, w.vocab.offsets)
    dfa = T.CharDFA(w.dfas[0].trans, w.dfas[0].accept, w.dfas[0].start)
    rows = dfa.n_states
    out = (torch.empty((rows, vocab.n_tokens), dtype=torch.int32, device="cuda"),
           torch.empty((rows, T.allow_row_words(vocab.n_tokens)), dtype=torch.int32, device="cuda"))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    T.trim()
    with torch.cuda.stream(side):
        T.compile_token_dfa(vocab, dfa, out=out).close()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        table = T.compile_token_dfa(vocab, dfa, out=out)
    for _ in range(3):
        out[0].fill_(7)
        out[1].fill_(0)
        graph.replay()
        torch.cuda.synchronize()
        G.check_rows(table, want, np.arange(rows))
        lg = torch.zeros((rows, (vocab.n_tokens + 3) // 4 * 4), device="cuda")
        st = torch.arange(rows, dtype=torch.int32, device="cuda")
        tok, new = torch.empty_like(st), torch.empty_like(st)
        T.mask_step(table, lg, st, tok, new)
        torch.cuda.synchronize()
        live = want >= 0
        first = np.where(live.any(axis=1), live.argmax(axis=1), -1)
        assert np.array_equal(tok.cpu().numpy(), first)       # (equal logits: the lowest allowed token)


def test_kept_memory_is_bounded(T):
    """What destroyed tables leave with the library: at most 4 GiB however many there were, no block of more than five
    quarters of what a table needs, and nothing that pushes an automaton's blocks out.  (2 MiB per block: the runtime's own
    granularity.)"""
    mib = 1 << 20
    n, v = 400, 40000
    tab = _upload_table(T, np.random.default_rng(9).integers(0, n, size=(n, v), dtype=np.int32))
    accept = np.ones(n, dtype=np.uint8)
    accept[::2] = 0

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    T.table_minimize(tab, accept, [0])[0].close()             # (what the first call sets up is there)
    T.trim()
    start = free()
    tables = [T.table_minimize(tab, accept, [0])[0] for _ in range(100)]
    assert start - free() > 100 * n * v * 4                   # 6.4 GB
    for t in tables:
        t.close()
    assert start - free() <= (4 << 30) + 256 * 2 * mib
    T.trim()
    assert start - free() <= 8 * mib
    # a table of five eighths the size does not take the larger table's block
    rows = np.arange(n) % (n * 5 // 8)
    merged = _upload_table(T, tab.delta.cpu().numpy()[rows])
    start = free()
    T.table_minimize(tab, accept, [0])[0].close()
    small, _, _ = T.table_minimize(merged, accept[rows], [0])
    assert small.n_rows == n * 5 // 8
    T.trim()
    assert start - free() <= n * 5 // 8 * v * 4 * 5 // 4 + 4 * mib


def test_set_up_calls_beside_a_capture(T, oracle):
    """Minimising and packing on one stream while another is captured (by a program that allows that: relaxed mode),
    with nothing in the cache and with blocks there that need a wait for the device: both times the same tables."""
    rng = np.random.default_rng(8)
    n, v = 300, 5000
    tab = rng.integers(0, n, size=(n, v), dtype=np.int32)
    accept = np.ones(n, dtype=np.uint8)
    accept[::2] = 0
    table = _upload_table(T, tab)
    work = torch.cuda.Stream()
    x = torch.zeros(1000, device="cuda")
    outs = [(torch.empty_like(table.delta), torch.empty_like(table.allow)) for _ in range(2)]
    torch.cuda.synchronize()
    T.trim()
    for out in outs:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode="relaxed"):
            x.add_(1.0)
            small, _, mp = T.table_minimize(table, accept, [0], stream=work)
            packed = T.table_pack(small, stream=work)
            x.add_(1.0)
        before = float(x[0])
        graph.replay()
        torch.cuda.synchronize()
        assert float(x[0]) == before + 2.0 and (mp == np.arange(n)).all()
        G.check_rows(T.table_concat([small], out=out)[0], tab, np.arange(n))
        assert packed.n_rows == n
        packed.close()
        small.close()


def test_bad_arguments(T):
    table = _upload_table(T, np.zeros((2, 3), dtype=np.int32))
    with pytest.raises(T.TdfaError):
        T.table_minimize(table, np.zeros(2, np.uint8), [5])
    with pytest.raises(ValueError):
        T.table_minimize(table, np.zeros(3, np.uint8), [0])
