"""GPU parity of the sampling step against the oracle: the noise bit for bit, then tokens, states
and masked rows of single steps and of chained decodes."""
import numpy as np
import pytest
import torch

from workloads import configs, logits as LG
import gpu_util as G

pytestmark = pytest.mark.gpu
DEAD = -1
F32, BF16 = 0, 1


@pytest.fixture(scope="module")
def T():
    import paper_2407_08103_amd as T
    assert torch.cuda.is_available()
    return T


def _upload_table(T, table_np):
    delta = torch.from_numpy(table_np).cuda()
    rw = T.allow_row_words(table_np.shape[1])
    allow = torch.from_numpy(G.bits_from_table(table_np, rw).view(np.int32)).cuda()
    return T.table_wrap(delta, allow)


def _to_dev(lg_np, dtype):
    if dtype == F32:
        return torch.from_numpy(lg_np).cuda()
    return torch.from_numpy(lg_np.view(np.int16)).cuda().view(torch.bfloat16)


def _bits(t: torch.Tensor) -> np.ndarray:
    if t.dtype == torch.float32:
        return t.cpu().numpy().view(np.uint32)
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def _rand_table(n_rows, n_tokens, p_live, seed):
    rng = np.random.default_rng(seed)
    t = rng.integers(0, n_rows, size=(n_rows, n_tokens), dtype=np.int32)
    t[rng.random((n_rows, n_tokens)) > p_live] = DEAD
    return t


def _step_and_check(T, oracle, table, table_np, lg_np, dtype, states_np, temperature, seed, offset, masked=True):
    B = len(states_np)
    lg = _to_dev(lg_np, dtype)
    st = torch.from_numpy(states_np).cuda()
    tok = torch.full((B,), -9, dtype=torch.int32, device="cuda")
    new = torch.full((B,), -9, dtype=torch.int32, device="cuda")
    out = torch.empty_like(lg) if masked else None
    T.sample_step(table, lg, st, temperature, seed, offset, tok, new, out)
    torch.cuda.synchronize()
    res = oracle.sample_step(table_np, lg_np, dtype, states_np, temperature, seed, offset, want_masked=masked,
                             n_threads=16)
    assert np.array_equal(tok.cpu().numpy(), res[0]), (tok.cpu().numpy()[:8], res[0][:8])
    assert np.array_equal(new.cpu().numpy(), res[1])
    if masked:
        V = table_np.shape[1]
        assert np.array_equal(_bits(out)[:, :V], res[2].view(_bits(out).dtype)[:, :V])
    return res


@pytest.mark.parametrize("batch,n_tokens,seed,offset", [(3, 1001, 1, 0), (2, 128256, 2 ** 63 + 5, 2 ** 40 + 9),
                                                         (70, 4099, 0, 2 ** 32 - 1)])
def test_noise_bit_for_bit(T, oracle, batch, n_tokens, seed, offset):
    """Every noise value, compared as bit patterns: the generator words, the uniform grid and both
    logarithms of each of them."""
    got = torch.empty((batch, n_tokens), dtype=torch.float32, device="cuda")
    T.sample_noise(got, seed, offset)
    torch.cuda.synchronize()
    want = oracle.sample_noise(batch, n_tokens, seed, offset)
    assert np.array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("p_live", [0.02, 0.9])
@pytest.mark.parametrize("n_tokens,batch", [(8, 1), (37 * 8 + 3, 3), (1000 * 8 + 8, 5), (40000, 2), (50021, 300), (131075, 112), (131075, 113)])
def test_random_tables(T, oracle, dtype, p_live, n_tokens, batch):
    """Sparse and dense allowed sets; sizes cover one group, ragged rows, many parts per row and one
    workgroup per row; states include sinks, DEAD and ids that are no row."""
    tab = _rand_table(11, n_tokens, p_live, n_tokens + batch)
    tab[3] = DEAD
    tab[4] = DEAD
    tab[4, n_tokens - 1] = 6
    table = _upload_table(T, tab)
    rng = np.random.default_rng(batch)
    stride = (n_tokens + 7) // 8 * 8
    for trial, temperature in enumerate((1.0, 0.35, 3.0)):
        states = rng.integers(-1, 12, size=batch).astype(np.int32)
        states[: min(batch, 2)] = [3, 4][: min(batch, 2)]
        x = np.zeros((batch, stride), dtype=np.float32)
        x[:, :n_tokens] = rng.normal(0, 2, size=(batch, n_tokens))
        lg = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        got = _sample_strided(T, oracle, table, tab, lg, dtype, states, temperature, 1234 + trial, 77 * trial,
                              masked=trial != 1)
    assert (got[0] >= 0).any() or batch <= 2


def _sample_strided(T, oracle, table, table_np, lg_np, dtype, states_np, temperature, seed, offset, masked, top_k=0):
    """Rows padded to a multiple of 8 elements (the alignment rule); the padding is not touched."""
    B, stride = lg_np.shape
    V = table_np.shape[1]
    lg = _to_dev(lg_np, dtype)
    st = torch.from_numpy(states_np).cuda()
    tok = torch.full((B,), -9, dtype=torch.int32, device="cuda")
    new = torch.full((B,), -9, dtype=torch.int32, device="cuda")
    out = torch.full_like(lg, 7.0) if masked else None
    T.sample_step(table, lg, st, temperature, seed, offset, tok, new, out, top_k=top_k)
    torch.cuda.synchronize()
    res = oracle.sample_step(table_np, lg_np, dtype, states_np, temperature, seed, offset, row_stride=stride,
                             want_masked=masked, n_threads=16, top_k=top_k)
    assert np.array_equal(tok.cpu().numpy(), res[0]), (tok.cpu().numpy()[:8], res[0][:8])
    assert np.array_equal(new.cpu().numpy(), res[1])
    if masked:
        assert np.array_equal(_bits(out)[:, :V], res[2].view(_bits(out).dtype)[:, :V])
        assert (out[:, V:].float() == 7.0).all()
    return res


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("p_live", [0.02, 0.9])
@pytest.mark.parametrize("n_tokens,batch", [(8, 1), (37 * 8 + 3, 3), (40000, 2), (50021, 200)])
def test_top_k(T, oracle, dtype, p_live, n_tokens, batch):
    """The cut at the k-th largest allowed logit: k from 1 to more than the vocabulary, logits with
    many ties (rounded), NaN and infinities, one and many workgroups per row."""
    tab = _rand_table(11, n_tokens, p_live, 7 * n_tokens + batch)
    tab[3] = DEAD
    tab[4] = DEAD
    tab[4, n_tokens - 1] = 6
    table = _upload_table(T, tab)
    rng = np.random.default_rng(batch + 1)
    stride = (n_tokens + 7) // 8 * 8
    for trial, k in enumerate((1, 2, 7, 50, 4000, 10 ** 6)):
        states = rng.integers(-1, 12, size=batch).astype(np.int32)
        states[: min(batch, 2)] = [3, 4][: min(batch, 2)]
        x = np.zeros((batch, stride), dtype=np.float32)
        x[:, :n_tokens] = rng.normal(0, 2, size=(batch, n_tokens))
        if trial % 3 == 1:
            x = np.round(x * 2) / 2                                  # heavy ties, also across the cut
        if trial % 3 == 2:
            x[:, rng.integers(0, n_tokens, max(1, n_tokens // 50))] = np.nan
            x[:, rng.integers(0, n_tokens, max(1, n_tokens // 200))] = -np.inf
            x[:, rng.integers(0, n_tokens, 2)] = np.inf
            x[:, rng.integers(0, n_tokens, max(1, n_tokens // 100))] = -0.0
        lg = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        _sample_strided(T, oracle, table, tab, lg, dtype, states, (1.0, 0.4, 2.5)[trial % 3], 99 + trial, trial,
                        masked=trial == 0, top_k=k)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("n_tokens", [2051, 32768, 32771, 131072, 131077])
def test_top_k_edges(T, oracle, dtype, n_tokens):
    """Around the sizes where the cut changes its way: rows that do and do not fit the threads' registers, states on
    both sides of the 2,048 tokens that are collected whole, k beyond the number of threads, ties across the cut,
    zeros of both signs at the cut, NaN at the top; the masked row in place every other time.  Exact integers."""
    rng = np.random.default_rng(n_tokens + dtype)
    counts = [0, 1, 60, 2047, 2048, 2049, n_tokens // 2, n_tokens]
    tab = np.full((len(counts) + 1, n_tokens), DEAD, dtype=np.int32)
    for q, c in enumerate(counts):
        tab[q, rng.choice(n_tokens, size=c, replace=False)] = q
    tab[-1, n_tokens - 11:] = 3                               # the last groups only, the partial one among them
    table, _ = T.table_concat([_upload_table(T, tab)])
    states = np.arange(-1, len(tab) + 1).astype(np.int32)
    batch, stride = len(states), (n_tokens + 7) // 8 * 8
    for trial, k in enumerate((1, 50, 129, 700, 1025, 3000)):
        x = np.zeros((batch, stride), dtype=np.float32)
        x[:, :n_tokens] = rng.normal(0, 2, size=(batch, n_tokens))
        if trial % 3 == 1:
            x = np.minimum(np.round(x), 2.0)                  # thousands of equal logits at the top
        if trial == 2:
            x = -np.abs(x)
            x[:, rng.integers(0, n_tokens, 40)] = 0.0
            x[:, rng.integers(0, n_tokens, 400)] = -0.0
        if trial == 5:
            x[::2, rng.integers(0, n_tokens, 30)] = np.nan
            x[1::2] = -np.inf
        lg = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        if dtype == BF16 and trial == 5:
            lg[np.isnan(x)] = 0x7FC1
            lg[0, :9] = 0xFFFF
        dev = _to_dev(lg, dtype)
        st = torch.from_numpy(states).cuda()
        tok = torch.full((batch,), -9, dtype=torch.int32, device="cuda")
        new = torch.full((batch,), -9, dtype=torch.int32, device="cuda")
        out = dev if trial % 2 else None
        T.sample_step(table, dev, st, 0.8, 21, trial, tok, new, out, top_k=k)
        torch.cuda.synchronize()
        want = oracle.sample_step(tab, lg, dtype, states, 0.8, 21, trial, row_stride=stride, want_masked=True, top_k=k, n_threads=16)
        assert np.array_equal(tok.cpu().numpy(), want[0]), (trial, k, tok.cpu().numpy(), want[0])
        assert np.array_equal(new.cpu().numpy(), want[1])
        if out is not None:
            assert np.array_equal(_bits(out)[:, :n_tokens], want[2].view(_bits(out).dtype)[:, :n_tokens])


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_top_k_of_rows_with_more_allowed_tokens_than_counted(T, oracle, dtype):
    """The caller allows further tokens in rows of its own buffers, which the library has counted before: the cut is
    made where the row as it is allows k tokens or more, whatever the count says."""
    rng = np.random.default_rng(4)
    v, k = 5000, 50
    tab = np.full((4, v), DEAD, dtype=np.int32)
    for q, c in enumerate((3, 49, 50, 2000)):
        tab[q, rng.choice(v, size=c, replace=False)] = q
    table, _ = T.table_concat([_upload_table(T, tab)])
    more = tab.copy()
    for q in range(4):
        more[q, rng.choice(v, size=1500, replace=False)] = q
    both = _upload_table(T, more)
    table.delta.copy_(both.delta)
    table.allow.copy_(both.allow)
    states = np.arange(64, dtype=np.int32) % 4
    lg = rng.normal(0, 2, size=(64, v)).astype(np.float32)
    lg = lg if dtype == F32 else LG.f32_to_bf16_bits(lg)
    st, dev = torch.from_numpy(states).cuda(), _to_dev(lg, dtype)
    tok, new = torch.empty_like(st), torch.empty_like(st)
    T.sample_step(table, dev, st, 3.0, 2, 1, tok, new, top_k=k)         # (hot: without the cut other tokens are drawn)
    torch.cuda.synchronize()
    want = oracle.sample_step(more, lg, dtype, states, 3.0, 2, 1, top_k=k)
    free = oracle.sample_step(more, lg, dtype, states, 3.0, 2, 1)
    assert (want[0] != free[0]).sum() > 16
    assert np.array_equal(tok.cpu().numpy(), want[0]) and np.array_equal(new.cpu().numpy(), want[1])


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("n_tokens", [40000, 131077])
def test_top_k_among_thousands_of_zeros(T, oracle, dtype, n_tokens):
    """More logits at the cut than are collected, zeros of both signs among small and negative numbers: the selection over
    the row starts from the bound that the threads' maxima give, and -0 counts as +0 there as well."""
    rng = np.random.default_rng(n_tokens)
    tab = _rand_table(3, n_tokens, 0.8, 7)
    table = _upload_table(T, tab)
    states = (np.arange(6) % 3).astype(np.int32)
    x = -np.abs(rng.normal(0, 2, size=(6, (n_tokens + 7) // 8 * 8))).astype(np.float32)
    kind = rng.random(x.shape)
    x[kind < 0.2] = 0.0
    x[(kind >= 0.2) & (kind < 0.4)] = -0.0
    x[(kind >= 0.4) & (kind < 0.41)] = np.float32(-1e-39)
    x[4:, ::3] = np.float32(1e-39)
    lg = x if dtype == F32 else LG.f32_to_bf16_bits(x)
    for k in (1, 60, 1000, 20000):
        _sample_strided(T, oracle, table, tab, lg, dtype, states, 0.9, 5, k, masked=k == 60, top_k=k)


def test_steps_on_two_streams_at_once(T):
    """Draws and greedy steps whose rows several workgroups share, on two streams that are held back until both have all
    of theirs waiting: the same tokens as one after the other, and again afterwards."""
    rng = np.random.default_rng(12)
    v, steps = 40000, 40
    table = _upload_table(T, _rand_table(5, v, 0.7, 3))
    big, small = 256, 24
    st = torch.from_numpy((np.arange(big) % 5).astype(np.int32)).cuda()
    lg = [torch.from_numpy(rng.normal(0, 2, size=(big, v)).astype(np.float32)).cuda().bfloat16() for _ in range(2)]

    def run(which, tok, new):
        for i in range(steps):
            T.sample_step(table, lg[which], st, 1.0, 5, i + 100 * which, tok[i], new[i])
            T.mask_step(table, lg[which][i:i + small], st[:small], tok[steps + i], new[steps + i])

    def empty():
        return torch.full((2, 2 * steps, big), -9, dtype=torch.int32, device="cuda")

    want, want_new = empty(), empty()
    for which in range(2):
        run(which, want[which], want_new[which])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    a = torch.ones((8192, 8192), dtype=torch.bfloat16, device="cuda")
    held = [torch.empty_like(a) for _ in streams]
    for _ in range(2):
        tok, new = empty(), empty()
        torch.cuda.synchronize()
        for s, out in zip(streams, held):
            with torch.cuda.stream(s):
                for _ in range(8):
                    torch.mm(a, a, out=out)
        for which, s in enumerate(streams):
            with torch.cuda.stream(s):
                run(which, tok[which], new[which])
        torch.cuda.synchronize()
        assert torch.equal(tok, want) and torch.equal(new, want_new)
    tok, new = empty(), empty()
    run(0, tok[0], new[0])
    torch.cuda.synchronize()
    assert torch.equal(tok[0], want[0])


def test_draws_in_a_graph(T):
    """Draws of rows in several parts, recorded one after the other on states advanced in place: every replay is what the
    same calls gave before, with other steps on the same stream between the replays."""
    rng = np.random.default_rng(8)
    v, batch = 64008, 256
    tab = np.full((6, v), DEAD, dtype=np.int32)
    for q, n in enumerate((0, 30, v // 200, v // 9, v // 2, v)):
        tab[q, rng.permutation(v)[:n]] = rng.integers(0, 6, size=n)
    table = T.table_pack(_upload_table(T, tab))
    lg = torch.from_numpy(rng.normal(0, 2, size=(batch, v)).astype(np.float32)).cuda().bfloat16()
    first = torch.from_numpy(rng.integers(-1, 6, size=batch).astype(np.int32)).cuda()
    states, tok = first.clone(), torch.empty((3, batch), dtype=torch.int32, device="cuda")

    def steps():
        states.copy_(first)
        for i in range(3):
            T.sample_step(table, lg, states, 1.0, 5, i, tok[i], states)

    steps()
    torch.cuda.synchronize()
    want = tok.clone(), states.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        steps()
    other, new = torch.empty_like(states), torch.empty_like(states)
    for i in range(4):
        tok.fill_(-9)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(tok, want[0]) and torch.equal(states, want[1])
        T.mask_step(table, lg[:16 + i], first[:16 + i], other[:16 + i], new[:16 + i])
        T.sample_step(table, lg[:40], first[:40], 1.0, 5, 0, other[:40], new[:40])
        torch.cuda.synchronize()
        assert torch.equal(other[:40], want[0][0, :40])


def test_states_changed_under_a_draw(T):
    """A caller changes the states on another stream while draws of rows in several parts run: what those draws say is
    open, but the steps that come after them are right."""
    rng = np.random.default_rng(31)
    v, batch, steps = 64008, 256, 60
    tab = np.full((4, v), DEAD, dtype=np.int32)
    for q, n in enumerate((1, v // 3, 40, v)):
        tab[q, rng.permutation(v)[:n]] = q
    table = T.table_pack(_upload_table(T, tab))
    lg = torch.from_numpy(rng.normal(0, 2, size=(batch, v)).astype(np.float32)).cuda().bfloat16()
    sets = [torch.from_numpy(((np.arange(batch) + k) % 4).astype(np.int32)).cuda() for k in range(3)]
    states = sets[0].clone()

    def draws():
        out = torch.full((3, 2, batch), -9, dtype=torch.int32, device="cuda")
        for k in range(3):
            states.copy_(sets[k])
            T.sample_step(table, lg, states, 1.0, 5, k, out[k, 0], out[k, 1])
        torch.cuda.synchronize()
        return out

    want = draws()
    assert (want >= 0).all()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    a = torch.ones((8192, 8192), dtype=torch.bfloat16, device="cuda")
    held = [torch.empty_like(a) for _ in streams]
    junk = torch.empty((2, batch), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for s, out in zip(streams, held):
        with torch.cuda.stream(s):
            for _ in range(8):
                torch.mm(a, a, out=out)
    for i in range(steps):
        with torch.cuda.stream(streams[0]):
            T.sample_step(table, lg, states, 1.0, 5, i, junk[0], junk[1])
        with torch.cuda.stream(streams[1]):
            for k in range(8):
                states.copy_(sets[(i + k) % 3])
    torch.cuda.synchronize()
    for s in (*streams, torch.cuda.current_stream()):
        with torch.cuda.stream(s):
            assert torch.equal(draws(), want)


def test_draw_beyond_2_30_tokens(T):
    """A row of more than 2^30 tokens, few of them allowed: the numbers of the tokens' generator blocks outgrow 28 bits.  At a
    temperature of 1 a score is the logit plus the noise, rounded once, and the noise is what sample_noise gives."""
    v = 2 ** 30 + 2 ** 21 + 5
    n, rw = 300, T.allow_row_words(v)
    rng = np.random.default_rng(3)
    tokens = np.unique(np.concatenate([rng.integers(0, 2 ** 30, n // 4), rng.integers(2 ** 30, v, n), [2 ** 30, v - 1]]))
    bits = torch.zeros((1, rw), dtype=torch.int32, device="cuda")
    words, values = tokens >> 5, (np.uint32(1) << (tokens & 31).astype(np.uint32))
    first = np.flatnonzero(np.r_[True, words[1:] != words[:-1]])
    bits[0, torch.from_numpy(words[first]).cuda()] = torch.from_numpy(np.bitwise_or.reduceat(values, first).view(np.int32)).cuda()
    delta = torch.zeros((1, v), dtype=torch.int32, device="cuda")
    table = T.table_wrap(delta, bits)
    lg = torch.zeros((1, (v + 7) // 8 * 8), dtype=torch.bfloat16, device="cuda")
    at = torch.from_numpy(tokens).cuda()
    lg[0, at] = torch.from_numpy(rng.normal(0, 2, len(tokens)).astype(np.float32)).cuda().bfloat16()
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    tok, new = torch.empty_like(st), torch.empty_like(st)
    noise = torch.empty((1, v), dtype=torch.float32, device="cuda")
    for offset in range(6):
        T.sample_noise(noise, 11, offset)
        T.sample_step(table, lg, st, 1.0, 11, offset, tok, new)
        torch.cuda.synchronize()
        score = (lg[0, at].float() + noise[0, at]).cpu().numpy()
        assert int(tok[0]) == tokens[int(score.argmax())] and int(new[0]) == 0


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("n_tokens,batch", [(9001, 4), (16389, 512), (40003, 257), (128261, 64), (16384, 1024), (8200, 1025)])
def test_rows_shared_out_by_cost(T, oracle, dtype, n_tokens, batch):
    """States of every cost, as counted by a packed table: none, one token, few, either side of the line from which every quad
    is drawn, all tokens; states apart and written in place, against the oracle."""
    rng = np.random.default_rng(n_tokens)
    V = n_tokens
    counts = [0, 1, 2, V // 256 - 1, V // 256 + 1, V // 250, V // 249 + 1, V // 40, V // 10 - 1, V // 10 + 1, V // 2, V]
    tab = np.full((len(counts), V), DEAD, dtype=np.int32)
    for q, n in enumerate(counts):
        where = rng.permutation(V)[:n] if q % 3 else np.arange(V - n, V)           # (clustered at the row's end as well)
        tab[q, where] = rng.integers(0, len(counts), size=n)
    table = T.table_pack(_upload_table(T, tab))
    states = rng.integers(-1, len(counts) + 1, size=batch).astype(np.int32)
    stride = (V + 7) // 8 * 8
    x = np.zeros((batch, stride), dtype=np.float32)
    x[:, :V] = rng.normal(0, 2, size=(batch, V))
    x[::5, rng.integers(0, V, size=7)] = np.array([np.nan, np.inf, -np.inf, 1e30, -1e30, 0.0, -0.0], dtype=np.float32)
    lg = x if dtype == F32 else LG.f32_to_bf16_bits(x)
    got = _sample_strided(T, oracle, table, tab, lg, dtype, states, 0.8, 99, 7, masked=False)
    st = torch.from_numpy(states).cuda()
    tok = torch.full((batch,), -9, dtype=torch.int32, device="cuda")
    T.sample_step(table, _to_dev(lg, dtype), st, 0.8, 99, 7, tok, st)
    torch.cuda.synchronize()
    assert np.array_equal(tok.cpu().numpy(), got[0]) and np.array_equal(st.cpu().numpy(), got[1])


@pytest.mark.parametrize("n_tokens,batch", [(61, 5), (2003, 1), (2003, 1100), (9001, 40), (33003, 1030), (140003, 3), (128261, 256)])
def test_listed_tokens_and_quads(T, oracle, n_tokens, batch):
    """States around the numbers that decide how a row is drawn: as many allowed tokens, or quads, to a wavefront as it has lanes,
    lists that are full, half of the quads; whole lists and those cut to the part, or to half of it, also where a wavefront
    has all of its quads to list and the others none; with and without counts."""
    rng = np.random.default_rng(n_tokens)
    V, quads = n_tokens, (n_tokens + 3) // 4
    rows = []
    for n in (1, 63, 64, 65, 255, 256, 257, 300):                                  # tokens in a stretch, and anywhere
        rows += [np.arange(min(n, V)) + (V - min(n, V)) // 3, rng.permutation(V)[:n]]
    for n in (64, 65, 256, 257, quads // 2 - 1, quads // 2, quads // 2 + 2, quads):       # quads, a token or all of each
        at = rng.permutation(quads)[:n]
        rows += [4 * at + rng.integers(0, 4, size=len(at)), (4 * at[:, None] + np.arange(4)).reshape(-1)]
    for first in (0, quads // 3):                                                # a token of each quad in a stretch
        at = first + np.arange(quads // 13)
        rows.append(4 * at + rng.integers(0, 4, size=len(at)))
    tab = np.full((len(rows), V), DEAD, dtype=np.int32)
    for q, at in enumerate(rows):
        at = at[at < V]
        tab[q, at] = rng.integers(0, len(rows), size=len(at))
    dense = _upload_table(T, tab)
    states = (np.arange(batch) % len(rows)).astype(np.int32)
    x = rng.normal(0, 2, size=(batch, (V + 7) // 8 * 8)).astype(np.float32)
    lg = LG.f32_to_bf16_bits(x)
    for i, table in enumerate((T.table_pack(dense), dense)):                      # (the second holds caller's arrays: no counts)
        for first in range(0, len(rows), batch):
            _sample_strided(T, oracle, table, tab, lg, BF16, (states + first) % len(rows), 0.9, 17, first, masked=False)


@pytest.mark.parametrize("n_tokens,batch", [(128261, 256), (128261, 512), (128261, 513), (262145, 227), (262145, 228), (32768, 1025), (32769, 1025)])
def test_lines_of_the_rule_that_cuts_rows(T, oracle, n_tokens, batch):
    """Batches and rows on either side of the sizes from which parts are so long that their bits are not read by single words."""
    test_rows_shared_out_by_cost(T, oracle, BF16, n_tokens, batch)


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_special_values(T, oracle, dtype):
    n_tokens = 4096 + 64
    tab = _rand_table(5, n_tokens, 0.3, 1)
    table = _upload_table(T, tab)
    rng = np.random.default_rng(9)
    states = np.array([0, 1, 2, 3, 4, 0, 1], dtype=np.int32)
    B = len(states)
    cases = [np.full((B, n_tokens), 1.25, np.float32)]                                 # the noise alone decides
    x = rng.normal(0, 2, size=(B, n_tokens)).astype(np.float32)
    x[:, rng.integers(0, n_tokens, 200)] = np.nan
    x[:, rng.integers(0, n_tokens, 50)] = -np.inf
    cases.append(x.copy())
    x[:, rng.integers(0, n_tokens, 50)] = np.inf                                       # several +inf: lowest allowed id
    cases.append(x)
    y = np.full((B, n_tokens), -np.inf, np.float32)                                    # no mass anywhere
    y[:, rng.integers(0, n_tokens, 500)] = np.nan
    cases.append(y)
    cases.append(np.full((B, n_tokens), 3.0e38, np.float32))                           # l / T overflows at T < 1
    cases.append(rng.normal(0, 1e-30, size=(B, n_tokens)).astype(np.float32))          # tiny logits
    for i, x in enumerate(cases):
        lg = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        if dtype == BF16 and np.isnan(x).any():
            lg = lg.copy()
            nan_pos = np.argwhere(np.isnan(x))
            lg[nan_pos[::2, 0], nan_pos[::2, 1]] = 0xFFFF
            lg[nan_pos[1::2, 0], nan_pos[1::2, 1]] = 0x7F81
        for temperature in (1.0, 0.01, 100.0):
            _step_and_check(T, oracle, table, tab, lg, dtype, states, temperature, 5 + i, i)
    with pytest.raises(T.TdfaError):
        T.sample_step(table, _to_dev(cases[0], F32), torch.from_numpy(states).cuda(), 0.0, 1, 0,
                      torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty(B, dtype=torch.int32, device="cuda"))


def _decode(T, oracle, table, table_np, w, start_states, steps, check_steps, seed, temperature, noise_seed):
    """Chained sampled steps on the device, offset = step number; the listed steps are checked
    against the oracle fed with the device's own input states."""
    m = w.mask
    B, V = m.batch, w.vocab.n_tokens
    tdt = torch.float32 if m.dtype == "f32" else torch.bfloat16
    dt = F32 if m.dtype == "f32" else BF16
    hist_states = torch.empty((steps + 1, B), dtype=torch.int32, device="cuda")
    hist_tok = torch.empty((steps, B), dtype=torch.int32, device="cuda")
    hist_states[0] = torch.from_numpy(start_states.astype(np.int32)).cuda()
    logits = torch.empty((B, V), dtype=tdt, device="cuda")
    kept = {}
    stream = torch.cuda.current_stream().cuda_stream
    for s in range(steps):
        LG.gen_logits_device(logits.data_ptr(), seed, s, B, V, V, m.sigma, m.dtype, stream)
        if s in check_steps:
            kept[s] = logits.clone()
        T.sample_step(table, logits, hist_states[s], temperature, noise_seed, s, hist_tok[s], hist_states[s + 1])
    torch.cuda.synchronize()
    hs, ht = hist_states.cpu().numpy(), hist_tok.cpu().numpy()
    for s in sorted(check_steps):
        lg_np = _bits(kept[s]) if dt == BF16 else kept[s].cpu().numpy()
        tok, new = oracle.sample_step(table_np, lg_np, dt, hs[s], temperature, noise_seed, s, n_threads=16)
        assert np.array_equal(ht[s], tok), f"step {s}: tokens differ"
        assert np.array_equal(hs[s + 1], new), f"step {s}: states differ"
    return hs, ht


def test_c2_sampled_decode(T, oracle):
    """JSON-like constraint: 64 sequences, 128 sampled steps, every step checked; what was generated
    stays inside the language (the states never go DEAD) and differs between sequences."""
    w = configs.get("c2")
    d = w.dfas[0]
    v = T.Vocab(w.vocab.data, w.vocab.offsets)
    table = T.compile_token_dfa(v, T.CharDFA(d.trans, d.accept, d.start))
    tab = oracle.compile_walk(d.trans, w.vocab.data, w.vocab.offsets, n_threads=8)
    hs, ht = _decode(T, oracle, table, tab, w, np.full(64, d.start), 128, set(range(128)), configs.logits_seed(2), 1.0, 42)
    assert (hs >= 0).all()
    stopped = ht[-1] < 0
    assert d.accept[hs[-1][stopped]].all()
    assert len({tuple(r) for r in ht.T.tolist()}) > 32


def test_c3_sampled_full_size(T, oracle):
    """The API-call union at its full shape (128,256 tokens, batch 256, one workgroup per row), 40
    steps of a sampled decode, every step checked."""
    w = configs.get("c3")
    d = w.dfas[0]
    v = T.Vocab(w.vocab.data, w.vocab.offsets)
    table = T.compile_token_dfa(v, T.CharDFA(d.trans, d.accept, d.start))
    tab = oracle.compile_walk(d.trans, w.vocab.data, w.vocab.offsets, n_threads=16)
    hs, ht = _decode(T, oracle, table, tab, w, np.full(256, d.start), 40, set(range(40)), configs.logits_seed(3),
                     0.8, 7)
    assert len(np.unique(hs)) > 50


def test_offset_from_device_memory_in_a_graph(T, oracle):
    """tdfa_sample_step_at: a recorded decode loop whose offset lives in device memory and is
    advanced by the loop itself; every replay, with eager work between the replays, gives what
    the eager loop with explicit offsets gives (and step 0 what the oracle gives)."""
    n_tokens, B, S = 5003, 16, 6
    tab = _rand_table(9, n_tokens, 0.3, 21)
    table = _upload_table(T, tab)
    rng = np.random.default_rng(2)
    stride = (n_tokens + 7) // 8 * 8
    xs = [np.zeros((B, stride), dtype=np.float32) for _ in range(S)]
    for x in xs:
        x[:, :n_tokens] = rng.normal(0, 2, size=(B, n_tokens))
    lgs = [_to_dev(LG.f32_to_bf16_bits(x), BF16) for x in xs]
    start_np = rng.integers(0, 9, size=B).astype(np.int32)
    start = torch.from_numpy(start_np).cuda()
    seed, first = 77, 1000

    def loop(states, tokens, offset):
        states[0].copy_(start)
        for s in range(S):
            off = offset if isinstance(offset, torch.Tensor) else offset + s
            T.sample_step(table, lgs[s], states[s], 0.9, seed, off, tokens[s], states[s + 1], top_k=40)
            if isinstance(offset, torch.Tensor):
                offset.add_(1)

    ref_states = torch.empty((S + 1, B), dtype=torch.int32, device="cuda")
    ref_tokens = torch.empty((S, B), dtype=torch.int32, device="cuda")
    loop(ref_states, ref_tokens, first)
    torch.cuda.synchronize()
    tok0, new0 = oracle.sample_step(tab, LG.f32_to_bf16_bits(xs[0]), BF16, start_np, 0.9, seed, first, row_stride=stride, top_k=40)
    assert np.array_equal(ref_tokens[0].cpu().numpy(), tok0) and np.array_equal(ref_states[1].cpu().numpy(), new0)
    assert len({tuple(r) for r in ref_tokens.cpu().numpy().tolist()}) > 1          # the steps do differ

    counter = torch.full((1,), first, dtype=torch.int64, device="cuda")
    g_states = torch.empty_like(ref_states)
    g_tokens = torch.empty_like(ref_tokens)
    loop(g_states, g_tokens, counter)                                            # eager, device offset
    torch.cuda.synchronize()
    assert torch.equal(g_tokens, ref_tokens) and torch.equal(g_states, ref_states)
    assert int(counter.item()) == first + S
    graph = torch.cuda.CUDAGraph()
    counter.fill_(first)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        loop(g_states, g_tokens, counter)
    for replay in range(3):
        g_tokens.fill_(-5)
        counter.fill_(first)
        scratch = (torch.arange(1000, device="cuda") * (replay + 1)).sum()      # the program's own eager work
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g_tokens, ref_tokens) and torch.equal(g_states, ref_states), f"replay {replay}"
        assert int(counter.item()) == first + S and int(scratch.item()) >= 0


@pytest.mark.parametrize("batch,n_tokens", [(3, 3000), (250, 40000)])
def test_masked_row_in_place(T, oracle, batch, n_tokens):
    """masked_out may be the logits themselves, states may be advanced in place, with a top-k cut."""
    tab = _rand_table(7, n_tokens, 0.2, 2)
    table = _upload_table(T, tab)
    rng = np.random.default_rng(batch)
    x = rng.normal(0, 2, size=(batch, n_tokens)).astype(np.float32)
    bits = LG.f32_to_bf16_bits(x)
    states = rng.integers(0, 7, size=batch).astype(np.int32)
    want_tok, want_new, want_masked = oracle.sample_step(tab, bits, BF16, states, 1.3, 8, 4, want_masked=True, top_k=25,
                                                         n_threads=16)
    lg = _to_dev(bits, BF16)
    st = torch.from_numpy(states).cuda()
    tok = torch.empty(batch, dtype=torch.int32, device="cuda")
    T.sample_step(table, lg, st, 1.3, 8, 4, tok, st, lg, top_k=25)
    torch.cuda.synchronize()
    assert np.array_equal(tok.cpu().numpy(), want_tok) and np.array_equal(st.cpu().numpy(), want_new)
    assert np.array_equal(_bits(lg), want_masked)
