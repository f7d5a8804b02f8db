"""GPU parity of the decode step (mask, argmax, advance) against the oracle, bit for bit."""
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
    """Device table from an oracle-side table (bits derived from it on the host)."""
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


def _step_and_check(T, oracle, table, table_np, lg_np, dtype, states_np, masked=True, stride=None):
    B = len(states_np)
    lg = _to_dev(lg_np, dtype)
    st = torch.from_numpy(states_np).cuda()
    tok = torch.full((B,), -9, dtype=torch.int32, device="cuda")
    new = torch.full((B,), -9, dtype=torch.int32, device="cuda")
    out = torch.empty_like(lg) if masked else None
    T.mask_step(table, lg, st, tok, new, out)
    torch.cuda.synchronize()
    res = oracle.mask_step(table_np, lg_np, dtype, states_np, row_stride=stride, want_masked=masked)
    assert np.array_equal(tok.cpu().numpy(), res[0]), (tok.cpu().numpy()[:8], res[0][:8])
    assert np.array_equal(new.cpu().numpy(), res[1])
    if masked:
        V = table_np.shape[1]
        assert np.array_equal(_bits(out)[:, :V], res[2].view(_bits(out).dtype)[:, :V])
    return res


def _rand_table(n_rows, n_tokens, p_live, seed):
    rng = np.random.default_rng(seed)
    t = rng.integers(0, n_rows, size=(n_rows, n_tokens), dtype=np.int32)
    t[rng.random((n_rows, n_tokens)) > p_live] = DEAD
    return t


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("n_tokens,batch", [(8, 1), (37 * 8, 3), (1000 * 8 + 8, 5), (40000, 2), (50024, 300),
                                            (5, 2), (37 * 8 + 3, 3), (1000 * 8 + 1, 5), (50021, 300), (98313, 48), (131075, 64), (131080, 200)])
def test_random_tables(T, oracle, dtype, n_tokens, batch):
    """Random sparse tables; sizes cover one group, ragged parts, many parts per row, one part per
    row, and rows whose length is not a multiple of the eight tokens a lane reads at once (the row
    stride is then rounded up, and the padding holds large values that must not be read)."""
    tab = _rand_table(11, n_tokens, 0.05, n_tokens + batch)
    tab[3] = DEAD
    tab[4] = DEAD
    tab[4, n_tokens - 1] = 6                                            # the only token allowed is the row's last
    tab[5, n_tokens - 1] = 2
    table = _upload_table(T, tab)
    rng = np.random.default_rng(batch)
    stride = (n_tokens + 7) // 8 * 8
    for trial in range(3):
        states = rng.integers(-1, 12, size=batch).astype(np.int32)      # includes DEAD and out of range
        states[: min(batch, 3)] = [3, 4, 5][: min(batch, 3)]
        x = np.full((batch, stride), 1000.0, dtype=np.float32)
        x[:, :n_tokens] = rng.normal(0, 2, size=(batch, n_tokens))
        if trial == 2:
            x[:, n_tokens - 1] = 50.0                                   # the winner sits in the last, partial group
        lg = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        _step_and_check(T, oracle, table, tab, lg, dtype, states, masked=trial != 1, stride=stride)


@pytest.mark.parametrize("n_tokens,batch", [(128256, 200), (128256, 7), (300000, 193), (300011, 16), (5000, 250),
                                            (400003, 193), (400003, 5),           # more than 64 KB of LDS for the allowed bits
                                            (1200011, 192), (983049, 288)])       # rows too long for the bits to sit in LDS at all
def test_sparse_and_mixed_rows(T, oracle, n_tokens, batch):
    _sparse_and_mixed_rows(T, oracle, n_tokens, batch, BF16)


@pytest.mark.parametrize("dtype,n_tokens,batch", [(BF16, v, b) for v, b in [
    (8192, 20), (8193, 20), (32760, 200), (32767, 16), (32769, 15), (32769, 16), (33003, 128), (33003, 129), (65528, 191), (65529, 192),
    (65536, 319), (65536, 320), (65537, 170), (65545, 171), (98307, 64), (131081, 65), (140000, 191), (250003, 100), (250003, 172),
    (48000, 171), (48001, 171), (56000, 170), (56001, 170),
    # the kernel with four groups per lane in flight: last groups, passes and wavefronts that are not whole, and more than 64 KB of LDS
    (65537, 288), (65545, 383), (128256, 300), (131075, 330), (460003, 288),
    (65528, 319), (65528, 320), (65536, 287), (65537, 287), (65545, 384)]] +
    [(F32, v, b) for v, b in [(98304, 48), (98312, 47), (98313, 48), (98313, 64), (131075, 102), (131075, 103), (131075, 191), (131075, 192)]])
def test_rows_at_the_edges_of_the_launch_shapes(T, oracle, dtype, n_tokens, batch):
    """Around the row lengths and batches at which rows are split into another number of workgroups, or of another size."""
    _sparse_and_mixed_rows(T, oracle, n_tokens, batch, dtype)


@pytest.mark.parametrize("n_tokens,batch", [(33003, 767), (33003, 768), (65521, 767), (65521, 768), (32003, 20), (50001, 64), (65545, 40), (131081, 300)])
def test_packed_rows_at_the_edges_of_the_launch_shapes(T, oracle, n_tokens, batch):
    _sparse_and_mixed_rows(T, oracle, n_tokens, batch, BF16, packed=True)


@pytest.mark.parametrize("n_tokens,batch", [(128256, 200), (128256, 7), (300011, 16), (5000, 250), (37 * 8 + 3, 3), (400003, 5)])
def test_sparse_and_mixed_rows_fp32(T, oracle, n_tokens, batch):
    _sparse_and_mixed_rows(T, oracle, n_tokens, batch, F32)


def _sparse_and_mixed_rows(T, oracle, n_tokens, batch, dtype, packed=False):
    """Rows from empty to full in one batch, around the density at which a wavefront stops fetching
    single groups and streams its stretch instead, with clustered rows (one stretch dense, the rest
    empty), heavy ties (rounded logits, so equal keys meet in every order) and special values."""
    rng = np.random.default_rng(n_tokens + batch)
    dens = [0.0, 1e-5, 2e-4, 1e-3, 4e-3, 7e-3, 8.5e-3, 1.2e-2, 5e-2, 0.5, 1.0]
    n_rows = len(dens) + 3
    tab = np.full((n_rows, n_tokens), DEAD, dtype=np.int32)
    for r, d in enumerate(dens):
        live = rng.random(n_tokens) < d
        tab[r, live] = rng.integers(0, n_rows, size=int(live.sum()), dtype=np.int32)
    r = len(dens)
    tab[r, : n_tokens // 40] = 1                                        # one dense cluster at the start
    tab[r + 1, n_tokens - n_tokens // 50:] = 2                          # one at the end, through the last group
    tab[r + 2, ::997] = 3                                               # a regular sprinkle
    tab[r + 2, n_tokens // 2: n_tokens // 2 + 700] = 4                  # plus a cluster in the middle
    table = _upload_table(T, tab)
    if packed:
        table = T.table_pack(table)
    stride = (n_tokens + 7) // 8 * 8
    for trial in range(3):
        states = rng.integers(0, n_rows, size=batch).astype(np.int32)
        states[: min(batch, n_rows)] = np.arange(n_rows)[: min(batch, n_rows)]
        x = np.full((batch, stride), 1000.0, dtype=np.float32)
        if trial == 0:
            x[:, :n_tokens] = rng.normal(0, 2, size=(batch, n_tokens))
        elif trial == 1:
            x[:, :n_tokens] = np.round(rng.normal(0, 1.5, size=(batch, n_tokens)))      # heavy ties
        else:
            x[:, :n_tokens] = rng.normal(-3, 1, size=(batch, n_tokens))
            x[:, rng.integers(0, n_tokens, 2000)] = np.nan
            x[:, rng.integers(0, n_tokens, 500)] = -np.inf
            x[:, rng.integers(0, n_tokens, 300)] = 0.0
        lg = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        _step_and_check(T, oracle, table, tab, lg, dtype, states, masked=False, stride=stride)


@pytest.mark.parametrize("dtype", [F32, BF16])
def test_special_values_and_ties(T, oracle, dtype):
    n_tokens = 4096 + 64
    tab = _rand_table(5, n_tokens, 0.3, 1)
    table = _upload_table(T, tab)
    rng = np.random.default_rng(9)
    states = np.array([0, 1, 2, 3, 4, 0, 1], dtype=np.int32)
    B = len(states)
    cases = []
    cases.append(np.full((B, n_tokens), 1.25, np.float32))                             # all equal
    cases.append(np.tile(np.arange(n_tokens, dtype=np.float32) / 64.0 - 20, (B, 1)))   # ramp up
    cases.append(np.tile(-np.arange(n_tokens, dtype=np.float32) / 64.0, (B, 1)))       # ramp down
    x = rng.normal(0, 2, size=(B, n_tokens)).astype(np.float32)
    x[:, rng.integers(0, n_tokens, 200)] = np.nan
    x[:, rng.integers(0, n_tokens, 50)] = np.inf
    x[:, rng.integers(0, n_tokens, 50)] = -np.inf
    cases.append(x)
    y = np.full((B, n_tokens), -np.inf, np.float32)                                    # only -inf and NaN
    y[:, rng.integers(0, n_tokens, 500)] = np.nan
    cases.append(y)
    cases.append(np.round(rng.normal(0, 2, size=(B, n_tokens))).astype(np.float32))    # heavy ties
    cases.append(np.where(rng.random((B, n_tokens)) < 0.5, -0.0, 0.0).astype(np.float32))   # signed zeros
    for x in cases:
        lg = x if dtype == F32 else LG.f32_to_bf16_bits(x)
        if dtype == BF16 and np.isnan(x).any():
            lg = lg.copy()
            nan_pos = np.argwhere(np.isnan(x))
            lg[nan_pos[::2, 0], nan_pos[::2, 1]] = 0xFFFF          # negative-sign NaN patterns too
            lg[nan_pos[1::2, 0], nan_pos[1::2, 1]] = 0x7F81
        _step_and_check(T, oracle, table, tab, lg, dtype, states)
        _step_and_check(T, oracle, table, tab, lg, dtype, states, masked=False)


@pytest.mark.parametrize("n_tokens,batch", [(8192, 1), (40000, 3), (16384, 200), (128256, 600)])
def test_rows_of_the_smallest_key(T, oracle, n_tokens, batch):
    """bf16 rows whose allowed logits are all the NaN pattern 0xFFFF, the only one whose order key is 0, in one stretch,
    in one part or in the whole row: every wavefront there has the same candidate, and one of them may speak for the
    workgroup.  The steps that follow find the words through which workgroups meet as they should be.  Dense and packed."""
    rng = np.random.default_rng(n_tokens)
    tab = _rand_table(4, n_tokens, 0.6, 5)
    dense = _upload_table(T, tab)
    counted, _ = T.table_concat([dense])
    tables = (dense, counted, T.table_pack(dense))
    states = (np.arange(batch) % 4).astype(np.int32)
    stride = (n_tokens + 7) // 8 * 8
    plain = LG.f32_to_bf16_bits(rng.normal(0, 2, size=(batch, stride)).astype(np.float32))
    whole, part = plain.copy(), plain.copy()
    whole[:, :] = 0xFFFF
    part[:, :n_tokens // 2] = 0xFFFF
    one = whole.copy()
    one[:, n_tokens - 5:] = plain[:, n_tokens - 5:]
    st = torch.from_numpy(states).cuda()
    for lg in (whole, plain, part, plain, one, whole, plain):
        want = oracle.mask_step(tab, lg, BF16, states, row_stride=stride)
        dev = _to_dev(lg, BF16)
        for table in tables:
            tok = torch.full((batch,), -9, dtype=torch.int32, device="cuda")
            new = torch.full((batch,), -9, dtype=torch.int32, device="cuda")
            T.mask_step(table, dev, st, tok, new)
            torch.cuda.synchronize()
            assert np.array_equal(tok.cpu().numpy(), want[0]) and np.array_equal(new.cpu().numpy(), want[1])


@pytest.mark.parametrize("n_tokens,batch", [(1, 3), (7, 2), (4093, 5), (4096, 5), (8197, 4), (16387, 9), (33001, 200), (32775, 193),
                                            (131075, 51), (131075, 52), (98313, 255), (98313, 256)])
def test_penalised_fp32_rows_at_the_edges(T, oracle, n_tokens, batch):
    """fp32 rows written with the penalty, around the 1,024 and 4,096 logits that a workgroup takes per load and per
    round, with partial groups, in place and into another buffer whose padding must stay as it was; bit for bit."""
    tab = _rand_table(6, n_tokens, 0.4, n_tokens)
    tab[2] = DEAD
    tab[3] = 1
    table = _upload_table(T, tab)
    rng = np.random.default_rng(batch)
    stride = (n_tokens + 3) // 4 * 4 + 8
    x = (np.round(rng.normal(0, 2, size=(batch, stride)) * 8) / 8).astype(np.float32)
    x[:, rng.integers(0, n_tokens, 3)] = np.nan
    states = (np.arange(batch) % 8 - 1).astype(np.int32)
    want = oracle.mask_step(tab, x, F32, states, row_stride=stride, want_masked=True)
    for in_place in (False, True):
        lg = _to_dev(x, F32)
        out = lg if in_place else torch.full_like(lg, 7.0)
        tok = torch.full((batch,), -9, dtype=torch.int32, device="cuda")
        new = torch.full((batch,), -9, dtype=torch.int32, device="cuda")
        T.mask_step(table, lg, torch.from_numpy(states).cuda(), tok, new, out)
        torch.cuda.synchronize()
        assert np.array_equal(tok.cpu().numpy(), want[0]) and np.array_equal(new.cpu().numpy(), want[1])
        got = _bits(out)
        assert np.array_equal(got[:, :n_tokens], want[2].view(np.uint32)[:, :n_tokens])
        rest = x[:, n_tokens:].view(np.uint32) if in_place else np.full((batch, stride - n_tokens), np.float32(7.0).view(np.uint32))
        assert np.array_equal(got[:, n_tokens:], rest)


@pytest.mark.parametrize("how", ["graphs", "noalloc"])
def test_penalised_fp32_rows_of_two_steps_at_once(T, oracle, how):
    """256 rows and more, written with the penalty: such rows meet through no scratch, so two recorded steps of one stream,
    or two steps through the library's static scratch, may run side by side; and eager ones, which do, give the same."""
    n_tokens, batch = 100003, 300
    tab = _rand_table(6, n_tokens, 0.4, 5)
    table = _upload_table(T, tab)
    rng = np.random.default_rng(6)
    side = [torch.cuda.Stream() for _ in range(3)]
    step = {"graphs": T.mask_step, "noalloc": T.mask_step_noalloc}[how]
    runs = []
    for i in range(2):
        x = (np.round(rng.normal(0, 2, size=(batch, n_tokens + 5)) * 8) / 8).astype(np.float32)
        states = rng.integers(-1, 6, size=batch).astype(np.int32)
        want = oracle.mask_step(tab, x, F32, states, row_stride=n_tokens + 5, want_masked=True)
        dev = _to_dev(x, F32)
        args = [dev, torch.from_numpy(states).cuda()] + [torch.full((batch,), -9, dtype=torch.int32, device="cuda") for _ in range(2)] + [torch.zeros_like(dev)]
        T.mask_step(table, *args)
        torch.cuda.synchronize()
        assert np.array_equal(args[2].cpu().numpy(), want[0]) and np.array_equal(args[3].cpu().numpy(), want[1])
        graph = None
        if how == "graphs":
            with torch.cuda.stream(side[2]):
                step(table, *args)
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side[2]):
                step(table, *args)
        runs.append((args, want, graph))
    torch.cuda.synchronize()
    for _ in range(10):
        for args, _, _ in runs:
            args[2].fill_(-9)
            args[4].zero_()
        torch.cuda.synchronize()
        for i, (args, _, graph) in enumerate(runs):
            with torch.cuda.stream(side[i]):
                if graph is not None:
                    graph.replay()
                else:
                    step(table, *args)
        torch.cuda.synchronize()
        for args, want, _ in runs:
            assert np.array_equal(args[2].cpu().numpy(), want[0]) and np.array_equal(args[3].cpu().numpy(), want[1])
            assert np.array_equal(_bits(args[4])[:, :n_tokens], want[2].view(np.uint32)[:, :n_tokens])


def test_stride_inplace_and_alias(T, oracle):
    n_tokens = 3000
    tab = _rand_table(7, n_tokens, 0.2, 2)
    table = _upload_table(T, tab)
    rng = np.random.default_rng(1)
    B = 9
    wide = rng.normal(0, 2, size=(B, 3008)).astype(np.float32)
    wide_b = LG.f32_to_bf16_bits(wide)
    states = rng.integers(0, 7, size=B).astype(np.int32)
    want_tok, want_new, want_masked = oracle.mask_step(tab, wide_b, BF16, states, row_stride=3008, want_masked=True)
    lg = _to_dev(wide_b, BF16)
    st = torch.from_numpy(states).cuda()
    tok = torch.empty(B, dtype=torch.int32, device="cuda")
    T.mask_step(table, lg, st, tok, st, lg)          # states advanced in place, logits masked in place
    torch.cuda.synchronize()
    assert np.array_equal(tok.cpu().numpy(), want_tok) and np.array_equal(st.cpu().numpy(), want_new)
    got = _bits(lg)
    assert np.array_equal(got[:, :n_tokens], want_masked[:, :n_tokens])
    assert np.array_equal(got[:, n_tokens:], wide_b[:, n_tokens:])      # padding columns untouched
    with pytest.raises(T.TdfaError):
        T.mask_step(table, lg[:, 1:], st, tok, st)                       # misaligned rows


def _decode(T, oracle, table, table_np, w, start_states, steps, seed, block=64):
    """Runs `steps` chained steps on the device, in blocks of `block` steps with no host sync inside
    a block, and checks every step: the oracle runs its own chained decode from the same start
    states on the same logits (each step's device logits are kept and handed over), and the
    device's tokens and states must equal the oracle's at every step."""
    m = w.mask
    B, V = m.batch, w.vocab.n_tokens
    tdt = torch.float32 if m.dtype == "f32" else torch.bfloat16
    dt = F32 if m.dtype == "f32" else BF16
    hist_states = torch.empty((steps + 1, B), dtype=torch.int32, device="cuda")
    hist_tok = torch.empty((steps, B), dtype=torch.int32, device="cuda")
    hist_states[0] = torch.from_numpy(start_states.astype(np.int32)).cuda()
    kept = torch.empty((min(block, steps), B, V), dtype=tdt, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    orc_states = start_states.astype(np.int32)
    for s0 in range(0, steps, block):
        s1 = min(steps, s0 + block)
        for s in range(s0, s1):
            LG.gen_logits_device(kept[s - s0].data_ptr(), seed, s, B, V, V, m.sigma, m.dtype, stream)
            T.mask_step(table, kept[s - s0], hist_states[s], hist_tok[s], hist_states[s + 1])
        torch.cuda.synchronize()
        hs, ht = hist_states[s0:s1 + 1].cpu().numpy(), hist_tok[s0:s1].cpu().numpy()
        for s in range(s0, s1):
            lg_np = _bits(kept[s - s0]) if dt == BF16 else kept[s - s0].cpu().numpy()
            assert np.array_equal(hs[s - s0], orc_states), f"step {s}: input states differ"
            tok, orc_states = oracle.mask_step(table_np, lg_np, dt, orc_states, n_threads=16)
            assert np.array_equal(ht[s - s0], tok), f"step {s}: tokens differ"
            assert np.array_equal(hs[s - s0 + 1], orc_states), f"step {s}: states differ"
    return hist_states.cpu().numpy(), hist_tok.cpu().numpy()


def test_device_logits_match_host(T):
    for dtype, tdt in (("f32", torch.float32), ("bf16", torch.bfloat16)):
        B, V = 5, 128256
        buf = torch.empty((B, V), dtype=tdt, device="cuda")
        LG.gen_logits_device(buf.data_ptr(), 777, 12, B, V, V, 2.0, dtype, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        host = LG.gen_logits(777, 12, B, V, 2.0, dtype)
        got = buf.cpu().numpy() if dtype == "f32" else _bits(buf)
        assert np.array_equal(got, host)


def _compile_all(T, w):
    v = T.Vocab(w.vocab.data, w.vocab.offsets)
    return v, [T.compile_token_dfa(v, T.CharDFA(d.trans, d.accept, d.start)) for d in w.dfas]


def _dfa_handles(T, w):
    return [T.CharDFA(d.trans, d.accept, d.start) for d in w.dfas]


def test_c1_decode(T, oracle):
    w = configs.get("c1")
    v, (table,) = _compile_all(T, w)
    d = w.dfas[0]
    tab = oracle.compile_compose(d.trans, w.vocab.data, w.vocab.offsets)
    hs, ht = _decode(T, oracle, table, tab, w, np.full(4, d.start), 16, configs.logits_seed(1))
    assert (ht >= 0).any()


def test_c2_decode(T, oracle):
    w = configs.get("c2")
    v, (table,) = _compile_all(T, w)
    d = w.dfas[0]
    tab = oracle.compile_walk(d.trans, w.vocab.data, w.vocab.offsets, n_threads=8)
    hs, ht = _decode(T, oracle, table, tab, w, np.full(64, d.start), 256, configs.logits_seed(2))
    # sequences that stopped did so in a final state (the caller's check)
    stopped = ht[-1] < 0
    assert d.accept[hs[-1][stopped]].all()


def test_c3_decode_full_size(T, oracle):
    w = configs.get("c3")
    v, (table,) = _compile_all(T, w)
    d = w.dfas[0]
    tab = oracle.compile_walk(d.trans, w.vocab.data, w.vocab.offsets, n_threads=16)
    hs, ht = _decode(T, oracle, table, tab, w, np.full(256, d.start), 512, configs.logits_seed(3))
    assert len(np.unique(hs)) > 50          # the batch spreads over many states


def test_c5_decode_full_size(T, oracle):
    """64 constraints, 1,024 sequences: compile all, stack, compare the whole stacked table, decode."""
    w = configs.get("c5")
    v, tabs = _compile_all(T, w)
    big, offs = T.table_concat(tabs)
    torch.cuda.synchronize()
    want = [oracle.compile_walk(d.trans, w.vocab.data, w.vocab.offsets, n_threads=16) for d in w.dfas]
    ref, ref_offs = oracle.concat_tables(want)
    del want
    assert np.array_equal(offs, ref_offs)
    # the same stacked table written in place, one compile per constraint into its slice
    direct, offs2 = T.compile_stacked(v, _dfa_handles(T, w))
    torch.cuda.synchronize()
    assert np.array_equal(offs2, ref_offs)
    for lo in range(0, ref.shape[0], 1024):
        hi = min(ref.shape[0], lo + 1024)
        G.check_rows(big, ref[lo:hi], np.arange(lo, hi))
        G.check_rows(direct, ref[lo:hi], np.arange(lo, hi))
    del big
    # and as bench.py compiles it: the union of the 64 automata as one automaton
    union, offs3 = T.dfa_union(_dfa_handles(T, w))
    whole = T.compile_token_dfa(v, union)
    torch.cuda.synchronize()
    assert np.array_equal(offs3, ref_offs)
    for lo in range(0, ref.shape[0], 1024):
        hi = min(ref.shape[0], lo + 1024)
        G.check_rows(whole, ref[lo:hi], np.arange(lo, hi))
    del whole, union
    big = direct
    start = np.array([offs[c] + w.dfas[c].start for c in w.binding], dtype=np.int32)
    hs, ht = _decode(T, oracle, big, ref, w, start, 512, configs.logits_seed(5), block=32)
    # every sequence stays inside its own constraint's rows
    lo, hi = offs[w.binding], offs[w.binding + 1]
    assert ((hs >= lo) & (hs < hi)).all()


def test_decode_twice_same_bytes(T, oracle):
    """Determinism: the same 64 chained steps run twice (the second time with the rows split over
    several workgroups' worth of other traffic in between) give the same tokens and states."""
    w = configs.get("c2")
    v, (table,) = _compile_all(T, w)
    d, m = w.dfas[0], w.mask
    B, V, S = m.batch, w.vocab.n_tokens, 64
    logits = torch.empty((S, B, V), dtype=torch.bfloat16, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    for s in range(S):
        LG.gen_logits_device(logits[s].data_ptr(), configs.logits_seed(2), s, B, V, V, m.sigma, m.dtype, stream)
    runs = []
    for r in range(2):
        states = torch.empty((S + 1, B), dtype=torch.int32, device="cuda")
        tokens = torch.empty((S, B), dtype=torch.int32, device="cuda")
        states[0].fill_(d.start)
        for s in range(S):
            T.mask_step(table, logits[s], states[s], tokens[s], states[s + 1])
        torch.cuda.synchronize()
        runs.append((states, tokens))
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])
