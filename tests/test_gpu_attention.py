"""GPU parity and bitwise-consistency tests of the unified attention path.

Parity: GPU outputs vs the fp64 oracle under the gate (mean |err| <= 5e-4,
per element |err| <= 4e-3 + 2^-8 |ref|).  Consistency (Eq. (1) at operator
level, Section 3.2): every decoded row equals the full-sequence row at the
same position bit for bit, under varied batch mixes, orders and splits.
"""
import numpy as np
import pytest

import oracle
from paper_2609_35140_amd import inputs

pytestmark = pytest.mark.gpu

gu = pytest.importorskip("gpu_util")


@pytest.fixture(scope="module")
def ua():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_35140_amd import uattn
    uattn.lib()
    return uattn


def _prefill(ua, pk, lse=True):
    out, l = ua.prefill(pk.q, pk.k, pk.v, pk.cu_dev, pk.max_seqlen, return_lse=True)
    return out, l


SMALL = [
    ("tiny_s1", lambda: inputs.tiny(), 1),
    ("tiny_s42", lambda: inputs.tiny(), 42),
    ("tiny_s1023", lambda: inputs.tiny(), 1023),
    ("d128_g4_ragged", lambda: inputs.custom(8, 2, 128, [1, 63, 64, 65, 300, 700], sigma=1.0, page_size=64), 42),
    ("d64_g5_ragged", lambda: inputs.custom(10, 2, 64, [31, 257, 513, 130], sigma=1.0, page_size=16), 42),
    ("d128_g8", lambda: inputs.custom(16, 2, 128, [1000, 257], sigma=0.5, page_size=64), 42),
    ("d128_mha", lambda: inputs.custom(3, 3, 128, [200, 77], sigma=1.0, page_size=32), 42),
    ("d64_g32", lambda: inputs.custom(32, 1, 64, [300], sigma=1.0, page_size=128), 42),
]


@pytest.mark.parametrize("name,mk,seed", SMALL, ids=[s[0] for s in SMALL])
def test_prefill_matches_oracle(ua, name, mk, seed):
    w = mk()
    pk = gu.Pack(w, seed=seed)
    out, lse = _prefill(ua, pk)
    o64, lse64 = oracle.causal_attention_fp64(pk.host["q"], pk.host["k"], pk.host["v"], pk.cu)
    rep = oracle.parity_report(gu.host_f64(out), o64)
    print(name, rep, flush=True)
    assert rep["pass"], rep
    lg = lse.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(lg - lse64)) < oracle.LSE_ABS, np.max(np.abs(lg - lse64))


@pytest.mark.parametrize("name,mk,seed", SMALL, ids=[s[0] for s in SMALL])
def test_decode_every_position_bitwise_equals_prefill(ua, name, mk, seed):
    """Decode of every (sequence, position) in one batched call equals the
    full-sequence output rows bit for bit, lse included."""
    w = mk()
    pk = gu.Pack(w, seed=seed)
    out, lse = _prefill(ua, pk)
    entries = [(s, p) for s, L in enumerate(w.seq_lens) for p in range(L)]
    q, table, seqlens, maxs, tok = pk.decode_rows(entries)
    dout, dlse = ua.decode(q, pk.kp, pk.vp, table, seqlens, maxs, return_lse=True)
    a = gu.host_bits(dout)
    b = gu.host_bits(out)[tok]
    eq = gu.rows_equal_bits(a, b)
    print(name, "bitwise rows", eq.mean(), flush=True)
    assert eq.all(), f"{(~eq).sum()} of {eq.size} rows differ"
    assert np.array_equal(dlse.cpu().numpy().view(np.uint32), lse.cpu().numpy()[tok].view(np.uint32))
    # and the decode result itself meets the oracle gate
    o64, _ = oracle.paged_decode_fp64(pk.host["q"][tok], pk.kp_host, pk.vp_host, pk.table[[s for s, _ in entries]],
                                      [p + 1 for _, p in entries])
    assert oracle.parity_report(gu.host_f64(dout), o64)["pass"]


@pytest.mark.parametrize("name,mk,seed", SMALL, ids=[s[0] for s in SMALL])
def test_long_walk_split_merge_bitwise(ua, name, mk, seed):
    """A walk of at least 16 items per CU (forced here by a max_seqlen far
    above the lengths) keeps its chunk partials in LDS, writes them in bursts
    and folds them in a kernel of its own after the walk: every decoded
    position still equals its prefill row bit for bit, lse included, and the
    call with the tight max_seqlen."""
    import torch
    w = mk()
    entries = [(s, p) for s, L in enumerate(w.seq_lens) for p in range(L)]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    nchunk = -(-16 * cus // (len(entries) * w.num_kv_heads)) + 1
    big = max(256 * nchunk, max(w.seq_lens))
    page = w.page_size
    pk = gu.Pack(w, seed=seed, table_slack=-(-big // page))
    assert pk.table.shape[1] * pk.page >= big
    assert len(entries) * w.num_kv_heads * (-(-big // 256)) >= 16 * cus
    out, lse = _prefill(ua, pk)
    q, table, seqlens, maxs, tok = pk.decode_rows(entries)
    dout, dlse = ua.decode(q, pk.kp, pk.vp, table, seqlens, big, return_lse=True)
    eq = gu.rows_equal_bits(gu.host_bits(dout), gu.host_bits(out)[tok])
    print(name, "long walk bitwise rows", eq.mean(), "max_seqlen", big, flush=True)
    assert eq.all(), f"{(~eq).sum()} of {eq.size} rows differ"
    assert np.array_equal(dlse.cpu().numpy().view(np.uint32), lse.cpu().numpy()[tok].view(np.uint32))
    tight, tight_lse = ua.decode(q, pk.kp, pk.vp, table, seqlens, maxs, return_lse=True)
    assert torch.equal(tight.view(torch.int16), dout.view(torch.int16))
    assert torch.equal(tight_lse.view(torch.int32), dlse.view(torch.int32))


def test_rising_scores_rescale_path(ua):
    """Keys growing along the sequence make the online softmax's running
    maximum jump inside and across chunks (large rescales and fold factors):
    the prefill meets the oracle gate and every decoded position equals its
    prefill row bit for bit, lse included."""
    w = inputs.custom(8, 2, 128, [700, 300, 65], sigma=0.5, page_size=64)
    pk = gu.Pack(w, seed=42, key_ramp=8.0)
    out, lse = _prefill(ua, pk)
    o64, lse64 = oracle.causal_attention_fp64(pk.host["q"], pk.host["k"], pk.host["v"], pk.cu)
    rep = oracle.parity_report(gu.host_f64(out), o64)
    print("rising scores", rep, flush=True)
    assert rep["pass"], rep
    lg = lse.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(lg - lse64)) < oracle.LSE_ABS
    entries = [(s, p) for s, L in enumerate(w.seq_lens) for p in range(L)]
    q, table, seqlens, maxs, tok = pk.decode_rows(entries)
    dout, dlse = ua.decode(q, pk.kp, pk.vp, table, seqlens, maxs, return_lse=True)
    eq = gu.rows_equal_bits(gu.host_bits(dout), gu.host_bits(out)[tok])
    assert eq.all(), f"{(~eq).sum()} of {eq.size} rows differ"
    assert np.array_equal(dlse.cpu().numpy().view(np.uint32), lse.cpu().numpy()[tok].view(np.uint32))


def test_rollout_replay_eq1(ua):
    """Eq. (1): full prefill of p||y equals prefill(p) at prompt rows and
    token-by-token decode (batch of all sequences each step) at response rows."""
    import torch
    w = inputs.custom(8, 2, 128, [64 + 64, 200 + 100, 300 + 40], sigma=1.0, page_size=16,
                      prompt_lens=[64, 200, 300])
    pk = gu.Pack(w, seed=7)
    full = gu.host_bits(_prefill(ua, pk)[0])
    # rollout prefill over prompts only (its own pack of the prompt tokens)
    P = w.prompt_lens
    idx = np.concatenate([np.arange(pk.cu[s], pk.cu[s] + P[s]) for s in range(w.num_seqs)])
    it = torch.from_numpy(idx).cuda()
    cu_p = gu.dev_i32(inputs.cu_seqlens(P))
    pout = gu.host_bits(ua.prefill(pk.q[it].contiguous(), pk.k[it].contiguous(), pk.v[it].contiguous(), cu_p, max(P)))
    assert np.array_equal(pout, full[idx]), "prompt rows: prefill(p) != prefill(p||y)"
    # token-by-token decode; finished sequences drop out of the batch
    R = [L - p for L, p in zip(w.seq_lens, P)]
    mism = 0
    for step in range(max(R)):
        entries = [(s, P[s] + step) for s in range(w.num_seqs) if step < R[s]]
        q, table, seqlens, maxs, tok = pk.decode_rows(entries)
        d = gu.host_bits(ua.decode(q, pk.kp, pk.vp, table, seqlens, max(w.seq_lens)))
        mism += int((~gu.rows_equal_bits(d, full[tok])).sum())
    assert mism == 0, mism


def test_decode_batch_mix_permutation_and_split_invariance(ua):
    """The same decode entry gives the same bits alone, in a batch, in any
    order, with any max_seqlen (grid/workspace size)."""
    w = inputs.custom(8, 2, 128, [1500, 900, 77, 2100], sigma=0.5, page_size=64)
    pk = gu.Pack(w, seed=11)
    rng = np.random.default_rng(5)
    entries = [(s, int(rng.integers(0, w.seq_lens[s]))) for s in range(4) for _ in range(9)]
    q, table, seqlens, maxs, tok = pk.decode_rows(entries)
    ref = gu.host_bits(ua.decode(q, pk.kp, pk.vp, table, seqlens, maxs))
    for trial in range(3):
        perm = rng.permutation(len(entries))
        q2, t2, s2, m2, _ = pk.decode_rows([entries[i] for i in perm])
        cap = pk.table.shape[1] * pk.page          # largest max_seqlen the block table allows
        got = gu.host_bits(ua.decode(q2, pk.kp, pk.vp, t2, s2, [m2, m2 + 257, cap][trial]))
        assert np.array_equal(got, ref[perm])
    for i in [0, 17, 35]:
        q1, t1, s1, m1, _ = pk.decode_rows([entries[i]])
        assert np.array_equal(gu.host_bits(ua.decode(q1, pk.kp, pk.vp, t1, s1, m1)), ref[i:i + 1])


def test_prefill_pack_order_and_max_seqlen_invariance(ua):
    w = inputs.custom(4, 1, 128, [333, 64, 1025], sigma=1.0)
    pk = gu.Pack(w, seed=3)
    ref = gu.host_bits(_prefill(ua, pk)[0])
    import torch
    order = [2, 0, 1]
    idx = np.concatenate([np.arange(pk.cu[s], pk.cu[s + 1]) for s in order])
    it = torch.from_numpy(idx).cuda()
    cu2 = gu.dev_i32(inputs.cu_seqlens([w.seq_lens[s] for s in order]))
    got = gu.host_bits(ua.prefill(pk.q[it].contiguous(), pk.k[it].contiguous(), pk.v[it].contiguous(), cu2, 4000))
    assert np.array_equal(got, ref[idx])


def test_run_to_run_determinism(ua):
    w = inputs.custom(8, 2, 128, [700, 300], sigma=1.0)
    pk = gu.Pack(w, seed=13)
    a = gu.host_bits(_prefill(ua, pk)[0])
    b = gu.host_bits(_prefill(ua, pk)[0])
    assert np.array_equal(a, b)
    entries = [(0, 699), (1, 299), (0, 256), (0, 255)]
    q, t, s, m, _ = pk.decode_rows(entries)
    x = gu.host_bits(ua.decode(q, pk.kp, pk.vp, t, s, m))
    y = gu.host_bits(ua.decode(q, pk.kp, pk.vp, t, s, m))
    assert np.array_equal(x, y)


def test_unwritten_slots_are_never_read(ua):
    """Cache slots past each context hold NaN (and +/-Inf): outputs are finite
    and unchanged versus a zero-filled cache."""
    w = inputs.custom(8, 2, 128, [100, 37, 300], sigma=1.0, page_size=64)
    nan = gu.Pack(w, seed=21, fill_bits=0x7FC0)
    inf = gu.Pack(w, seed=21, fill_bits=0xFF80)
    zero = gu.Pack(w, seed=21, fill_bits=0x0000)
    entries = [(0, 99), (1, 36), (2, 299), (2, 64), (0, 0)]
    outs = []
    for pk in (nan, inf, zero):
        q, t, s, m, _ = pk.decode_rows(entries)
        outs.append(gu.host_bits(ua.decode(q, pk.kp, pk.vp, t, s, m)))
    q, t, s, m, _ = nan.decode_rows(entries)
    assert not np.isnan(gu.host_f64(ua.decode(q, nan.kp, nan.vp, t, s, 300))).any()
    assert np.array_equal(outs[0], outs[2]) and np.array_equal(outs[1], outs[2])


def test_single_token_context_returns_v(ua):
    w = inputs.custom(8, 2, 128, [1, 1, 5], sigma=1.0, page_size=16)
    pk = gu.Pack(w, seed=2)
    out = gu.host_bits(_prefill(ua, pk)[0])
    v = pk.host["v"]
    for tok in [0, 1, 2]:
        for h in range(8):
            assert np.array_equal(out[tok, h], v[tok, h // 4])
    q, t, s, m, tk = pk.decode_rows([(0, 0), (2, 0)])
    d = gu.host_bits(ua.decode(q, pk.kp, pk.vp, t, s, m))
    assert np.array_equal(d[1, 5], v[2, 1])


def test_empty_sequences_in_pack(ua):
    w = inputs.custom(4, 2, 64, [0, 5, 0, 70, 0], sigma=1.0)
    pk = gu.Pack(w, seed=4)
    out, lse = _prefill(ua, pk)
    o64, _ = oracle.causal_attention_fp64(pk.host["q"], pk.host["k"], pk.host["v"], pk.cu)
    assert oracle.parity_report(gu.host_f64(out), o64)["pass"]


def test_hip_graph_replay_with_varying_inputs(ua):
    """Decode and prefill captured in a HIP graph, replayed with new inputs
    copied into the captured buffers: every replay equals eager execution."""
    import torch
    w = inputs.custom(8, 2, 128, [600, 300], sigma=1.0, page_size=64)
    pk = gu.Pack(w, seed=31)
    entries = [(0, 599), (1, 299)]
    q, t, s, m, _ = pk.decode_rows(entries)
    ws = ua.new_workspace(ua.decode_workspace_bytes(2, 600, 8, 128))
    dout = torch.empty_like(q)
    pout = torch.empty_like(pk.q)
    qbuf = pk.q.clone()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        ua.prefill(qbuf, pk.k, pk.v, pk.cu_dev, 600, out=pout)
        ua.decode(q, pk.kp, pk.vp, t, s, 600, out=dout, workspace=ws)
    rng = np.random.default_rng(0)
    for rep in range(4):
        newq = gu.dev(inputs.normal_bf16(tuple(pk.q.shape), 1.0, 77, rep))
        qbuf.copy_(newq)
        q.copy_(newq[torch.tensor([599, 600 + 299], device="cuda")])
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        eager_p = ua.prefill(newq, pk.k, pk.v, pk.cu_dev, 600)
        eager_d = ua.decode(q.clone(), pk.kp, pk.vp, t, s, 600)
        torch.cuda.synchronize()
        assert torch.equal(pout.view(torch.int16), eager_p.view(torch.int16)), rep
        assert torch.equal(dout.view(torch.int16), eager_d.view(torch.int16)), rep
        _ = rng


def test_mfma_column_slot_independence(ua):
    """The same query placed in different MFMA columns (different positions in
    a prefill wave, different head slots in decode) gives the same bits: a
    sequence whose every query row equals one vector, with K/V constant past
    position 0, forces rows across the wave to share arithmetic."""
    d, L = 128, 96
    w = inputs.custom(2, 1, d, [L], sigma=1.0)
    pk = gu.Pack(w, seed=5)
    import torch
    qrow = pk.q[0:1, 0:1, :]
    q = qrow.expand(L, 2, d).contiguous()
    out = gu.host_bits(ua.prefill(q, pk.k, pk.v, pk.cu_dev, L))
    # heads 0 and 1 (different decode columns) hold identical queries
    assert np.array_equal(out[:, 0], out[:, 1])
    ents = [(0, p) for p in range(L)]
    qd, t, s, m, tok = pk.decode_rows(ents)
    qd = q[torch.from_numpy(tok).cuda()].contiguous()
    d_out = gu.host_bits(ua.decode(qd, pk.kp, pk.vp, t, s, m))
    assert np.array_equal(d_out, out[tok])


def test_workspace_reuse_across_batch_sizes(ua):
    """One zero-filled workspace serves a run of calls of different batch sizes
    and lengths; results equal those with fresh workspaces, and the counter
    words are zero after every call."""
    import torch
    w = inputs.custom(8, 2, 128, [2100, 900, 1500, 300, 1800], sigma=0.5, page_size=64)
    pk = gu.Pack(w, seed=17)
    rng = np.random.default_rng(9)
    big = ua.decode_workspace_bytes(40, 2100, 8, 128)
    ws = ua.new_workspace(big)
    for trial, nb in enumerate([40, 7, 40, 3, 25, 1]):
        ents = [(int(s), int(rng.integers(0, w.seq_lens[s]))) for s in rng.integers(0, 5, size=nb)]
        q, t, s, m, _ = pk.decode_rows(ents)
        maxs = [2100, m, 2100, m, 1024 if m <= 1024 else m, m][trial]
        got = ua.decode(q, pk.kp, pk.vp, t, s, maxs, workspace=ws)
        ref = ua.decode(q, pk.kp, pk.vp, t, s, maxs)
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16)), trial
        torch.cuda.synchronize()
        cnt = ws[: ua.counter_bytes(nb, 8)].view(torch.int32)
        assert int(cnt.abs().sum().item()) == 0, trial


def test_workspace_at_a_reused_address_holding_garbage(ua):
    """A caller's workspace that is not from new_workspace, at a device address
    an earlier workspace used, holding garbage: the binding zeroes its counter
    region on first use (it keeps no record keyed by address), so results equal
    a fresh workspace's every time."""
    import torch
    w = inputs.custom(8, 2, 128, [2100, 900, 1500], sigma=0.5, page_size=64)
    pk = gu.Pack(w, seed=29)
    ents = [(0, 2099), (1, 899), (2, 1499), (0, 700)]
    q, t, s, m, _ = pk.decode_rows(ents)
    ref = ua.decode(q, pk.kp, pk.vp, t, s, m)
    need = ua.decode_workspace_bytes(len(ents), m, 8, 128)
    addrs = set()
    for trial in range(3):
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        addrs.add(ws.data_ptr())
        ws.fill_(0xA5)                      # garbage where the arrival counters live
        got = ua.decode(q, pk.kp, pk.vp, t, s, m, workspace=ws)
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16)), trial
        got = ua.decode(q, pk.kp, pk.vp, t, s, m, workspace=ws)   # second call on the same tensor
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16)), trial
        torch.cuda.synchronize()
        del ws, got                         # the caching allocator hands the same block out again
    print(f"workspace addresses seen: {len(addrs)} (1 means every trial reused the freed block)", flush=True)


def test_oversized_max_seqlen_gives_the_same_bits(ua):
    """max_seqlen far above every entry's length (a caller passing its
    allocation size): the kernel's walk stops after the longest entry's last
    chunk, and outputs and lse equal those with the true maximum and the
    prefill rows bit for bit."""
    import torch
    w = inputs.custom(32, 8, 128, [700, 300, 1200, 90, 513, 256, 1000, 64], sigma=0.5, page_size=64)
    pk = gu.Pack(w, seed=19, table_slack=112)          # table rows cover 8192 positions
    out, lse = ua.prefill(pk.q, pk.k, pk.v, pk.cu_dev, pk.max_seqlen, return_lse=True)
    rng = np.random.default_rng(23)
    ents = [(int(s), int(rng.integers(0, w.seq_lens[s]))) for s in rng.integers(0, len(w.seq_lens), size=48)]
    q, t, s, m, tok = pk.decode_rows(ents)
    assert pk.table.shape[1] * pk.page >= 8192
    big, big_lse = ua.decode(q, pk.kp, pk.vp, t, s, 8192, return_lse=True)
    tight, tight_lse = ua.decode(q, pk.kp, pk.vp, t, s, m, return_lse=True)
    ti = torch.from_numpy(tok).cuda()
    assert torch.equal(big.view(torch.int16), tight.view(torch.int16))
    assert torch.equal(big_lse.view(torch.int32), tight_lse.view(torch.int32))
    assert torch.equal(big.view(torch.int16), out[ti].view(torch.int16))
    assert torch.equal(big_lse.view(torch.int32), lse[ti].view(torch.int32))


@pytest.mark.parametrize("batch,hkv,group,d,longest", [(63, 8, 1, 64, 1024), (64, 8, 5, 128, 1030), (65, 8, 2, 64, 1024),
                                                       (130, 4, 17, 128, 900), (300, 8, 4, 64, 1500),
                                                       (1024, 2, 1, 64, 700), (1025, 2, 1, 64, 700)])
def test_ragged_decode_walk_lists_every_chunk(ua, batch, hkv, group, d, longest):
    """Long walks over ragged batches (with empty entries) list the chunks that hold keys, one or several entries to a
    lane, up to 1024 entries: every entry's output and lse equal those of short calls of 8 entries, empty ones stay
    unwritten."""
    import torch
    page = 64
    hq = hkv * group
    lens = inputs.rng(71, batch, longest).integers(0, longest, size=batch, endpoint=True)
    lens[inputs.rng(72, batch).integers(0, batch, size=max(1, batch // 10))] = 0
    lens[0], lens[-1] = (0, longest) if batch % 2 else (longest, 0)
    maxp = (longest + page - 1) // page
    pages = 97                                        # entries share pages of a small pool
    table = gu.dev_i32(inputs.rng(73, batch).integers(0, pages, size=(batch, maxp)))
    q = inputs.normal_bf16_device((batch, hq, d), 1.0, 74, batch)
    kp = inputs.normal_bf16_device((pages, hkv, page, d), 1.0, 75, batch)
    vp = inputs.normal_bf16_device((pages, hkv, page, d), 1.0, 76, batch)
    sl = gu.dev_i32(lens)
    out = torch.full_like(q, 7.0)
    lse = torch.full((batch, hq), 7.0, dtype=torch.float32, device="cuda")
    ua.decode(q, kp, vp, table, sl, longest, out=out, lse=lse)
    for i in range(0, batch, 8):
        j = min(batch, i + 8)
        o, e = torch.full_like(q[i:j], 7.0), torch.full_like(lse[i:j], 7.0)
        ua.decode(q[i:j].contiguous(), kp, vp, table[i:j].contiguous(), sl[i:j].contiguous(), longest, out=o, lse=e)
        assert torch.equal(o.view(torch.int16), out[i:j].view(torch.int16)), i
        assert torch.equal(e.view(torch.int32), lse[i:j].view(torch.int32)), i
    none = torch.from_numpy(lens == 0).cuda()
    assert bool((out[none] == 7.0).all()) and bool((lse[none] == 7.0).all())
    assert bool(torch.isfinite(out.float()).all()) and bool(torch.isfinite(lse).all())


# up to 4096 items on 256 CUs the list is one of chunks (while chunks x heads to a kv head are at most 400), and more than 64
# of them are several to a lane: 79, 65 (the last lane's are not full) and 129 chunks, 4, 5, 3 and 1 heads; 98 x 17 takes no
# list; longer walks list entries: 12, 70 (two to a lane) and 8 with more kv heads than workgroups
@pytest.mark.parametrize("batch,hkv,group,d,longest", [(5, 8, 4, 128, 20000), (7, 8, 5, 64, 16640), (3, 8, 3, 64, 33024),
                                                       (3, 8, 1, 128, 33024), (4, 4, 17, 128, 25000), (12, 8, 8, 128, 17000),
                                                       (70, 8, 2, 64, 16640), (8, 260, 1, 64, 700)])
def test_listed_walk_over_many_chunks(ua, batch, hkv, group, d, longest):
    """Every entry of a long ragged walk equals itself alone, in a call short enough to take the plain grid."""
    import torch
    page = 64
    hq = hkv * group
    lens = inputs.rng(78, batch).integers(0, longest, size=batch, endpoint=True)
    lens[1], lens[-1] = 0, longest
    table = gu.dev_i32(inputs.rng(79, batch).integers(0, 97, size=(batch, (longest + page - 1) // page)))
    q = inputs.normal_bf16_device((batch, hq, d), 1.0, 80, batch)
    kp, vp = (inputs.normal_bf16_device((97, hkv, page, d), 1.0, 81 + i, batch) for i in range(2))
    out, lse = torch.full_like(q, 7.0), torch.full((batch, hq), 7.0, dtype=torch.float32, device="cuda")
    ua.decode(q, kp, vp, table, gu.dev_i32(lens), longest, out=out, lse=lse)
    for i in range(batch):
        o, e = torch.full_like(q[i:i + 1], 7.0), torch.full_like(lse[i:i + 1], 7.0)
        ua.decode(q[i:i + 1], kp, vp, table[i:i + 1], gu.dev_i32(lens[i:i + 1]), max(int(lens[i]), 1), out=o, lse=e)
        assert torch.equal(o.view(torch.int16), out[i:i + 1].view(torch.int16)), i
        assert torch.equal(e.view(torch.int32), lse[i:i + 1].view(torch.int32)), i


@pytest.mark.parametrize("hq,hkv,d", [(16, 4, 128), (15, 3, 64), (16, 1, 128)])
def test_short_calls_give_the_bits_of_large_ones(ua, hq, hkv, d):
    """A call of few rows walks two chunks at once (128-row tiles): sequences that end at its edges (tiles of 64, rows of
    128, one to five chunks of 256, so a last round of one chunk and of two) alone equal themselves in a pack that takes
    the other kernel."""
    import torch
    lens = [1, 63, 65, 127, 128, 129, 255, 256, 257, 300, 511, 513, 640, 769, 1024, 1025, 1200]
    cu = inputs.cu_seqlens(lens)
    T = int(cu[-1])
    q, k, v = (gu.dev(inputs.normal_bf16((T, h, d), 1.0, 77, hq, d, i)) for i, h in enumerate((hq, hkv, hkv)))
    full, full_lse = ua.prefill(q, k, v, gu.dev_i32(cu), max(lens), return_lse=True)
    for lo, n in zip(cu[:-1], lens):
        rows = slice(int(lo), int(lo) + n)
        out, lse = ua.prefill(q[rows], k[rows], v[rows], gu.dev_i32([0, n]), n, return_lse=True)
        assert torch.equal(out.view(torch.int16), full[rows].view(torch.int16)), n
        assert torch.equal(lse.view(torch.int32), full_lse[rows].view(torch.int32)), n


@pytest.mark.parametrize("n", [40000, 60000])
def test_more_workgroups_than_one_grid(ua, n):
    """Mostly empty sequences, 32 heads and tiles for 1280 keys: 10 and 15 million workgroups of 512 threads in units of four
    tiles (6 and 10 million without), past the 2^32 threads of one grid.  Every row equals the few sequences alone."""
    import torch
    lens = [300, 1280, 1, 129, 640]
    T, h, d = sum(lens), 32, 64
    q, k, v = (inputs.normal_bf16_device((T, h, d), 1.0, 84, i) for i in range(3))
    want, want_lse = ua.prefill(q, k, v, gu.dev_i32(inputs.cu_seqlens(lens)), 1280, return_lse=True)
    spread = np.zeros(n, dtype=np.int64)
    spread[[7, n // 3, n // 2, n - 2000, n - 1]] = lens
    out, lse = torch.full_like(want, 7.0), torch.full_like(want_lse, 7.0)
    ua.prefill(q, k, v, gu.dev_i32(inputs.cu_seqlens(spread)), 1280, out=out, return_lse=True, lse=lse)
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))
    assert torch.equal(lse.view(torch.int32), want_lse.view(torch.int32))
