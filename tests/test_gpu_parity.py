"""GPU parity: the HIP path, called through the C ABI, against the fp64 oracle on the same seeded
bf16 inputs.  Tolerance (the benchmark's stated bar): max |diff| <= 2e-2 and mean |diff| <= 2e-3
over all output elements; the paged KV write must match bit for bit."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import c_oracle, reference

pytestmark = pytest.mark.gpu

MAX_ABS, MEAN_ABS = 2e-2, 2e-3


def _hydra():
    import paper_2505_12658_amd as hydra

    return hydra


def _f64(t):
    return reference.bf16_bits_to_f64(si.bf16_bits(t))


def _run_gpu(w, q, k, v, causal=None, scale=None, **kw):
    hydra = _hydra()
    dev = torch.device("cuda:0")
    cu = torch.from_numpy(w.cu_seqlens).to(dev)
    out = hydra.hydra_attn_varlen_fwd(q.to(dev), k.to(dev), v.to(dev), cu, max(w.max_seqlen, 1), w.causal if causal is None else causal,
                                      w.softmax_scale if scale is None else scale, **kw)
    torch.cuda.synchronize()
    return out


def _check(out, want):
    got = _f64(out)
    assert np.isfinite(got).all()
    diff = np.abs(got - want)
    print(f"max abs {diff.max():.3e}  mean abs {diff.mean():.3e}")
    assert diff.max() <= MAX_ABS
    assert diff.mean() <= MEAN_ABS


@pytest.mark.parametrize("causal", [False, True])
def test_tiny_config_full(causal):
    w = si.tiny(causal)
    q, k, v = si.make_qkv(w)
    out = _run_gpu(w, q, k, v)
    want = reference.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, causal, w.softmax_scale)
    _check(out, want)


CASES = [
    # lengths, Hq, Hkv, d
    ([1], 1, 1, 64),
    ([1, 1, 2, 3], 2, 1, 128),
    ([63, 64, 65, 0, 127, 128, 129], 4, 2, 64),
    ([17, 64, 100, 257], 2, 2, 128),
    ([17, 64, 100, 257], 2, 2, 80),
    ([300, 0, 0, 45, 513], 7, 1, 128),
    ([200, 333], 8, 2, 128),
    ([577, 577], 3, 3, 64),
    ([260, 1027], 2, 2, 80),
    ([1500], 14, 2, 128),
]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"L{'_'.join(map(str, c[0]))}-h{c[1]}k{c[2]}-d{c[3]}")
def test_ragged_cases_full(case, causal):
    lengths, hq, hkv, d = case
    w = si.custom(lengths, hq, hkv, d, causal, seed=len(lengths) * 1000 + hq)
    q, k, v = si.make_qkv(w)
    out = _run_gpu(w, q, k, v)
    want = c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, causal, w.softmax_scale)
    _check(out, want)


def test_scale_zero_gives_means():
    w = si.custom([70, 130], 2, 2, 64, True, seed=5)
    q, k, v = si.make_qkv(w)
    out = _run_gpu(w, q, k, v, scale=0.0)
    want = c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, True, 0.0)
    _check(out, want)


def test_fused_qkv_views_and_preallocated_buffers():
    """q/k/v as strided views into one [N, (Hq + 2 Hkv) * d] projection buffer."""
    hydra = _hydra()
    w = si.custom([90, 201, 64], 4, 2, 128, True, seed=9)
    q, k, v = si.make_qkv(w)
    dev = torch.device("cuda:0")
    fused = torch.cat([q.reshape(w.total_tokens, -1), k.reshape(w.total_tokens, -1), v.reshape(w.total_tokens, -1)], dim=1).to(dev)
    d = w.head_dim
    qv = fused[:, : 4 * d].view(w.total_tokens, 4, d)
    kv = fused[:, 4 * d: 6 * d].view(w.total_tokens, 2, d)
    vv = fused[:, 6 * d:].view(w.total_tokens, 2, d)
    assert not qv.is_contiguous()
    cu = torch.from_numpy(w.cu_seqlens).to(dev)
    out = torch.full((w.total_tokens, 4, d), float("nan"), dtype=torch.bfloat16, device=dev)
    ws = torch.empty(hydra.hydra_attn_workspace_bytes(w.batch, w.total_tokens, w.max_seqlen, 4, 2, d), dtype=torch.uint8, device=dev)
    hydra.hydra_attn_varlen_fwd(qv, kv, vv, cu, w.max_seqlen, True, w.softmax_scale, out=out, workspace=ws)
    torch.cuda.synchronize()
    want = c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, True, w.softmax_scale)
    _check(out, want)


def test_out_of_range_rows_untouched_and_deterministic():
    """Canary rows after the last token stay intact; two runs give identical bits."""
    hydra = _hydra()
    w = si.custom([100, 29], 2, 2, 64, False, seed=3)
    q, k, v = si.make_qkv(w)
    dev = torch.device("cuda:0")
    N = w.total_tokens
    big = torch.full((N + 64, 2, 64), 7.0, dtype=torch.bfloat16, device=dev)
    cu = torch.from_numpy(w.cu_seqlens).to(dev)
    qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
    hydra.hydra_attn_varlen_fwd(qd, kd, vd, cu, w.max_seqlen, False, w.softmax_scale, out=big[:N])
    torch.cuda.synchronize()
    assert (big[N:] == 7.0).all()
    again = hydra.hydra_attn_varlen_fwd(qd, kd, vd, cu, w.max_seqlen, False, w.softmax_scale)
    torch.cuda.synchronize()
    assert torch.equal(again.view(torch.int16), big[:N].view(torch.int16))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d", [64, 80, 128])
def test_large_scores_take_careful_path(d, causal):
    """Keys planted after the first key block whose scores lead the block-0 maximum by far more than
    the fast path's range (row sums beyond 2^40 times the reference term): the workgroup that notices redoes the
    item with the careful routine (if it did not, the affected rows would be inf/NaN or wrong).  Afterwards the
    queue heads in the workspace are all zero again, and a second call on the same workspace gives the same bits."""
    hydra = _hydra()
    w = si.custom([100, 257, 40, 64], 4, 2, d, causal, seed=77)
    q, k, v = si.make_qkv(w)
    cu_host = w.cu_seqlens
    k = k.clone()
    for b, j in ((0, 50), (1, 200), (3, 33)):       # sequence, key position (>= 32: not in key block 0)
        k[cu_host[b] + j] = 64.0                    # score = scale * 64 * sum(q): tens of units either way
    dev = torch.device("cuda:0")
    cu = torch.from_numpy(cu_host).to(dev)
    qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
    ws = hydra.hydra_attn_build_worklist(cu, w.total_tokens, w.max_seqlen, 4, 2, d, causal)
    out = torch.empty_like(qd)
    hydra.hydra_attn_varlen_fwd_prebuilt(qd, kd, vd, cu, w.max_seqlen, causal, w.softmax_scale, out, ws)
    torch.cuda.synchronize()
    want = c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), cu_host, causal, w.softmax_scale)
    # the planted keys really are out of the fast kernel's range for many rows
    z = w.softmax_scale * 64.0 * _f64(q).sum(axis=-1)
    assert (z * 1.4427 > 100).sum() > 50
    _check(out, want)
    # workspace: control block with the queue heads at int32 [32 + 32 x], back at zero after every call
    words = ws.cpu().numpy().view(np.int32)
    n_items = int(words[0])
    assert n_items > 0 and (words[32:32 + 256:32] == 0).all()
    again = torch.empty_like(qd)
    hydra.hydra_attn_varlen_fwd_prebuilt(qd, kd, vd, cu, w.max_seqlen, causal, w.softmax_scale, again, ws)
    torch.cuda.synchronize()
    assert torch.equal(again.view(torch.int16), out.view(torch.int16))


@pytest.mark.parametrize("amp", [2.0, 2.5, 3.0])
@pytest.mark.parametrize("d", [64, 80, 128])
def test_large_activations_stay_accurate_on_fast_path(d, amp):
    """Q and K at 2x, 2.5x and 3x the unit amplitude (scores of standard deviation 4 to 9, peaked softmax): the scale
    is applied to the fp32 scores, not folded into a re-rounded Q, so the error does not grow with the score.  At 2x
    and 2.5x every row stays on the fast path: the kernel hands a work item to the careful one only when a row sum,
    taken relative to the maximum of the row's first key block, goes beyond 2^40 (computed here from the fp64
    scores); at 3x some rows come close to that limit and either kernel may serve."""
    causal = d != 80
    w = si.custom([300, 577, 64, 33], 4, 2, d, causal, seed=int(amp * 100) + d)
    q, k, v = si.make_qkv(w)
    q, k = (q.float() * amp).bfloat16(), (k.float() * amp).bfloat16()
    # (a peaked softmax returns single V values; at unit amplitude some lie in [4, 8), where rounding the OUTPUT to
    # bf16 alone costs up to 1.6e-2.  Halving V keeps that term at 7.8e-3, so that the bound tests the scores.)
    v = (v.float() * 0.5).bfloat16()
    qf, kf = _f64(q), _f64(k)
    worst = 0.0  # largest row sum relative to the reference term (exponent of 2)
    for b in range(w.batch):
        s0, s1 = int(w.cu_seqlens[b]), int(w.cu_seqlens[b + 1])
        for h in range(4):
            z = w.softmax_scale * qf[s0:s1, h] @ kf[s0:s1, h // 2].T
            if causal:
                z = np.where(np.tril(np.ones_like(z, dtype=bool)), z, -np.inf)
            ref = z[:, :32].max(axis=1, keepdims=True)
            worst = max(worst, float(np.log2(np.exp(z - ref).sum(axis=1)).max()))
    print(f"largest row sum 2^{worst:.1f}")
    assert amp > 2.5 or worst < 38
    out = _run_gpu(w, q, k, v)
    _check(out, c_oracle.attn_varlen(qf, kf, _f64(v), w.cu_seqlens, causal, w.softmax_scale))


@pytest.mark.parametrize("d,hq,hkv,causal", [(64, 4, 2, False), (80, 2, 2, False), (128, 7, 1, True)])
def test_shared_variant_matches_plain_call(d, hq, hkv, causal):
    """The variant for two-stream callers (fewer persistent workgroups per compute unit) against the
    oracle, and bit for bit against the plain call, for one workgroup per CU, the kernel's own number and
    a larger request; once more with a paged decode step running on a second stream at the same time."""
    hydra = _hydra()
    w = si.custom([300, 17, 1, 640, 129, 64, 1000], hq, hkv, d, causal, seed=5)
    q, k, v = si.make_qkv(w)
    dev = torch.device("cuda:0")
    cu = torch.from_numpy(w.cu_seqlens).to(dev)
    qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
    ws = hydra.hydra_attn_build_worklist(cu, w.total_tokens, w.max_seqlen, hq, hkv, d, causal)
    plain = torch.empty_like(qd)
    hydra.hydra_attn_varlen_fwd_prebuilt(qd, kd, vd, cu, w.max_seqlen, causal, w.softmax_scale, plain, ws)
    torch.cuda.synchronize()
    _check(plain, c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, causal, w.softmax_scale))
    for per_cu in (1, 2, 3, 100):
        out = torch.full_like(qd, float("nan"))
        hydra.hydra_attn_varlen_fwd_shared(qd, kd, vd, cu, w.max_seqlen, causal, w.softmax_scale, out, ws, per_cu)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), plain.view(torch.int16)), per_cu
    # beside a decode step on another stream
    h = si.HybridBatch("decode", [1] * 64, [1024] * 64, 28, 4, 128, seed=9)
    pq, kc, vc, tables = si.make_paged_inputs(h)
    pq, kc, vc, tables = pq.to(dev), kc.to(dev), vc.to(dev), torch.from_numpy(tables).to(dev)
    cu_q, kv_lens = torch.from_numpy(h.cu_seqlens_q).to(dev), torch.tensor(h.kv_lens, dtype=torch.int32, device=dev)
    alone = hydra.hydra_attn_paged_fwd(pq, kc, vc, tables, cu_q, kv_lens, 1, h.softmax_scale, use_workspace=False)
    torch.cuda.synchronize()
    side = torch.cuda.Stream(device=dev)
    out = torch.full_like(qd, float("nan"))
    beside = torch.empty_like(alone)
    hydra.hydra_attn_varlen_fwd_shared(qd, kd, vd, cu, w.max_seqlen, causal, w.softmax_scale, out, ws, 1)
    with torch.cuda.stream(side):
        hydra.hydra_attn_paged_fwd(pq, kc, vc, tables, cu_q, kv_lens, 1, h.softmax_scale, out=beside, use_workspace=False)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), plain.view(torch.int16))
    assert torch.equal(beside.view(torch.int16), alone.view(torch.int16))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (4, 4, 64)])
def test_worklist_covers_every_tile_once_and_ends_with_cheap_items(hq, hkv, d, causal):
    """The device-built work list read back from the workspace: every group of four wave tiles of every
    (sequence, KV head) appears exactly once, the eight queues partition the list, and the end of every
    queue (as many items as the library says it orders) is in order of non-increasing cost."""
    hydra = _hydra()
    rng = np.random.default_rng(3)
    lengths = rng.integers(1, 900, size=37).tolist() + [0, 2048, 33]
    w = si.custom(lengths, hq, hkv, d, causal, seed=1)
    dev = torch.device("cuda:0")
    cu = torch.from_numpy(w.cu_seqlens).to(dev)
    ws = hydra.hydra_attn_build_worklist(cu, w.total_tokens, w.max_seqlen, hq, hkv, d, causal)
    torch.cuda.synchronize()
    words = ws.cpu().numpy().view(np.int32)
    g = hq // hkv
    expected = set()
    for b, L in enumerate(lengths):
        wave_tiles = -(-L // 32) * g
        for kv in range(hkv):
            for f0 in range(0, wave_tiles, 4):
                expected.add((int(w.cu_seqlens[b]), L, f0, kv))
    n_items, starts = int(words[0]), words[1:10]
    assert n_items == len(expected) and starts[0] == 0 and starts[8] == n_items and (np.diff(starts) >= 0).all()
    rows = (w.batch * hkv + 7) // 8
    items_at = (1152 + 4 * w.batch + 32 * rows + 15) // 16 * 16
    items = words[items_at // 4: items_at // 4 + 4 * n_items].reshape(n_items, 4)
    assert set(map(tuple, items.tolist())) == expected

    def cost(start, L, f0, kv):
        tiles = -(-L // 64)
        if causal:
            f_last = min(f0 + 3, -(-L // 32) * g - 1)
            tiles = min(tiles, -(-((f_last // g + 1) * 32) // 64))
        return tiles

    tail = min(128, (3 << 20) // (4 * 32 * d * 4 // g))
    for x in range(8):
        q = [cost(*it) for it in items[starts[x]:starts[x + 1]].tolist()]
        t = q[-tail:]
        assert all(a >= b for a, b in zip(t, t[1:])), (x, t)


@pytest.mark.parametrize("lengths,hq,hkv,d,causal", [
    ([37], 1, 1, 64, False),                                     # one item
    ([5 + 3 * i for i in range(64)], 16, 16, 64, True),          # as many sequences as lanes, more pairs than one scan takes
    ([100] * 65, 2, 2, 64, False),                               # one sequence too many: the work list
    ([0, 70, 0, 70, 33, 0], 8, 2, 80, True),                     # empty sequences in between
    ([64] * 24, 14, 2, 128, True),                               # equal lengths (not ranked)
    ([33] * 37, 5, 5, 64, False),                                # the same, with one pair in the last row
    ([300] * 11, 7, 1, 128, True),                               # 18 items for every pair, three pairs in the last row
    ([1] * 64, 3, 1, 128, True),
    ([900, 1, 1, 32, 700, 33], 7, 1, 128, True),                 # one KV head: one pair per die and row
])
def test_one_workgroup_per_item(lengths, hq, hkv, d, causal):
    """Batches that run with one workgroup per item: without a work list (the plain call) against the oracle; with one,
    and with persistent workgroups over it, the same bits; keys out of the fast path's range as well."""
    hydra = _hydra()
    w = si.custom(lengths, hq, hkv, d, causal, seed=7 * len(lengths) + hq)
    q, k, v = si.make_qkv(w)
    dev = torch.device("cuda:0")
    cu = torch.from_numpy(w.cu_seqlens).to(dev)
    for planted in (False, True):
        if planted:
            if max(lengths) < 60:
                continue
            k = k.clone()
            for b, L in enumerate(lengths):
                if L > 50:
                    k[w.cu_seqlens[b] + 45] = 64.0  # (see test_large_scores_take_careful_path)
        qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
        out = _run_gpu(w, q, k, v)
        _check(out, c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, causal, w.softmax_scale))
        ws = hydra.hydra_attn_build_worklist(cu, w.total_tokens, w.max_seqlen, hq, hkv, d, causal)
        listed, shared = torch.full_like(qd, float("nan")), torch.full_like(qd, float("nan"))
        hydra.hydra_attn_varlen_fwd_prebuilt(qd, kd, vd, cu, w.max_seqlen, causal, w.softmax_scale, listed, ws)
        hydra.hydra_attn_varlen_fwd_shared(qd, kd, vd, cu, w.max_seqlen, causal, w.softmax_scale, shared, ws, 3)
        torch.cuda.synchronize()
        assert torch.equal(listed.view(torch.int16), out.view(torch.int16)) and torch.equal(shared.view(torch.int16), out.view(torch.int16))


UNITS = 256  # compute units
HALVED = {((65,), 1, 1, 64), ((65,), 3, 1, 128), ((129, 70, 65), 2, 2, 80), ((191, 64, 130, 66), 7, 1, 128), ((1000,), 4, 4, 128), ((2049,), 3, 1, 64),
          ((577,), 16, 16, 64), ((96, 160), 16, 8, 80)}


@pytest.mark.parametrize("lengths,hq,hkv,d,causal", [
    # two teams: every item of two wave tiles has a compute unit
    ([65], 1, 1, 64, False),               # a key tile and one key more: the second team has one key
    ([65], 3, 1, 128, True),               # ... that only the last row sees; wave tiles without keys of the second team
    ([129, 70, 65], 2, 2, 80, True),       # tiles that do not divide by two; odd numbers of key blocks
    ([191, 64, 130, 66], 7, 1, 128, True),
    ([1000], 4, 4, 128, False),
    ([2049], 3, 1, 64, True),
    ([577], 16, 16, 64, False),
    ([96, 160], 16, 8, 80, False),         # KV heads spread evenly over the dies
    # loading waves: every item of four wave tiles has one
    ([577, 577], 16, 16, 64, False),
    ([640], 32, 32, 128, True),
    ([700], 28, 4, 128, True),             # a single request: pairs in turn
    ([1100], 16, 16, 80, False),
    ([1400], 28, 4, 128, True),            # ... of more items than units
    ([65] * 9 + [66], 16, 16, 64, False),  # halves would not all have one
    ([65, 66, 65, 65, 65], 28, 4, 128, True),  # they would, but two key tiles do not pay for them
    # neither: items of four wave tiles that may not all have one
    ([129, 130, 129, 129, 129], 32, 32, 128, True),
])
def test_a_unit_for_every_item(lengths, hq, hkv, d, causal, batch_rules):
    """Batches so small that items have compute units of their own, on both sides of where items are halved and of where they
    have waves that load: against the oracle, the same bits from a work list and for a call that shares the chip, and with keys far
    out of the fast path's range at either end of the sequences.  Loading waves change no bit: the same sequences in a larger batch."""
    hydra = _hydra()
    halved = batch_rules.halved_items(d, len(lengths), sum(lengths), hq, hkv, UNITS)
    loading = batch_rules.loading_waves(int(causal), len(lengths), sum(lengths), max(lengths), hq, hkv, UNITS)
    sizes = (tuple(lengths), hq, hkv, d)
    assert halved == (sizes in HALVED) and loading == (halved or sizes != ((129, 130, 129, 129, 129), 32, 32, 128))
    w = si.custom(lengths, hq, hkv, d, causal, seed=3 * sum(lengths) + hq)
    q, k, v = si.make_qkv(w)
    dev = torch.device("cuda:0")
    cu = torch.from_numpy(w.cu_seqlens).to(dev)

    def bits(qd, kd, vd, cu, longest, how):
        out = torch.full_like(qd, float("nan"))
        if how == "plain":
            hydra.hydra_attn_varlen_fwd(qd, kd, vd, cu, longest, causal, w.softmax_scale, out=out)
        else:
            ws = hydra.hydra_attn_build_worklist(cu, qd.shape[0], longest, hq, hkv, d, causal)
            if how == "listed":
                hydra.hydra_attn_varlen_fwd_prebuilt(qd, kd, vd, cu, longest, causal, w.softmax_scale, out, ws)
            else:
                hydra.hydra_attn_varlen_fwd_shared(qd, kd, vd, cu, longest, causal, w.softmax_scale, out, ws, how)
        torch.cuda.synchronize()
        return out

    for planted in (None, 40, -2):
        if planted is not None:
            k = k.clone()
            for b in range(w.batch):
                k[w.cu_seqlens[b] + (planted if planted > 0 else lengths[b] + planted)] = 64.0  # (see test_large_scores_take_careful_path)
        qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
        out = bits(qd, kd, vd, cu, w.max_seqlen, "plain")
        _check(out, c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, causal, w.softmax_scale))
        for longest, how in ((w.max_seqlen, "listed"), (3 * w.max_seqlen, "plain"), (w.max_seqlen, 1), (w.max_seqlen, 3)):
            assert torch.equal(bits(qd, kd, vd, cu, longest, how).view(torch.int16), out.view(torch.int16)), (planted, how)
        if planted is None and hq * sum(-(-L // 32) for L in lengths) > 512:
            more = [*lengths, 900, 900, 900, 900, 900, 900]
            big = si.custom(more, hq, hkv, d, causal, seed=1)
            qb, kb, vb = (t.to(dev) for t in si.make_qkv(big))
            for t, own in ((qb, qd), (kb, kd), (vb, vd)):
                t[:w.total_tokens] = own
            with_others = bits(qb, kb, vb, torch.from_numpy(big.cu_seqlens).to(dev), big.max_seqlen, "plain")[:w.total_tokens]
            assert torch.equal(with_others.view(torch.int16), out.view(torch.int16))


@pytest.mark.parametrize("batch,hkv", [(2, 1), (4, 1), (2, 2), (1, 2), (1, 4)])
@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("causal", [False, True])
def test_few_pairs_of_one_length(batch, hkv, d, causal, batch_rules):
    """Two or four (sequence, KV head) pairs of one length with more than 32 items each, in halved items, with loading waves and without:
    the oracle, and the same bits from a work list, over outputs of NaN."""
    hydra = _hydra()
    dev = torch.device("cuda:0")
    group, pairs = 16, batch * hkv
    for tiles in (5, 40 // pairs, 80 // pairs):  # of 32 tokens: 40 items of two wave tiles per pair; 160 of four together; 320
        w = si.custom([32 * tiles - 7] * batch, group * hkv, hkv, d, causal, seed=tiles + 10 * pairs + batch)
        sizes = (batch, w.total_tokens, w.max_seqlen, group * hkv, hkv, UNITS)
        assert batch_rules.halved_items(d, batch, w.total_tokens, *sizes[3:]) == (tiles == 5)
        assert batch_rules.loading_waves(int(causal), *sizes) == (tiles <= 40 // pairs or (causal and batch == 1))
        q, k, v = si.make_qkv(w)
        qd, kd, vd, cu = q.to(dev), k.to(dev), v.to(dev), torch.from_numpy(w.cu_seqlens).to(dev)
        out, listed = torch.full_like(qd, float("nan")), torch.full_like(qd, float("nan"))
        hydra.hydra_attn_varlen_fwd(qd, kd, vd, cu, w.max_seqlen, causal, w.softmax_scale, out=out)
        ws = hydra.hydra_attn_build_worklist(cu, w.total_tokens, w.max_seqlen, w.n_q_heads, hkv, d, causal)
        hydra.hydra_attn_varlen_fwd_prebuilt(qd, kd, vd, cu, w.max_seqlen, causal, w.softmax_scale, listed, ws)
        torch.cuda.synchronize()
        assert torch.equal(listed.view(torch.int16), out.view(torch.int16)), tiles
        _check(out, c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, causal, w.softmax_scale))


@pytest.mark.parametrize("lengths,hq,hkv,d", [
    ([1500], 7, 1, 128),             # one pair: seven dies have no queue of their own
    ([900, 40], 14, 2, 64),          # four pairs of two lengths
    ([700, 650, 30], 12, 12, 64),    # pairs in rows and a half
    ([260] * 5, 3, 3, 80),
    ([64] * 9, 1, 1, 64),            # nine pairs of one item: the ninth item is the second of its die
    ([558], 28, 4, 128),             # queues of 32 items on four dies: every die does its own
    ([4096], 1, 1, 64),              # 32 items of one pair, and 33
    ([4097], 1, 1, 64),
    ([20] * 700, 8, 8, 80),          # 5600 items: more rounds than other head dimensions do with a workgroup per item
])
def test_items_are_handed_out_whole_for_any_bound(lengths, hq, hkv, d):
    """Batches whose (sequence, KV head) pairs do not spread evenly over the dies, with an exact, a loose and an understated
    max_seqlen (it limits addressing only): every item is done, with and without a work list, the same bits."""
    hydra = _hydra()
    w = si.custom(lengths, hq, hkv, d, True, seed=len(lengths) + hq)
    q, k, v = si.make_qkv(w)
    dev = torch.device("cuda:0")
    cu = torch.from_numpy(w.cu_seqlens).to(dev)
    qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
    want = c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, True, w.softmax_scale)
    first = None
    for bound in (w.max_seqlen, 20 * w.max_seqlen, 1):
        ws = hydra.hydra_attn_build_worklist(cu, w.total_tokens, bound, hq, hkv, d, True)
        plain, listed = torch.full_like(qd, float("nan")), torch.full_like(qd, float("nan"))
        hydra.hydra_attn_varlen_fwd(qd, kd, vd, cu, bound, True, w.softmax_scale, out=plain)
        hydra.hydra_attn_varlen_fwd_prebuilt(qd, kd, vd, cu, bound, True, w.softmax_scale, listed, ws)
        torch.cuda.synchronize()
        if first is None:
            first = plain
            _check(first, want)
        assert torch.equal(plain.view(torch.int16), first.view(torch.int16)) and torch.equal(listed.view(torch.int16), first.view(torch.int16))


@pytest.mark.parametrize("lengths,hq,hkv,d", [
    ([40] * 3, 2, 1, 64),                 # fewer items than workgroups on every die: nothing is claimed
    ([20] * 800, 1, 1, 64),               # more items than workgroups on some dies
    ([64] * 1024 + [1], 1, 1, 128),       # twice the workgroups everywhere and one over
    ([3000], 8, 1, 128),                  # one queue holds everything, the other dies live off it
])
def test_repeated_calls_on_one_work_list(lengths, hq, hkv, d):
    """Several attention calls on one work list, back to back and with fewer workgroups in between: every call has to
    leave the control block as it found it (heads and counts zero), or the next one would skip items."""
    hydra = _hydra()
    w = si.custom(lengths, hq, hkv, d, True, seed=len(lengths))
    q, k, v = si.make_qkv(w)
    dev = torch.device("cuda:0")
    cu = torch.from_numpy(w.cu_seqlens).to(dev)
    qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
    ws = hydra.hydra_attn_build_worklist(cu, w.total_tokens, w.max_seqlen, hq, hkv, d, True)
    first = None
    for per_cu in (None, 3, 3, 1, None, 2, 3):
        out = torch.full_like(qd, float("nan"))
        if per_cu is None:
            hydra.hydra_attn_varlen_fwd_prebuilt(qd, kd, vd, cu, w.max_seqlen, True, w.softmax_scale, out, ws)
        else:
            hydra.hydra_attn_varlen_fwd_shared(qd, kd, vd, cu, w.max_seqlen, True, w.softmax_scale, out, ws, per_cu)
        torch.cuda.synchronize()
        words = ws.cpu().numpy().view(np.int32)
        assert words[10] == 0 and (words[32:32 + 256:32] == 0).all() and (words[48:48 + 256:32] == 0).all()
        if first is None:
            first = out
            _check(out, c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, True, w.softmax_scale))
        assert torch.equal(out.view(torch.int16), first.view(torch.int16))


@pytest.mark.parametrize("seed", range(48))
def test_random_ragged_batches(seed):
    """Seeded random batches (number of sequences, lengths with zeros and tile-boundary values mixed in, head
    grouping, head_dim, mask, softmax scale off the usual 1/sqrt(d)) against the C oracle, whole output."""
    rng = np.random.default_rng(1000 + seed)
    hq, hkv = [(1, 1), (2, 1), (4, 2), (7, 1), (8, 8), (6, 3)][int(rng.integers(6))]
    d = [64, 80, 128][int(rng.integers(3))]
    causal = bool(rng.integers(2))
    n = int(rng.integers(1, 40))
    special = np.array([0, 1, 31, 32, 33, 63, 64, 65, 127, 128, 129])
    lengths = np.where(rng.random(n) < 0.3, special[rng.integers(len(special), size=n)], rng.integers(0, 600, size=n)).tolist()
    if sum(lengths) == 0:
        lengths[0] = 5
    w = si.custom(lengths, hq, hkv, d, causal, seed=seed)
    q, k, v = si.make_qkv(w)
    scale = w.softmax_scale * float(rng.choice([1.0, 1.0, 0.37, 1.9]))
    out = _run_gpu(w, q, k, v, scale=scale)
    _check(out, c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, causal, scale))


def test_many_short_sequences():
    """More sequences than the work-list builder keeps in LDS (4096): exercises its global-memory path,
    queue rows beyond one wave, and zero-length sequences in between."""
    rng = np.random.default_rng(11)
    lengths = rng.integers(0, 4, size=5000).tolist()
    lengths[17] = 70
    lengths[4999] = 33
    w = si.custom(lengths, 2, 1, 64, True, seed=5)
    q, k, v = si.make_qkv(w)
    out = _run_gpu(w, q, k, v)
    want = c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, True, w.softmax_scale)
    _check(out, want)


@pytest.mark.parametrize("causal", [False, True])
def test_one_long_sequence(causal):
    """A single long sequence (many KV tiles per item, ring wrap-around many times), GQA group 3, d = 80."""
    w = si.custom([4200], 6, 2, 80, causal, seed=9)
    q, k, v = si.make_qkv(w)
    out = _run_gpu(w, q, k, v)
    tokens = np.concatenate([np.arange(0, 40), np.arange(2040, 2120), np.arange(4150, 4200)])
    rows = [(int(t), h) for t in tokens for h in range(6)]
    want = c_oracle.attn_rows(_f64(q), _f64(k), _f64(v), w.cu_seqlens, causal, w.softmax_scale, rows)
    got_all = _f64(out)
    assert np.isfinite(got_all).all()
    got = np.stack([got_all[t, h] for t, h in rows])
    diff = np.abs(got - want)
    print(f"max abs {diff.max():.3e}  mean abs {diff.mean():.3e}")
    assert diff.max() <= MAX_ABS and diff.mean() <= MEAN_ABS


FULL = ["clip_vit_l14_336_encode", "llava15_7b_prefill", "qwen2vl_vit_encode", "qwen2vl_7b_prefill"]


@pytest.mark.parametrize("name", FULL)
def test_full_size_configs_whole_output(name):
    """Benchmark-size workloads in the launch configuration the benchmark times (persistent workgroups, per-die
    queues with stealing, ordered queue tails): EVERY output element against the C oracle."""
    w = si.WORKLOADS[name]()
    q, k, v = si.make_qkv(w)
    out = _run_gpu(w, q, k, v)
    want = c_oracle.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, w.causal, w.softmax_scale)
    print(name, end=": ")
    _check(out, want)
    # every output is a convex combination of V rows: bounded by the global V range
    assert out.float().abs().max() <= v.float().abs().max() * 1.01


def _kv_case(w, strided=False, skip_fraction=0.0, spare=8):
    hydra = _hydra()
    dev = torch.device("cuda:0")
    _, k, v = si.make_qkv(w)
    slots, nb = si.make_slot_mapping(w.lengths, w.block_size, spare_blocks=spare, seed=w.seed, skip_fraction=skip_fraction)
    kc0 = si.make_cache_sentinel(nb, w.block_size, w.n_kv_heads, w.head_dim, seed=1)
    vc0 = si.make_cache_sentinel(nb, w.block_size, w.n_kv_heads, w.head_dim, seed=2)
    want_k, want_v = reference.kv_cache_write(si.bf16_bits(k), si.bf16_bits(v), kc0, vc0, slots, w.block_size)
    kc = torch.from_numpy(kc0.view(np.int16)).view(torch.bfloat16).to(dev)
    vc = torch.from_numpy(vc0.view(np.int16)).view(torch.bfloat16).to(dev)
    if strided:
        fused = torch.cat([k.reshape(w.total_tokens, -1), v.reshape(w.total_tokens, -1)], dim=1).to(dev)
        hd = w.n_kv_heads * w.head_dim
        kd = fused[:, :hd].view(w.total_tokens, w.n_kv_heads, w.head_dim)
        vd = fused[:, hd:].view(w.total_tokens, w.n_kv_heads, w.head_dim)
    else:
        kd, vd = k.to(dev), v.to(dev)
    hydra.hydra_kv_cache_write(kd, vd, kc, vc, torch.from_numpy(slots).to(dev))
    torch.cuda.synchronize()
    assert np.array_equal(si.bf16_bits(kc), want_k)
    assert np.array_equal(si.bf16_bits(vc), want_v)


def test_kv_write_tiny_bit_exact():
    _kv_case(si.tiny(True), spare=34)


def test_kv_write_strided_and_skipped():
    _kv_case(si.tiny(True), strided=True, skip_fraction=0.2)
    _kv_case(si.custom([3, 2], 1, 1, 64, True, kv_cache=True, seed=2))               # a row smaller than one wave
    _kv_case(si.custom([70], 9, 9, 80, True, kv_cache=True, seed=3), strided=True)  # rows of one wave and a part of another
    _kv_case(si.custom([5, 300, 1], 4, 4, 80, True, kv_cache=True, seed=4), strided=True)


@pytest.mark.parametrize("name", ["llava15_7b_prefill", "qwen2vl_7b_prefill"])
def test_kv_write_full_size_bit_exact(name):
    _kv_case(si.WORKLOADS[name]())


# --- paged image cache ---------------------------------------------------------------------------
def _bits_tensor(a, dev):
    return torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).to(dev)


@pytest.mark.parametrize("batch", [si.ImageCacheBatch("small", [5, 0, 12, 1, 700], 64, page_rows=16), si.llava15_image_cache(), si.qwen2vl_image_cache()],
                         ids=lambda b: b.name)
def test_page_cache_write_and_gather_bit_exact(batch):
    """Both directions against the oracle, bit for bit, untouched cache rows and skipped packed rows included; the
    packed side is a row-strided view."""
    hydra = _hydra()
    dev = torch.device("cuda:0")
    rows = si.make_image_rows(batch)
    slots, pages = si.make_slot_mapping(batch.tokens, batch.page_rows, spare_blocks=3, seed=batch.seed, skip_fraction=0.02)
    cache0 = si.make_cache_sentinel(pages, batch.page_rows, 1, batch.hidden, seed=5)[:, :, 0, :].copy()
    wide = torch.zeros((batch.n_rows, batch.hidden + 64), dtype=torch.bfloat16, device=dev)
    view = wide[:, 32 : 32 + batch.hidden]
    view.copy_(rows.to(dev))
    cache = _bits_tensor(cache0, dev)
    slots_d = torch.from_numpy(slots).to(dev)
    hydra.hydra_page_cache_write(view, cache, slots_d)
    torch.cuda.synchronize()
    want_cache = reference.page_cache_write(si.bf16_bits(rows), cache0, slots)
    assert np.array_equal(si.bf16_bits(cache), want_cache)
    out0 = si.make_cache_sentinel(1, batch.n_rows, 1, batch.hidden + 64, seed=6)[0, :, 0, :].copy()
    out = _bits_tensor(out0, dev)
    hydra.hydra_page_cache_gather(cache, slots_d, out[:, 32 : 32 + batch.hidden])
    torch.cuda.synchronize()
    want_out = out0.copy()
    want_out[:, 32 : 32 + batch.hidden] = reference.page_cache_gather(want_cache, slots, out0[:, 32 : 32 + batch.hidden])
    assert np.array_equal(si.bf16_bits(out), want_out)


def test_page_cache_more_rows_than_one_grid_holds():
    """More rows of one piece than the workgroups of one launch cover: the copy goes on in a second launch."""
    hydra = _hydra()
    dev = torch.device("cuda:0")
    n = 4 * (1 << 23) + 5
    rows = torch.arange(n * 4, dtype=torch.int32, device=dev).view(torch.bfloat16).view(n, 8)
    slots = torch.arange(n - 1, -1, -1, dtype=torch.int64, device=dev)
    cache = torch.zeros((n, 8), dtype=torch.bfloat16, device=dev)
    hydra.hydra_page_cache_write(rows, cache, slots)
    assert torch.equal(cache.view(torch.int32), rows.view(torch.int32).flip(0))
    back = torch.zeros_like(rows)
    hydra.hydra_page_cache_gather(cache, slots, back)
    assert torch.equal(back.view(torch.int32), rows.view(torch.int32))


@pytest.mark.parametrize("row", [8, 16, 64, 72, 200, 504, 512, 520, 720, 1024])
def test_rows_of_any_width(row):
    """Row copies of rows that do and do not fill whole waves (64 pieces of 16 bytes), from strided views, with skipped rows:
    the KV scatter and the image cache in both directions, bit for bit, and nothing else written."""
    hydra = _hydra()
    dev = torch.device("cuda:0")
    gen = torch.Generator().manual_seed(row)
    n, num = 1003, 1040
    bits = lambda *shape: torch.randint(-2**15, 2**15, shape, generator=gen, dtype=torch.int16)  # noqa: E731
    wide, cache0, out0 = bits(n, 2 * row + 24), bits(2, num, row), bits(n, row + 8)
    slots = torch.randperm(num, generator=gen)[:n]
    slots[torch.rand(n, generator=gen) < 0.1] = -1
    kept = slots >= 0
    k, v = wide[:, 8: 8 + row], wide[:, 16 + row: 16 + 2 * row]
    want = cache0.clone()
    want[0, slots[kept]], want[1, slots[kept]] = k[kept], v[kept]
    wide_d, caches = wide.to(dev).view(torch.bfloat16), cache0.to(dev).view(torch.bfloat16)
    kd, vd = wide_d[:, 8: 8 + row], wide_d[:, 16 + row: 16 + 2 * row]
    hydra.hydra_kv_cache_write(kd.view(n, 2, row // 2), vd.view(n, 2, row // 2), caches[0].view(num // 16, 16, 2, row // 2),
                               caches[1].view(num // 16, 16, 2, row // 2), slots.to(dev))
    torch.cuda.synchronize()
    assert torch.equal(caches.cpu().view(torch.int16), want)
    pages = cache0[0].to(dev).view(torch.bfloat16)
    hydra.hydra_page_cache_write(kd, pages, slots.to(dev))
    back = out0.to(dev).view(torch.bfloat16)
    hydra.hydra_page_cache_gather(pages, slots.to(dev), back[:, 8:])
    torch.cuda.synchronize()
    assert torch.equal(pages.cpu().view(torch.int16), want[0])
    want_back = out0.clone()
    want_back[kept, 8:] = k[kept]
    assert torch.equal(back.cpu().view(torch.int16), want_back)


def test_numbers_of_the_wrong_kind():
    """Sizes that are not whole numbers are refused where they were never converted, and bounds are the C ABI's 32 bits of them."""
    hydra = _hydra()
    w = si.custom([40, 7], 4, 2, 64, True, seed=2)
    q, k, v = si.make_qkv(w)
    dev = torch.device("cuda:0")
    cu = torch.from_numpy(w.cu_seqlens).to(dev)
    qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
    for sizes in ((4.0, 2, 64), (4, 2.9, 64), (4, 2, "64"), (4, 2, None)):
        with pytest.raises(TypeError):
            hydra.hydra_attn_build_worklist(cu, 47, 40, *sizes, True)
    for bound in (40.5, "40", None):
        with pytest.raises(TypeError):
            hydra.hydra_attn_varlen_fwd(qd, kd, vd, cu, bound, True, w.softmax_scale)
        with pytest.raises(TypeError):
            hydra.hydra_attn_build_worklist(cu, 47, bound, 4, 2, 64, True)
    with pytest.raises(hydra.HydraError, match="invalid argument"):  # (nothing keeps the exception, whose frames hold device tensors)
        hydra.hydra_attn_varlen_fwd(qd, kd, vd, cu, 2**31, True, w.softmax_scale)
    ws = hydra.hydra_attn_build_worklist(cu, np.int64(47), 2**32 + 40, 4, np.int32(2), 64, True)
    want = hydra.hydra_attn_varlen_fwd(qd, kd, vd, cu, np.int64(40), True, w.softmax_scale)
    out = torch.empty_like(qd)
    hydra.hydra_attn_varlen_fwd_prebuilt(qd, kd, vd, cu, 40.0, 1, str(w.softmax_scale), out, ws)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("lengths,hq,hkv,causal", [
    ([256] * 30, 16, 16, False),                                    # 960 items, counted from max_seqlen
    ([256] * 27, 16, 16, False),                                    # 864: just past the least for bidirectional batches
    ([256] * 25, 16, 16, True),                                     # 800: three workgroups
    ([256] * 26, 16, 16, True),                                     # 832: two
    ([384] * 11, 28, 4, False),                                     # 924, too long where nothing is masked
    ([40 + 13 * i % 400 for i in range(50)], 14, 2, True),          # an estimate
    ([256] * 32, 16, 16, True),                                     # 1024
])
def test_four_short_items_per_unit(lengths, hq, hkv, causal):
    """Batches at head_dim 80 on both sides of the rule that keeps a third workgroup off the compute units: every row is there,
    with a list and without, and the bits do not depend on it (a looser bound on the lengths turns the count into an estimate)."""
    hydra = _hydra()
    w = si.Workload("short", lengths, hq, hkv, 80, causal, seed=len(lengths))
    q, k, v = (t.to("cuda:0") for t in si.make_qkv(w))
    cu = torch.from_numpy(w.cu_seqlens).to("cuda:0")
    out = hydra.hydra_attn_varlen_fwd(q, k, v, cu, w.max_seqlen, causal, w.softmax_scale)
    loose = hydra.hydra_attn_varlen_fwd(q, k, v, cu, 3 * w.max_seqlen, causal, w.softmax_scale)
    ws = hydra.hydra_attn_build_worklist(cu, w.total_tokens, w.max_seqlen, hq, hkv, 80, causal)
    listed = torch.empty_like(out)
    hydra.hydra_attn_varlen_fwd_prebuilt(q, k, v, cu, w.max_seqlen, causal, w.softmax_scale, listed, ws)
    torch.cuda.synchronize()
    _check(out, reference.attn_varlen(_f64(q.cpu()), _f64(k.cpu()), _f64(v.cpu()), w.cu_seqlens, causal, w.softmax_scale))
    assert torch.equal(out.view(torch.int16), loose.view(torch.int16)) and torch.equal(out.view(torch.int16), listed.view(torch.int16))


def _work_list(lengths, hq, hkv, d, causal):
    """The work list as csrc/worklist.hpp describes it: entries (first token, length, first wave tile, KV head) of the eight queues."""
    group = hq // hkv
    starts = np.concatenate([[0], np.cumsum(lengths)])
    order = sorted(range(len(lengths)), key=lambda b: (-lengths[b], b))
    queues = [[] for _ in range(8)]
    for r in range(len(lengths) * hkv):
        b, head, row, at = order[r // hkv], r % hkv, r // 8, r % 8
        tiles = -(-lengths[b] // 32) * group
        n = -(-tiles // 4)
        for j in range(n):
            i = n - 1 - j if causal else j
            keys = (min(4 * i + 3, tiles - 1) // group + 1) * 32 if causal else lengths[b]
            queues[7 - at if row & 1 else at].append((-(-min(keys, lengths[b]) // 64), (int(starts[b]), lengths[b], 4 * i, head)))
    tail = min(128, (3 << 20) // (128 * d * 4 // group))
    return [[e for _, e in q[:-tail]] + [e for _, e in sorted(q[-tail:], key=lambda x: -x[0])] for q in queues]


@pytest.mark.parametrize("batch,hq,hkv,d,causal", [(1, 28, 4, 128, True), (3, 4, 4, 64, False), (64, 7, 1, 128, True), (127, 8, 2, 64, True),
                                                   (128, 2, 2, 80, False), (129, 4, 1, 64, True), (512, 2, 1, 64, True), (513, 1, 1, 64, False)])
def test_work_list(batch, hq, hkv, d, causal):
    """Entry for entry, at both ends of every way of ranking the sequences, with equal and empty ones among them."""
    import paper_2505_12658_amd as hydra

    rng = np.random.default_rng(batch)
    lengths = [int(x) for x in rng.integers(0, 700, size=batch)]
    for i in range(0, batch - 1, 3):
        lengths[i] = lengths[i + 1]
    lengths[-1] = max(lengths[-1], 1)
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32, device="cuda:0")
    ws = hydra.hydra_attn_build_worklist(cu, sum(lengths), max(lengths), hq, hkv, d, causal)
    torch.cuda.synchronize()
    words = ws.cpu().numpy()[: ws.numel() // 4 * 4].view(np.int32)
    want = _work_list(lengths, hq, hkv, d, causal)
    assert words[0] == sum(len(q) for q in want)
    assert words[1:10].tolist() == np.concatenate([[0], np.cumsum([len(q) for q in want])]).tolist()
    at = (128 + 8 * 128 + 4 * batch + 32 * -(-batch * hkv // 8) + 15) // 16 * 4
    got = words[at : at + 4 * words[0]].reshape(-1, 4).tolist()
    assert got == [list(e) for q in want for e in q]
