"""GPU parity of attention over the paged KV cache: the HIP kernel, called through the C ABI, against
the fp64 oracle on the same seeded bf16 inputs.  Same tolerance as the packed attention: max |diff| <=
2e-2 and mean |diff| <= 2e-3 over all output elements."""
import ctypes

import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import reference

pytestmark = pytest.mark.gpu

MAX_ABS, MEAN_ABS = 2e-2, 2e-3


def _f64(t):
    return reference.bf16_bits_to_f64(si.bf16_bits(t))


def _run_gpu(h, q, k_cache, v_cache, tables, scale=None, out=None, max_q_len=None, **kw):
    import paper_2505_12658_amd as hydra

    dev = torch.device("cuda:0")
    res = hydra.hydra_attn_paged_fwd(q.to(dev), k_cache.to(dev), v_cache.to(dev), torch.from_numpy(tables).to(dev),
                                     torch.from_numpy(h.cu_seqlens_q).to(dev), torch.tensor(h.kv_lens, dtype=torch.int32, device=dev),
                                     max(h.max_q_len, 1) if max_q_len is None else max_q_len, h.softmax_scale if scale is None else scale,
                                     out=out, **kw)
    torch.cuda.synchronize()
    return res


def _want(h, q, k_cache, v_cache, tables, scale=None):
    return reference.attn_paged(_f64(q), _f64(k_cache), _f64(v_cache), tables, h.cu_seqlens_q, h.kv_lens,
                                h.softmax_scale if scale is None else scale)


def _check(out, want):
    got = _f64(out)
    assert np.isfinite(got).all()
    diff = np.abs(got - want)
    print(f"max abs {diff.max():.3e}  mean abs {diff.mean():.3e}")
    assert diff.max() <= MAX_ABS
    assert diff.mean() <= MEAN_ABS


CASES = [
    # q_lens, kv_lens, Hq, Hkv, d, block_size
    ([1], [1], 1, 1, 64, 16),
    ([1, 1, 1], [1, 16, 17], 2, 1, 128, 16),
    ([1, 0, 3, 5], [7, 4, 3, 11], 4, 2, 64, 4),
    ([17, 64, 100, 257], [17, 64, 100, 257], 2, 2, 64, 16),           # full prefills
    ([17, 64, 100, 257], [40, 64, 1000, 300], 2, 2, 128, 16),         # chunks at the end of longer contexts
    ([63, 64, 65, 1, 129], [63, 128, 65, 700, 129 + 64], 7, 1, 128, 16),
    ([1] * 9 + [200], [33, 64, 65, 127, 128, 129, 511, 512, 513, 333], 28, 4, 128, 16),
    ([5, 130], [260, 1027], 2, 2, 80, 16),
    ([1, 70], [2000, 70], 8, 2, 80, 32),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"q{'_'.join(map(str, c[0]))}-h{c[2]}k{c[3]}-d{c[4]}-b{c[5]}")
def test_ragged_hybrid_batches_full(case):
    q_lens, kv_lens, hq, hkv, d, bs = case
    h = si.HybridBatch("case", q_lens, kv_lens, hq, hkv, d, block_size=bs, seed=len(q_lens) * 100 + hq)
    q, kc, vc, tables = si.make_paged_inputs(h)
    _check(_run_gpu(h, q, kc, vc, tables), _want(h, q, kc, vc, tables))


def test_many_requests_with_scattered_chunks():
    """More requests than the threads of a workgroup, with prefill chunks (ragged lengths, some shorter than a
    wave tile, some invalid or empty requests) scattered among decode steps: the workgroups of the wave-tile
    form locate their request by a scan over all requests, several per thread here."""
    rng = np.random.default_rng(8)
    n = 700
    q_lens = [1] * n
    kv_lens = rng.integers(1, 90, size=n).tolist()
    for pos, ql, extra in ((0, 33, 0), (1, 200, 40), (255, 64, 64), (256, 5, 3), (257, 129, 1), (511, 6, 100), (512, 40, 0), (699, 300, 77), (300, 0, 9)):
        q_lens[pos], kv_lens[pos] = ql, ql + extra
    h = si.HybridBatch("many", q_lens, kv_lens, 8, 2, 64, seed=21)
    q, kc, vc, tables = si.make_paged_inputs(h)
    _check(_run_gpu(h, q, kc, vc, tables), _want(h, q, kc, vc, tables))


@pytest.mark.parametrize("seed", range(24))
def test_random_hybrid_batches(seed):
    """Seeded random hybrid batches: decode steps, short and long chunks, whole prefills, empty requests, in
    random order, random head grouping, head_dim and block size; whole output against the oracle."""
    rng = np.random.default_rng(2000 + seed)
    hq, hkv = [(1, 1), (4, 1), (4, 2), (7, 1), (8, 8), (28, 4)][int(rng.integers(6))]
    d = [64, 80, 128][int(rng.integers(3))]
    bs = [1, 4, 16, 32][int(rng.integers(4))]
    q_lens, kv_lens = [], []
    for _ in range(int(rng.integers(1, 60))):
        kind = int(rng.integers(5))
        ql = [1, int(rng.integers(2, 9)), int(rng.integers(9, 200)), int(rng.integers(1, 150)), 0][kind]
        extra = 0 if kind == 3 else int(rng.integers(0, 400))
        q_lens.append(ql)
        kv_lens.append(ql + extra if ql else int(rng.integers(0, 50)))
    if sum(q_lens) == 0:
        q_lens[0], kv_lens[0] = 3, 10
    h = si.HybridBatch("random", q_lens, kv_lens, hq, hkv, d, block_size=bs, seed=seed)
    q, kc, vc, tables = si.make_paged_inputs(h)
    _check(_run_gpu(h, q, kc, vc, tables), _want(h, q, kc, vc, tables))


PIPELINED_CASES = [
    # q_lens, kv_lens, Hq, Hkv, d, block_size: prefill chunks whose groups of wave tiles run on the packed kernel's
    # pipeline (head_dim 64 or 128, a load instruction's rows inside one cache block); contexts of many key tiles,
    # new tokens that start anywhere inside a key block, last tiles partly filled
    ([300], [1500], 4, 2, 128, 4),
    ([300, 1, 77], [1500, 900, 1077], 7, 1, 128, 8),
    ([512, 512], [2048, 513], 28, 4, 128, 16),
    ([129, 64, 33], [129 + 31, 64 + 1, 33 + 1000], 8, 2, 64, 8),
    ([200, 40], [777, 40], 4, 4, 64, 64),
    ([100], [1000], 2, 1, 128, 256),
    ([65, 300], [65, 301], 2, 2, 64, 4),               # head_dim 64 with blocks of 4 rows: the plain loop
    ([5, 33, 9], [7, 40, 9], 7, 1, 128, 16),           # a handful of new tokens whose grouped heads fill more than one tile of rows
    ([2, 6], [2, 70], 28, 4, 64, 16),                  # one key tile, one key block; a context barely longer than a tile
]


@pytest.mark.parametrize("case", PIPELINED_CASES, ids=lambda c: f"q{'_'.join(map(str, c[0]))}-kv{max(c[1])}-h{c[2]}k{c[3]}-d{c[4]}-b{c[5]}")
def test_chunks_over_long_contexts_and_block_sizes(case):
    q_lens, kv_lens, hq, hkv, d, bs = case
    h = si.HybridBatch("case", q_lens, kv_lens, hq, hkv, d, block_size=bs, seed=7 * len(q_lens) + bs)
    q, kc, vc, tables = si.make_paged_inputs(h)
    _check(_run_gpu(h, q, kc, vc, tables), _want(h, q, kc, vc, tables))


@pytest.mark.parametrize("d", [64, 128])
def test_large_scores_in_a_chunk_are_recomputed(d):
    """Keys planted behind the first key block of a chunk's context whose scores lead the block-0 maximum by far more
    than the pipelined path's range: the workgroup notices (row sums beyond 2^40 times the reference term) and
    computes its group of wave tiles again with the plain loop, which rescales at every tile; if it did not, the
    rows would be inf / NaN or wrong."""
    h = si.HybridBatch("planted", [100, 1, 257], [400, 300, 257], 4, 2, d, seed=77)
    q, kc, vc, tables = si.make_paged_inputs(h)
    kc = kc.clone()
    for b, j in ((0, 50), (0, 350), (2, 200)):       # request, key position (>= 32: not in key block 0)
        kc[tables[b, j // 16], j % 16] = 64.0        # score = scale * 64 * sum(q): tens of units either way
    z = h.softmax_scale * 64.0 * _f64(q).sum(axis=-1)
    assert (z * 1.4427 > 100).sum() > 50
    _check(_run_gpu(h, q, kc, vc, tables), _want(h, q, kc, vc, tables))


def test_full_size_hybrid_batch():
    """The benchmark's hybrid batch (96 decode requests + 4 prefill chunks of 512, 28 / 4 heads of 128), whole output."""
    h = si.qwen2vl_hybrid()
    q, kc, vc, tables = si.make_paged_inputs(h)
    _check(_run_gpu(h, q, kc, vc, tables), _want(h, q, kc, vc, tables))


def test_matches_packed_kernel_after_cache_write():
    """A packed causal prefill, its K/V scattered into the cache with hydra_kv_cache_write, then the paged
    kernel over that cache: both HIP paths against the oracle of the packed attention."""
    import paper_2505_12658_amd as hydra

    dev = torch.device("cuda:0")
    w = si.custom([100, 257, 16], 4, 2, 128, True, seed=5, kv_cache=True)
    q, k, v = si.make_qkv(w)
    slots, num_blocks = si.make_slot_mapping(w.lengths, 16, seed=5)
    kc = torch.zeros((num_blocks, 16, 2, 128), dtype=torch.bfloat16, device=dev)
    vc = torch.zeros_like(kc)
    hydra.hydra_kv_cache_write(k.to(dev), v.to(dev), kc, vc, torch.from_numpy(slots).to(dev))
    width = max((L + 15) // 16 for L in w.lengths)
    tables = np.full((w.batch, width), -1, dtype=np.int32)
    for b in range(w.batch):
        s = int(w.cu_seqlens[b])
        for n in range((w.lengths[b] + 15) // 16):
            tables[b, n] = slots[s + 16 * n] // 16
    h = si.HybridBatch("after_write", w.lengths, w.lengths, 4, 2, 128)
    out = _run_gpu(h, q, kc, vc, tables)
    want = reference.attn_varlen(_f64(q), _f64(k), _f64(v), w.cu_seqlens, True, w.softmax_scale)
    _check(out, want)


def test_strided_q_canaries_and_determinism():
    """q as a view into a wider buffer; rows of `out` that belong to no request keep their contents; two runs agree bit for bit."""
    import paper_2505_12658_amd as hydra

    dev = torch.device("cuda:0")
    h = si.HybridBatch("views", [3, 1, 70], [19, 300, 70], 4, 2, 128, seed=9)
    q, kc, vc, tables = si.make_paged_inputs(h)
    wide = torch.zeros((h.total_q + 5, 4 * 128 + 64), dtype=torch.bfloat16, device=dev)
    qv = wide[: h.total_q, 64:].view(h.total_q, 4, 128)
    qv.copy_(q.to(dev))
    out = torch.full((h.total_q, 4, 128), 7.0, dtype=torch.bfloat16, device=dev)
    args = (kc.to(dev), vc.to(dev), torch.from_numpy(tables).to(dev), torch.from_numpy(h.cu_seqlens_q).to(dev),
            torch.tensor(h.kv_lens, dtype=torch.int32, device=dev), h.max_q_len, h.softmax_scale)
    first = hydra.hydra_attn_paged_fwd(qv, *args, out=out).clone()
    second = hydra.hydra_attn_paged_fwd(qv, *args)
    torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int16), second.view(torch.int16))
    _check(first, _want(h, q, kc, vc, tables))
    # a batch whose cu_seqlens_q stops short of the buffer: the rows after it are not written
    short = si.HybridBatch("short", [3, 1], [19, 300], 4, 2, 128, seed=9)
    out.fill_(7.0)
    hydra.hydra_attn_paged_fwd(qv[:4], args[0], args[1], args[2][:2].contiguous(), torch.from_numpy(short.cu_seqlens_q).to(dev),
                               args[4][:2].contiguous(), 3, h.softmax_scale, out=out[:4])
    torch.cuda.synchronize()
    assert bool((out[4:] == 7.0).all())


def test_scale_zero_and_generous_max_q_len():
    """softmax_scale 0 gives plain means of the visible V rows; max_q_len may exceed the batch's longest request."""
    h = si.HybridBatch("zero", [2, 1], [40, 9], 2, 2, 64, seed=3)
    q, kc, vc, tables = si.make_paged_inputs(h)
    _check(_run_gpu(h, q, kc, vc, tables, scale=0.0, max_q_len=500), _want(h, q, kc, vc, tables, scale=0.0))


SPLIT_CASES = [
    # q_lens, kv_lens, Hq, Hkv, d: few requests with long contexts, so that the packed-rows form splits them over workgroups
    ([1, 1, 1], [5000, 40, 1300], 28, 4, 128),          # shares of the short contexts are empty
    ([4, 1], [3000, 2500], 8, 2, 64),                   # 4 tokens x 4 grouped heads = 16 packed rows, end-aligned mask inside a share
    ([1] * 6, [8192, 100, 4097, 33, 2048, 700], 14, 2, 80),
    ([1, 300], [6000, 900], 28, 4, 128),                # a split decode request next to a chunk in the wave-tile form
    ([1, 1, 1], [4100, 1089, 545], 8, 2, 128),          # contexts one key past a multiple of the share size (544 keys here)
]


@pytest.mark.parametrize("seed", range(12))
def test_random_batches_of_long_contexts(seed):
    """Seeded random small batches of ragged, long contexts with one or a few new tokens each (the packed-rows form,
    contexts cut into shares of equal length over several workgroups and merged), random head grouping, head_dim and
    block size; whole output against the oracle."""
    rng = np.random.default_rng(3000 + seed)
    hq, hkv = [(1, 1), (4, 1), (4, 2), (7, 1), (8, 8), (28, 4), (16, 2)][int(rng.integers(7))]
    d = [64, 80, 128][int(rng.integers(3))]
    bs = [4, 16, 32, 64][int(rng.integers(4))]
    g = hq // hkv
    top = [1500, 3000, 6000][int(rng.integers(3))]
    q_lens, kv_lens = [], []
    for _ in range(int(rng.integers(1, 6))):
        ql = int(rng.integers(1, max(2, 32 // g + 1))) if rng.random() < 0.9 else 0
        kv = int(rng.integers(ql, top)) if rng.random() < 0.7 else top - int(rng.integers(0, 40))
        q_lens.append(ql)
        kv_lens.append(max(kv, ql))
    if sum(q_lens) == 0:
        q_lens[0], kv_lens[0] = 1, top
    h = si.HybridBatch("long", q_lens, kv_lens, hq, hkv, d, block_size=bs, seed=seed)
    q, kc, vc, tables = si.make_paged_inputs(h)
    _check(_run_gpu(h, q, kc, vc, tables), _want(h, q, kc, vc, tables))


@pytest.mark.parametrize("case", SPLIT_CASES, ids=lambda c: f"q{'_'.join(map(str, c[0]))}-kv{max(c[1])}-h{c[2]}k{c[3]}-d{c[4]}")
def test_contexts_split_over_workgroups(case):
    """Small batches of long contexts: with the workspace the library asks for, contexts are split over several
    workgroups and merged by the combine kernel; without it one workgroup walks each context.  Both against the oracle."""
    import paper_2505_12658_amd as hydra

    q_lens, kv_lens, hq, hkv, d = case
    h = si.HybridBatch("split", q_lens, kv_lens, hq, hkv, d, seed=hq + len(q_lens))
    q, kc, vc, tables = si.make_paged_inputs(h)
    assert hydra.hydra_attn_paged_workspace_bytes(h.batch, hkv, d, tables.shape[1], 16) > 0
    want = _want(h, q, kc, vc, tables)
    _check(_run_gpu(h, q, kc, vc, tables), want)
    _check(_run_gpu(h, q, kc, vc, tables, use_workspace=False), want)
    # a workspace too small for the preferred number of shares still gives the right answer (fewer shares)
    small = torch.empty(hydra.hydra_attn_paged_workspace_bytes(h.batch, hkv, d, tables.shape[1], 16) // 3, dtype=torch.uint8, device="cuda:0")
    _check(_run_gpu(h, q, kc, vc, tables, workspace=small), want)


def test_requests_pages_move_to_another_cache():
    """What a migration between instances does to a request on the sending and on the receiving GPU (Section 4.3:
    its cache pages are copied, its page table is rewritten), done here between two caches on one GPU with the
    paged-cache copy calls, one row per cache block: the pages of every request are gathered into one contiguous
    buffer (what would travel), written into other blocks of a second cache, and attention over the second cache with
    the rewritten block table gives the same output bit for bit; blocks of the second cache that received nothing
    keep their contents."""
    import paper_2505_12658_amd as hydra

    dev = torch.device("cuda:0")
    h = si.HybridBatch("move", [1, 70, 1, 3], [300, 200, 77, 19], 8, 2, 128, seed=55)
    q, kc, vc, tables = si.make_paged_inputs(h)
    qd, kcd, vcd = q.to(dev), kc.to(dev), vc.to(dev)
    cu = torch.from_numpy(h.cu_seqlens_q).to(dev)
    kv = torch.tensor(h.kv_lens, dtype=torch.int32, device=dev)
    before = hydra.hydra_attn_paged_fwd(qd, kcd, vcd, torch.from_numpy(tables).to(dev), cu, kv, h.max_q_len, h.softmax_scale)
    # the blocks that hold context, request by request, and their new places in a cache of another size
    bs = 16
    used = [tables[b, : (k + bs - 1) // bs] for b, k in enumerate(h.kv_lens)]
    src = np.concatenate(used).astype(np.int64)
    n_dst = len(src) + 13
    rng = np.random.default_rng(5)
    dst = rng.permutation(n_dst)[: len(src)].astype(np.int64)
    tables2 = np.zeros_like(tables)
    at = 0
    for b, u in enumerate(used):
        tables2[b, : len(u)] = dst[at : at + len(u)]
        at += len(u)
    row = bs * 2 * 128
    sentinel = 1.5
    kc2 = torch.full((n_dst, bs, 2, 128), sentinel, dtype=torch.bfloat16, device=dev)
    vc2 = torch.full((n_dst, bs, 2, 128), -sentinel, dtype=torch.bfloat16, device=dev)
    srcd, dstd = torch.from_numpy(src).to(dev), torch.from_numpy(dst).to(dev)
    for cache, cache2 in ((kcd, kc2), (vcd, vc2)):
        packed = torch.empty((len(src), row), dtype=torch.bfloat16, device=dev)
        hydra.hydra_page_cache_gather(cache.view(cache.shape[0], row), srcd, packed)
        hydra.hydra_page_cache_write(packed, cache2.view(n_dst, row), dstd)
    after = hydra.hydra_attn_paged_fwd(qd, kc2, vc2, torch.from_numpy(tables2).to(dev), cu, kv, h.max_q_len, h.softmax_scale)
    torch.cuda.synchronize()
    assert torch.equal(before.view(torch.int16), after.view(torch.int16))
    _check(after, _want(h, q, kc, vc, tables))
    untouched = np.setdiff1d(np.arange(n_dst), dst)
    assert (kc2[torch.from_numpy(untouched).to(dev)] == sentinel).all() and (vc2[torch.from_numpy(untouched).to(dev)] == -sentinel).all()


DECODE_CASES = [
    # q_lens, kv_lens, Hq, Hkv, d, block_size: requests of at most 16 rows (new tokens x grouped heads)
    ([1] * 9, [1, 15, 16, 17, 31, 32, 33, 127, 129], 4, 4, 128, 16),          # edges of a block of keys, of the waves' turns
    ([1, 2, 1, 0, 2], [700, 2, 64, 5, 33], 14, 2, 64, 16),                    # 14 rows, an empty request
    ([16, 3, 1], [16, 500, 40], 1, 1, 128, 64),                               # 16 rows of one head, causal limits inside the last keys
    ([1, 1], [4129, 9000], 16, 1, 64, 256),                                   # more than 32 steps per wave: a second load of table entries
    ([1, 2, 1], [16, 300, 9], 16, 2, 128, 32),
    ([1] * 258, [9000, 8193] + [5 + 3 * i for i in range(256)], 7, 1, 128, 16),  # more requests than compute units, long table: eight waves
]


@pytest.mark.parametrize("case", DECODE_CASES, ids=lambda c: f"n{len(c[0])}-kv{max(c[1])}-h{c[2]}k{c[3]}-d{c[4]}-b{c[5]}")
def test_decode_form(case):
    """Batches of requests with at most 16 rows each (the decode kernel), unsplit and split, whole output against the oracle."""
    q_lens, kv_lens, hq, hkv, d, bs = case
    h = si.HybridBatch("decode", q_lens, kv_lens, hq, hkv, d, block_size=bs, seed=3 * len(q_lens) + bs)
    q, kc, vc, tables = si.make_paged_inputs(h)
    want = _want(h, q, kc, vc, tables)
    _check(_run_gpu(h, q, kc, vc, tables, use_workspace=False), want)
    _check(_run_gpu(h, q, kc, vc, tables), want)


ORDERED_CASES = [
    # requests, KV heads, d, contexts (a function of the request's number), table keys: more pairs than compute units
    (33, 8, 64, lambda i: 257 + 7 * i, 0),                               # one register of lengths; 264 pairs, the shortest of all orders
    (64, 5, 128, lambda i: (0, 1, 31, 32, 33, 300, 1000)[i % 7], 0),     # many equal ones, and requests without context
    (65, 4, 64, lambda i: 900 - 11 * i, 0),                              # two registers, one lane of the second; longest first already
    (128, 3, 64, lambda i: 1 + 37 * i % 511, 4096),                      # a table wider than any context
    (129, 2, 64, lambda i: 600 if i == 128 else 40 + i % 5, 0),          # four registers; one long context, the last one
    (256, 2, 64, lambda i: 1 + 131 * i % 777, 0),                        # 512 pairs, eight waves
    (256, 2, 64, lambda i: 1 + 131 * i % 511, 4096),                     # eight waves of which four leave
    (116, 4, 128, lambda i: 40 * (i % 23), 0),                           # 464 pairs
    (70, 16, 64, lambda i: 20 + 53 * i % 500, 0),                        # 1120 pairs: more than the chip holds at once
    (80, 4, 64, lambda i: 1000 + i % 100, 0),                            # contexts within a quarter of each other
    (257, 1, 64, lambda i: 1 + 131 * i % 777, 0),                        # one request too many
]


@pytest.mark.parametrize("case", ORDERED_CASES, ids=lambda c: f"n{c[0]}-k{c[1]}-d{c[2]}-t{c[4]}-{c[3](1)}")
def test_pairs_in_the_order_of_their_contexts(case):
    """Decode batches of more (request, KV head) pairs than compute units, whose workgroups find their pair by the rank of its
    context: every row is there, against the oracle, and (where both launches deal the keys out to four streams) with the bits of
    the same requests in batches too small to be ordered."""
    n, hkv, d, context, table_keys = case
    kv_lens = [context(i) for i in range(n)]
    h = si.HybridBatch("ordered", [1 if k else 0 for k in kv_lens], kv_lens, 2 * hkv, hkv, d, block_size=16, seed=n + hkv)
    q, kc, vc, tables = si.make_paged_inputs(h)
    if table_keys:
        wide = np.full((n, table_keys // 16), -1, dtype=np.int32)
        wide[:, : tables.shape[1]] = tables
        tables = wide
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
    _run_gpu(h, q, kc, vc, tables, out=out)
    _check(out, _want(h, q, kc, vc, tables))
    keys = 16 * tables.shape[1]
    if (256 < n * hkv <= 512 and keys >= 768 and not (keys >= 4096 and max(kv_lens) < 512)) or n == 257:
        return  # eight streams: test_bits_of_a_decode_batch_whatever_its_order
    size = 256 // hkv
    for at in range(0, n, size):
        part = si.HybridBatch("part", h.q_lens[at:at + size], kv_lens[at:at + size], 2 * hkv, hkv, d, block_size=16)
        rows = slice(int(h.cu_seqlens_q[at]), int(h.cu_seqlens_q[at]) + part.total_q)
        alone = _run_gpu(part, q[rows], kc, vc, np.ascontiguousarray(tables[at:at + size]), use_workspace=False)
        assert torch.equal(alone.view(torch.int16), out[rows].view(torch.int16))


STREAM_CASES = [
    # requests, KV heads, d, contexts, table keys: 257 to 512 pairs, at most 256 requests
    (65, 4, 128, lambda i: 900 - 11 * i, 0),                                  # four waves with two streams each
    (86, 3, 64, lambda i: (0, 1, 31, 33, 128, 129, 256, 257, 1000)[i % 9], 0),  # streams of no, one and many blocks
    (80, 4, 128, lambda i: 1000 + i % 100, 0),                                # near enough to each other to stay in batch order
    (33, 14, 64, lambda i: 700 + 97 * i % 800, 0),                            # 462 pairs
    (116, 4, 64, lambda i: 40 + 50 * (i % 23), 0),                            # 464 pairs: eight waves
    (256, 2, 64, lambda i: 1 + 131 * i % 777, 0),                             # 512 pairs
    (128, 3, 128, lambda i: 1 + 37 * i % 511, 1024),                          # a table wider than any context
    (128, 3, 64, lambda i: 1 + 37 * i % 511, 4096),                           # and one so wide that short contexts have four streams
    (128, 3, 64, lambda i: 512 if i == 77 else 1 + 37 * i % 511, 4096),       # one context too long for that
]


@pytest.mark.parametrize("case", STREAM_CASES, ids=lambda c: f"n{c[0]}-k{c[1]}-d{c[2]}-t{c[4]}-{c[3](1)}-{c[3](77)}")
def test_bits_of_a_decode_batch_whatever_its_order(case):
    """How the keys of a context are dealt out to partial sums is settled by the number of pairs and the lengths, not by the
    order the pairs are taken in: the KV heads of a batch one after the other, as that many requests of one KV head (too many
    to be ordered), give the same bits."""
    n, hkv, d, context, table_keys = case
    kv_lens = [context(i) for i in range(n)]
    q_lens = [1 if k else 0 for k in kv_lens]
    h = si.HybridBatch("heads", q_lens, kv_lens, 2 * hkv, hkv, d, block_size=16, seed=n + hkv)
    q, kc, vc, tables = si.make_paged_inputs(h)
    if table_keys:
        wide = np.full((n, table_keys // 16), -1, dtype=np.int32)
        wide[:, : tables.shape[1]] = tables
        tables = wide
    out = _run_gpu(h, q, kc, vc, tables)
    _check(out, _want(h, q, kc, vc, tables))
    blocks = kc.shape[0]
    one = si.HybridBatch("requests", q_lens * hkv, kv_lens * hkv, 2, 1, d, block_size=16)

    def by_head(t, heads):  # [.., heads of every KV head, d] -> one KV head after the other along the first dimension
        return torch.cat([t[..., g * heads:(g + 1) * heads, :] for g in range(hkv)]).contiguous()

    tables_one = np.concatenate([np.where(tables >= 0, tables + g * blocks, -1) for g in range(hkv)]).astype(np.int32)
    got = _run_gpu(one, by_head(q, 2), by_head(kc, 1), by_head(vc, 1), tables_one)
    assert torch.equal(by_head(out, 2).view(torch.int16), got.view(torch.int16))


def _mix(steps, chunks, every=None):
    """q_lens, kv_lens of decode steps (their contexts) and chunks ((new tokens, context)), a chunk after every `every` steps."""
    q, k, at = [], [], 0
    every = every or max(1, len(steps) // max(1, len(chunks)))
    for i, n in enumerate(steps):
        q.append(1 if n else 0)
        k.append(n)
        if (i + 1) % every == 0 and at < len(chunks):
            q.append(chunks[at][0])
            k.append(chunks[at][1])
            at += 1
    for c, n in chunks[at:]:
        q.append(c)
        k.append(n)
    return q, k


MIXED_CASES = [
    # (q_lens, kv_lens), Hq, Hkv, d: decode steps and chunks over the two layers of the chip
    (_mix([], [(300, 900), (70, 70), (33, 1100)]), 4, 2, 64),                                       # chains only, some long
    (_mix([50], [(40, 40)]), 2, 1, 64),                                                             # one of each, neither long
    (_mix([10 + 9 * i for i in range(61)], [(64, 700), (96, 600), (40, 513)]), 4, 4, 64),           # 64 requests; steps short of a layer
    (_mix([10 + 9 * i for i in range(62)], [(64, 700), (96, 512), (40, 513)]), 8, 8, 64),           # 65; steps past one layer, long chains
    (_mix([5 + 7 * i % 400 for i in range(127)], [(200, 1100)]), 8, 4, 128),                        # 508 steps, chains longer than any of them
    (_mix([300 + 7 * i % 900 for i in range(140)], [(200, 600), (64, 64)]), 8, 4, 64),              # 560 steps, steps longer than the chains
    (_mix([(0, 33, 400)[i % 3] for i in range(200)], [(40, 40 + 20 * i) for i in range(56)]), 2, 1, 64),   # 256 requests, 56 chunks, many equal
    (_mix([1 + 5 * i % 99 for i in range(250)], [(33, 700), (64, 64)] * 3 + [(50, 60)]), 4, 2, 64),  # 257 requests: one too many
    (_mix([2100, 1700, 900], [(60, 60)]), 4, 1, 128),                                               # split contexts beside a chunk
    (_mix([700] * 9, [(100, 700)] * 9), 4, 2, 80),                                                  # the other forms, all of one length
]


@pytest.mark.parametrize("case", MIXED_CASES, ids=lambda c: f"n{len(c[0][0])}-q{sum(c[0][0])}-kv{max(c[0][1])}-h{c[1]}k{c[2]}-d{c[3]}")
def test_steps_and_chains_over_the_chip(case):
    """Hybrid batches whose workgroups find their step or chain from the lengths of the whole batch: every row is there."""
    (q_lens, kv_lens), hq, hkv, d = case
    h = si.HybridBatch("mix", q_lens, kv_lens, hq, hkv, d, block_size=16, seed=len(q_lens))
    q, kc, vc, tables = si.make_paged_inputs(h)
    want = _want(h, q, kc, vc, tables)
    for kw in ({}, {"use_workspace": False}):
        out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
        _check(_run_gpu(h, q, kc, vc, tables, out=out, **kw), want)


CHUNK_CASES = [
    # (q_lens, kv_lens), Hq, Hkv, d: chains whose chunk is found one by one, and by the search over their key tiles
    (_mix([20, 900], [(40, 64), (64, 65), (33, 700), (70, 129)]), 4, 2, 64),                         # four chunks and five
    (_mix([20, 900], [(40, 64), (64, 65), (33, 700), (70, 129), (50, 50)]), 4, 2, 64),
    (_mix([], [(33 + i, 64) for i in range(32)] * 2), 2, 1, 64),                                     # 64 chunks of one key tile
    (_mix([5] * 9, [(33 + i % 20, 64 * (1 + i % 4)) if i % 4 else (40 + i, 200 + i) for i in range(56)]), 7, 1, 128),  # 65 requests; whole tiles
    (_mix([300] * 3, [(33 + 7 * i % 40, 100 + 97 * i % 900) for i in range(253)]), 2, 1, 64),       # 256 requests, chunks over every register
    (_mix([1 + i for i in range(200)], [(64, 1024)] * 3 + [(100, 1025)] * 3), 8, 2, 64),             # the largest number of tiles a power of two, and one more
    (_mix([], [(200, 200 + 50 * (i % 3)) for i in range(70)]), 6, 3, 80),                            # groups of one chunk over several places
]


@pytest.mark.parametrize("case", CHUNK_CASES, ids=lambda c: f"n{len(c[0][0])}-q{sum(c[0][0])}-kv{max(c[0][1])}-h{c[1]}k{c[2]}-d{c[3]}")
def test_chains_of_many_chunks(case):
    """Batches of few and of many chunks: every row of every chunk is there."""
    (q_lens, kv_lens), hq, hkv, d = case
    h = si.HybridBatch("chunks", q_lens, kv_lens, hq, hkv, d, block_size=16, seed=len(q_lens) + 1)
    q, kc, vc, tables = si.make_paged_inputs(h)
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
    _check(_run_gpu(h, q, kc, vc, tables, out=out), _want(h, q, kc, vc, tables))


@pytest.mark.parametrize("group", [1, 2, 3, 5, 7, 16, 31, 32, 33])
def test_chunks_of_the_fewest_rows(group):
    """Chunks that are just too long for the packed-rows form, nothing else in the batch: as many workgroups as the host's bound
    from the number of new tokens allows."""
    q = 32 // group + 1
    for n in (1, 5, 70, 300):
        h = si.HybridBatch("fewest", [q] * n, [q + i % 40 for i in range(n)], group, 1, 64, block_size=16, seed=group)
        qs, kc, vc, tables = si.make_paged_inputs(h)
        out = torch.full(qs.shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
        _check(_run_gpu(h, qs, kc, vc, tables, out=out), _want(h, qs, kc, vc, tables))


ORDER_CASES = [
    # (q_lens, kv_lens), Hq, Hkv, d, table keys: batches that keep the order of their requests, and such that do not
    (_mix([30 + i for i in range(60)], [(40, 100), (9, 50)]), 8, 8, 64, 0),            # a narrow table says it
    (_mix([30 + i for i in range(60)], [(40, 100), (9, 50)]), 8, 8, 64, 4096),         # one register: a wide table does not
    (_mix([(0, 17, 300)[i % 3] for i in range(96)], [(40, 1024 + 64), (64, 64)]), 4, 2, 128, 4096),   # two registers, ordered by one chunk
    (_mix([(0, 17, 300)[i % 3] for i in range(96)], [(40, 440), (64, 64)]), 4, 2, 128, 4096),         # the limit, and one key more
    (_mix([(0, 17, 300)[i % 3] for i in range(96)], [(40, 441), (64, 64)]), 4, 2, 128, 4096),
    (_mix([1 + 3 * i % 500 for i in range(200)], [(64, 1024), (33, 40)] * 4), 8, 4, 128, 0),          # four registers: 832 pairs, limit 1109
    (_mix([1 + 3 * i % 500 for i in range(200)], [(64, 1110), (33, 40)] * 4), 8, 4, 128, 0),
    (_mix([1 + 3 * i % 500 for i in range(200)], [(64, 1024), (33, 40)] * 4), 8, 4, 128, 4096),
    (_mix([1900, 40, 700, 2500], [(40, 300), (9, 11)]), 2, 1, 64, 0),                   # split contexts
    (_mix([600, 40, 700, 30] * 20, [(40, 300)]), 8, 1, 64, 0),                          # 81 pairs, contexts cut in batch order
    # no chunks: 280 pairs on both sides of 140 keys, 240 pairs, 1040 pairs, and few pairs whose contexts are cut
    (([5] * 70, [5 + 2 * i % 136 for i in range(69)] + [140]), 16, 4, 128, 0),
    (([5] * 70, [5 + 2 * i % 136 for i in range(69)] + [141]), 16, 4, 128, 0),
    (([5] * 70, [5 + 2 * i % 136 for i in range(69)] + [141]), 16, 4, 128, 4096),
    (([5] * 60, [5 + 7 * i % 400 for i in range(60)]), 16, 4, 128, 0),
    (([2] * 130, [2 + 7 * i % 500 for i in range(130)]), 16, 8, 80, 0),
    (([1] * 130, [7 * i % 90 + 1 for i in range(129)] + [700]), 16, 8, 80, 4096),
    (([3, 0, 3, 3], [2000, 50, 3, 900]), 7, 1, 128, 0),
]


@pytest.mark.parametrize("case", ORDER_CASES, ids=lambda c: f"n{len(c[0][0])}-kv{max(c[0][1])}-h{c[1]}k{c[2]}-d{c[3]}-t{c[4]}")
def test_hybrid_batches_in_either_order(case):
    """Hybrid batches on both sides of the rule that keeps the order of the requests: every row is there."""
    (q_lens, kv_lens), hq, hkv, d, table_keys = case
    h = si.HybridBatch("order", q_lens, kv_lens, hq, hkv, d, block_size=16, seed=len(q_lens) + 2)
    q, kc, vc, tables = si.make_paged_inputs(h)
    want = _want(h, q, kc, vc, tables)
    if table_keys:
        wide = np.full((len(q_lens), table_keys // 16), -1, dtype=np.int32)
        wide[:, : tables.shape[1]] = tables
        tables = wide
    for kw in ({}, {"use_workspace": False}):
        out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
        _check(_run_gpu(h, q, kc, vc, tables, out=out, **kw), want)


def test_split_context_with_an_infinite_value():
    """A context of fewer shares than the launch has, whose last key holds an infinite V component: infinite in the output
    column it belongs to (the shares that do not exist must not turn it into NaN), everything else against the oracle."""
    h = si.HybridBatch("inf", [1, 1], [2000, 700], 4, 1, 128, block_size=16, seed=11)
    q, kc, vc, tables = si.make_paged_inputs(h)
    want = _want(h, q, kc, vc, tables)
    vc = vc.clone()
    vc[int(tables[1][699 // 16]), 699 % 16, 0, 3] = float("inf")
    out = _run_gpu(h, q, kc, vc, tables).cpu()
    assert (out[1, :, 3] == float("inf")).all()
    out[1, :, 3] = torch.from_numpy(want[1, :, 3])
    _check(out, want)


def test_fewer_chunk_workgroups_than_free_slots():
    """A workspace that holds 3 of the 5 shares asked for: 270 decode workgroups leave more of the chip's second layer free
    than the one small chunk has workgroups, and every share still has to find a workgroup."""
    import paper_2505_12658_amd as hydra

    h = si.HybridBatch("few", [33] + [1] * 89, [1500] * 90, 1, 1, 64, block_size=16, seed=5)
    q, kc, vc, tables = si.make_paged_inputs(h)
    record = (2 * 32 + 32 * 64) * 4
    assert hydra.hydra_attn_paged_workspace_bytes(90, 1, 64, tables.shape[1], 16) == 5 * 90 * record
    ws = torch.full((3 * 90 * record // 4,), float("nan"), device="cuda:0")
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
    _check(_run_gpu(h, q, kc, vc, tables, out=out, workspace=ws), _want(h, q, kc, vc, tables))


@pytest.mark.parametrize("d", [64, 80, 128])
def test_large_scale_with_masked_blocks(d):
    """Softmax scale 1: rows whose first keys in a wave are all masked (the early tokens of a short chunk see none of the
    last 8 keys, which one wave has alone) keep weight 0 for them."""
    h = si.HybridBatch("scale", [16, 3], [40, 33], 1, 1, d, block_size=16, seed=d)
    q, kc, vc, tables = si.make_paged_inputs(h)
    q = q * 0.125
    _check(_run_gpu(h, q, kc, vc, tables, scale=1.0), _want(h, q, kc, vc, tables, scale=1.0))


@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("rows", [8, 9, 16, 17, 31, 32])
def test_merge_of_requests_with_many_rows(d, rows):
    """Split contexts of requests with up to 32 rows: the merge's threads, 4 columns of one row each, fill one to four workgroups
    per (request, KV head)."""
    h = si.HybridBatch("rows", [rows, 1, rows - 1], [2500, 2100, 1400], 2, 2, d, block_size=16, seed=rows)
    q, kc, vc, tables = si.make_paged_inputs(h)
    _check(_run_gpu(h, q, kc, vc, tables), _want(h, q, kc, vc, tables))


@pytest.mark.parametrize("q_lens,kv_lens,hq,hkv,d,most", [
    ([1], [8192], 7, 1, 128, 64),                                          # 64 shares: eight for each of eight waves
    ([1] * 4, [8192, 128 * 33 + 1, 4096, 4097], 16, 1, 64, 64),            # 64, 34, 32 and 33 shares
    ([1] * 4, [4096, 128 * 17 + 1, 2048, 128], 7, 1, 128, 64),             # 32, 18, 16 and one
    ([1] * 3, [2177, 1100, 1025], 8, 1, 64, 64),                           # a table for 18 shares: 18, 9 and 9
    ([1] * 5, [1000, 513, 512, 257, 256], 28, 2, 128, 51),                 # a table for 8: 8, 5, 4, 3 and 2
    ([1] * 3, [700, 257, 129], 4, 2, 64, 64),                              # a table for 6: 6, 3 and 2
    ([1] * 16, [1500, 700, 300, 40] * 4, 8, 4, 64, 8),                     # 4 shares of 256 units, room for 8
    ([1] * 16, [1500, 700, 300, 40] * 4, 8, 8, 64, 4),                     # 2
    ([1] * 2, [250, 130], 4, 4, 128, 0),                                   # too short to be cut
    ([8, 3, 0, 1], [6000, 4100, 900, 2200], 4, 1, 128, 64),                # 32 rows, in the other form of the first kernel
    ([4, 1], [3000, 5000], 8, 1, 80, 64),
    ([1] * 20, [4096] * 10 + [1500] * 10, 4, 1, 128, 25),                  # 12 shares of 256 units, room for 25
])
def test_number_of_shares(q_lens, kv_lens, hq, hkv, d, most):
    """Contexts of few requests in up to 64 shares, around the numbers where the merge takes another way, over a workspace of NaN; and
    with an infinity in the last key's V, which one share has alone."""
    import paper_2505_12658_amd as hydra

    h = si.HybridBatch("shares", q_lens, kv_lens, hq, hkv, d, block_size=16, seed=len(q_lens))
    q, kc, vc, tables = si.make_paged_inputs(h)
    need = hydra.hydra_attn_paged_workspace_bytes(h.batch, hkv, d, tables.shape[1], 16)
    assert need == most * h.batch * hkv * (2 * 32 + 32 * d) * 4
    want = _want(h, q, kc, vc, tables)
    for records in sorted({most, most // 2, min(most, 16)}):
        ws = torch.full((max(records * h.batch * hkv * (2 * 32 + 32 * d), 4),), float("nan"), device="cuda:0")
        out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
        _check(_run_gpu(h, q, kc, vc, tables, out=out, workspace=ws), want)
    if q_lens[0] > 1:  # (its other tokens multiply the infinity by 0)
        return
    last = kv_lens[0] - 1
    vc = vc.clone()
    vc[int(tables[0][last // 16]), last % 16, 0, 5] = float("inf")
    got = _run_gpu(h, q, kc, vc, tables).cpu()
    assert (got[0, :hq // hkv, 5] == float("inf")).all()
    got[0, :hq // hkv, 5] = torch.from_numpy(want[0, :hq // hkv, 5])
    _check(got, want)


def test_more_than_a_million_pairs():
    """20 requests of one key with 60 000 heads: (request, KV head) pairs on both sides of 2^20, where their division takes another way.
    Each output row is the request's V row."""
    import paper_2505_12658_amd as hydra

    dev, batch, heads, d = torch.device("cuda:0"), 20, 60000, 64
    gen = torch.Generator(device=dev).manual_seed(3)
    table = torch.full((batch, 17), -1, dtype=torch.int32, device=dev)
    table[:, 0] = torch.randperm(batch, generator=gen, device=dev).to(torch.int32)
    q = torch.ones((batch, heads, d), dtype=torch.bfloat16, device=dev)
    kc = torch.ones((batch, 16, heads, d), dtype=torch.bfloat16, device=dev)
    vc = torch.full_like(kc, float("nan"))
    rows = torch.randn((batch, heads, d), generator=gen, device=dev).to(torch.bfloat16)
    vc[table[:, 0].long(), 0] = rows
    out = hydra.hydra_attn_paged_fwd(q, kc, vc, table, torch.arange(batch + 1, dtype=torch.int32, device=dev),
                                     torch.ones(batch, dtype=torch.int32, device=dev), 1, 0.125)
    assert torch.equal(out.view(torch.int16), rows.view(torch.int16))


@pytest.mark.parametrize("kv_lens,chunk,split", [
    ([1000, 120, 430], 128, False),     # the chunk's chain of key tiles is what the kernel waits for
    ([2500, 700, 90], 60, True),        # contexts far longer than the chunk
    ([8200] * 16, 33, True),            # 272 shares, more than compute units, and 24 of the 26 chunk workgroups trade places with them
    ([2000] * 170, 40, False),          # more than half of the compute units have a decode step
])
def test_shares_beside_chunks(kv_lens, chunk, split):
    """Decode steps and one prefill chunk: contexts are split (partial results in the workspace) only where that pays beside a chunk."""
    import paper_2505_12658_amd as hydra

    h = si.HybridBatch("beside", [1] * len(kv_lens) + [chunk], list(kv_lens) + [chunk + 600], 2, 1, 64, block_size=16, seed=chunk)
    q, kc, vc, tables = si.make_paged_inputs(h)
    need = hydra.hydra_attn_paged_workspace_bytes(h.batch, 1, 64, tables.shape[1], 16)
    ws = torch.full((max(need, 16) // 4,), float("nan"), device="cuda:0")
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
    _check(_run_gpu(h, q, kc, vc, tables, out=out, workspace=ws), _want(h, q, kc, vc, tables))
    assert bool(torch.isfinite(ws).any()) == split


@pytest.mark.parametrize("q_lens,kv_lens,hq,hkv,d,bs", [
    ([1, 1, 1, 1], [1200, 300, 655, 1480], 28, 4, 128, 16),        # the decode kernel
    ([1] * 8, [4096, 200, 3000, 17, 1, 33, 2222, 640], 8, 2, 64, 32),
    ([4, 2, 1], [2500, 900, 1400], 8, 1, 80, 16),                  # up to 32 rows, blocks and head_dim of the other form
    ([1] * 70, [2000 - 20 * i for i in range(70)], 4, 1, 128, 16), # more lengths than lanes
    ([1, 1, 40], [3000, 2100, 200], 14, 2, 128, 16),               # beside a chunk
])
def test_shares_follow_the_contexts_not_the_table(q_lens, kv_lens, hq, hkv, d, bs):
    """A block table 32 768 keys wide over contexts far shorter: split as under a table cut to the longest context; the same
    bits without a chunk in the batch (beside one the number of shares follows the table, their least length does not)."""
    import paper_2505_12658_amd as hydra

    h = si.HybridBatch("wide", q_lens, kv_lens, hq, hkv, d, block_size=bs, seed=max(kv_lens))
    q, kc, vc, tables = si.make_paged_inputs(h)
    wide = np.full((h.batch, 32768 // bs), -1, dtype=np.int32)
    wide[:, : tables.shape[1]] = tables
    outs = []
    for t in (tables, wide):
        need = hydra.hydra_attn_paged_workspace_bytes(h.batch, hkv, d, t.shape[1], bs)
        ws = torch.full((max(need, 16) // 4,), float("nan"), device="cuda:0")
        outs.append(_run_gpu(h, q, kc, vc, t, workspace=ws))
        assert bool(torch.isfinite(ws).any())
        _check(outs[-1], _want(h, q, kc, vc, tables))
    if max(q_lens) < 32:
        assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))


WIDE_CASES = [
    # q_lens, kv_lens, Hq, Hkv, d, block_size
    ([130], [130], 28, 4, 128, 16),                                              # chains alone
    ([1, 130, 1, 200, 1], [60, 130, 1, 500, 33], 28, 4, 128, 16),                # a unit for everything
    ([200, 100, 50, 25, 12, 6], [200, 300, 50, 225, 12, 6], 28, 4, 128, 16),     # chunks of unequal lengths
    ([1] * 70 + [150, 150], [8 * i + 1 for i in range(70)] + [150, 300], 28, 4, 128, 16),     # two decode steps to a workgroup, not for all
    ([1] * 101 + [250], [4 * i + 3 for i in range(101)] + [300], 5, 5, 64, 16),               # ... for all but one, an odd number
    ([1] * 90 + [300, 101], [3 * i + 1 for i in range(90)] + [300, 301], 14, 2, 128, 16),     # ... in a grid for all that there can be
    ([3, 1, 90, 4, 2], [100, 40, 190, 4, 77], 8, 1, 128, 16),                    # 24 and 32 rows beside 8
    ([1, 2, 100, 1], [50, 200, 100, 9], 8, 2, 64, 8),                            # blocks that the decode form does not take
    ([1, 70, 1], [30, 140, 190], 4, 2, 128, 4),
    ([0, 1, 100, 35, 0, 1, 40], [4, 220, 140, 35, 0, 90, 300], 7, 1, 128, 16),   # requests without new tokens
    ([1] * 127 + [300], [64] * 127 + [300], 4, 2, 64, 16),                       # two registers of lengths
    # chunks that are not the whole ones that their tokens look like: more chains than the grid has places
    ([101] + [5] * 50, [101] + [5 + 3 * i for i in range(50)], 28, 4, 128, 16),
    ([1] * 20 + [101] + [5] * 50, [60] * 20 + [101] + [5 + 3 * i for i in range(50)], 28, 4, 128, 16),
    ([1, 101, 1] + [5] * 50, [200, 101, 60] + [5 + 3 * i for i in range(50)], 28, 4, 64, 16),
]
FOUR_WAVE_CASES = [
    # of the same kind, but with more chains than pay, longer contexts, or chunks that the host cannot count on
    ([1] * 101 + [250], [6 * i + 3 for i in range(101)] + [700], 5, 5, 64, 16),
    ([64] + [33] * 20, [64] + [33 + 20 * i for i in range(20)], 64, 4, 64, 16),
    ([64] + [33] * 30, [64] + [33] * 30, 28, 4, 128, 16),
    ([1, 70, 1], [30, 140, 200], 4, 2, 128, 4),
    ([0, 1, 100, 5, 0, 1], [4, 20, 140, 5, 0, 90], 7, 1, 128, 16),
]


@pytest.mark.parametrize("case", WIDE_CASES + FOUR_WAVE_CASES, ids=lambda c: f"n{len(c[0])}-q{sum(c[0])}-kv{max(c[1])}-h{c[2]}k{c[3]}-d{c[4]}-b{c[5]}")
@pytest.mark.parametrize("planted", [False, True])
def test_hybrid_batches_in_wide_workgroups(case, planted, batch_rules):
    """Hybrid batches on both sides of the rule for workgroups of eight waves, which batches of more than 128 requests never take: the same
    requests with others that have no new token.  The oracle, and the same bits (without splits, which follow the number of requests) unless
    chains past the end of the grid take the plain form."""
    q_lens, kv_lens, hq, hkv, d, bs = case
    h = si.HybridBatch("wide", q_lens, kv_lens, hq, hkv, d, block_size=bs, seed=sum(q_lens))
    q, kc, vc, tables = si.make_paged_inputs(h)
    if planted:
        kc = kc.clone()
        for b, L in enumerate(kv_lens):
            if L > 50:
                kc[tables[b, 45 // bs], 45 % bs] = 64.0
    others = 129 - h.batch
    padded = si.HybridBatch("narrow", q_lens + [0] * others, kv_lens + [0] * others, hq, hkv, d, block_size=bs)
    padded_tables = np.full((padded.batch, tables.shape[1]), -1, dtype=np.int32)
    padded_tables[: h.batch] = tables

    rule = batch_rules.wide_workgroups
    rule.restype, rule.argtypes = ctypes.c_int64, [ctypes.c_int] * 6 + [ctypes.c_int64]
    group, keys = hq // hkv, tables.shape[1] * bs
    workgroups = rule(h.batch, h.total_q, h.max_q_len, group, hkv, 1, keys)
    assert (workgroups > 0) == (case in WIDE_CASES) and rule(padded.batch, h.total_q, h.max_q_len, group, hkv, 1, keys) == 0
    chains = hkv * sum(-(-(-(-n // 32) * group) // 4) for n in q_lens if n * group > 32)
    steps = hkv * sum(0 < n * group <= 32 for n in q_lens)
    past_the_grid = 0 < workgroups < chains
    assert workgroups == 0 or past_the_grid or chains + max((steps + 1) // 2, min(steps, 256 - chains)) + 15 <= workgroups
    assert past_the_grid == (case in WIDE_CASES[-3:])

    want = _want(h, q, kc, vc, tables)
    wide, narrow = _run_gpu(h, q, kc, vc, tables, use_workspace=False), _run_gpu(padded, q, kc, vc, padded_tables, use_workspace=False)
    _check(wide, want)
    _check(narrow, want)
    if not past_the_grid:
        assert torch.equal(wide.view(torch.int16), narrow.view(torch.int16))


@pytest.mark.parametrize("longest", [407, 511, 512])
def test_short_contexts_under_a_wide_table(longest):
    """Between 257 and 512 (request, KV head) pairs under a table of 8192 keys: launched with eight waves per workgroup, of which
    four leave when no context of the batch has 512 keys."""
    kv_lens = [1 + (37 * i) % longest for i in range(299)] + [longest]
    h = si.HybridBatch("short", [1] * 300, kv_lens, 7, 1, 128, block_size=16, seed=longest)
    q, kc, vc, tables = si.make_paged_inputs(h)
    wide = np.full((h.batch, 8192 // 16), -1, dtype=np.int32)
    wide[:, : tables.shape[1]] = tables
    want = _want(h, q, kc, vc, tables)
    tight, out = _run_gpu(h, q, kc, vc, tables), _run_gpu(h, q, kc, vc, wide)
    _check(out, want)
    # (the tight table is launched with four waves from the start: the same keys per wave, the same bits)
    assert torch.equal(tight.view(torch.int16), out.view(torch.int16)) == (longest < 512)


@pytest.mark.parametrize("d", [64, 80, 128])
def test_scale_near_the_end_of_the_range(d):
    """Scores of -8 under a scale whose products, 3.2e38 in units of log 2, the largest float just holds: equal weights for all
    visible keys (nothing that stands for 'no key yet' may lie above a score).  The products are exact, so the tolerance is the usual one."""
    h = si.HybridBatch("far", [1, 2], [100, 33], 2, 1, d, block_size=16, seed=d)
    q, kc, vc, tables = si.make_paged_inputs(h)
    q, kc = torch.zeros_like(q), kc.clone()
    q[..., 0] = 1.0
    kc[..., 0] = -8.0
    scale = 4.0e37 / 1.44269504088896340736
    _check(_run_gpu(h, q, kc, vc, tables, scale=scale), _want(h, q, kc, vc, tables, scale=scale))


@pytest.mark.parametrize("d", [64, 80, 128])
@pytest.mark.parametrize("bs", [16, 64])
def test_stale_rows_behind_a_context_do_not_count(d, bs):
    """NaN in every cache row that belongs to no context (the tails of pages, pages nobody has): contexts that end at every place
    of a block of keys, in the decode form and in the form for up to 32 rows, unsplit and split, beside a chunk."""
    ends = [1, 2, 3, 15, 16, 17, 30, 31]
    for kv_lens, q_lens in (([e for e in ends] + [32 + e for e in ends] + [700 + e for e in ends], None),
                            ([1600 + e for e in (1, 3, 15, 16, 17, 31)], None),
                            ([1600 + e for e in (3, 16, 31)], [8, 5, 1]),
                            ([500 + e for e in (1, 15, 16, 17, 31)] + [100], [1] * 5 + [70])):
        h = si.HybridBatch("stale", q_lens or [1] * len(kv_lens), kv_lens, 8, 2, d, block_size=bs, seed=len(kv_lens) + bs)
        q, kc, vc, tables = si.make_paged_inputs(h)
        owned = torch.zeros(kc.shape[:2], dtype=torch.bool)
        for b, n in enumerate(kv_lens):
            for at in range(0, n, bs):
                owned[int(tables[b, at // bs]), : min(bs, n - at)] = True
        assert not bool(owned.all())
        want = _want(h, q, kc, vc, tables)
        kc, vc = kc.clone(), vc.clone()
        kc[~owned], vc[~owned] = float("nan"), float("nan")
        _check(_run_gpu(h, q, kc, vc, tables), want)
        _check(_run_gpu(h, q, kc, vc, tables, use_workspace=False), want)
