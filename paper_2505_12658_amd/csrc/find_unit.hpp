// Which work a workgroup of attn_fwd_direct_kernel does: its entry in the dies' queues and, without a work list, its unit of a batch
// whose lengths it reads itself.  Everything here is index arithmetic over the lanes of a wave, on four wave-wide reads and the
// operations of wave_ops.hpp, so that a test can walk every workgroup of a batch on the host.
// Needs kXcds and, before it, wave_ops.hpp (or what stands in for both).
#pragma once
#include <stdint.h>

namespace hydra {

constexpr int kDirectSeqs = 64;
constexpr int kDieUnits = 32;  // compute units of a die

// Workgroups for items of `tiles` wave tiles: as many as there can be (a sequence of L tokens has at most (L + 31) / 32 * group wave tiles and
// pads less than an item), and as take_entry asks for; their order takes care of how the items spread over the dies.
// entry_tiles: wave tiles of an entry of the work list, which the workgroups share, or those of an item where there is no list.
inline int64_t direct_workgroups(int tiles, int entry_tiles, int32_t batch, int32_t total_tokens, int32_t group, int32_t n_kv_heads) {
  const int64_t wave_tiles = ((int64_t)total_tokens + 31 * (int64_t)batch) / 32 * group;
  const int64_t most = (wave_tiles + (entry_tiles - 1) * (int64_t)batch) / entry_tiles * (entry_tiles / tiles) * n_kv_heads;
  return most > kXcds * kDieUnits || n_kv_heads % kXcds == 0 ? most : kXcds * kDieUnits;
}

#if defined(__HIP_DEVICE_COMPILE__)
// The entry that this workgroup takes from the dies' queues: workgroup t the t-th of all entries by place and, at one
// place, by die.  While every queue has entries that is place t / 8 of the own die's queue (t % 8); dies that have run
// out, or never had a (sequence, KV head) pair, take their part of what the others still hold, at the same place in the
// order, so that neither the order by cost nor the grid depends on how the entries are spread over the dies.
// Only where all queues are short do the dies without entries stay idle: spread, every die would fetch rows that another one
// has (one request of 558 tokens, 28 / 4 heads of 128, queues of 32 entries on four dies: 15.5 us, 14.8 by the own dies).
// n: entries of queue lane % 8; the grid has kXcds * kDieUnits workgroups at least.  Called by whole waves; false for workgroups
// past the last entry.
// Without it (every queue done by its own die, the grid sized for the longest queue that max_seqlen allows), us: one request
// of 8192 tokens with 28 / 4 heads of 128 800 -> 422 (half of the dies had nothing; persistent workgroups that steal 518),
// with 8 / 1 heads 682 -> 155 (307); 12 requests of 200 .. 1047 tokens under a bound of 32 768 75.7 -> 59.7.  Counting the
// queues costs a workgroup some 0.1 us, seen in batches that were level without it (300, 1200 and 700 tokens, 28 / 4 heads,
// 26.3 -> 26.6).
__device__ __forceinline__ bool take_entry(int n, int t, int& die, int& place) {
  die = t % kXcds;
  place = t / kXcds;
  const uint32_t open_here = (uint32_t)__builtin_amdgcn_ballot_w64(n > place) & 0xff;
  if (open_here == 0xff) return true;
  // no queue is longer than its die has compute units: every die does its own
  if ((__builtin_amdgcn_ballot_w64(n > kDieUnits) & 0xff) == 0) return open_here >> die & 1;
  int count[kXcds], total = 0;
#pragma unroll
  for (int y = 0; y < kXcds; ++y) {
    count[y] = __builtin_amdgcn_readlane(n, y);
    total += count[y];
  }
  if (t >= total) return false;
  auto entries_before = [&](int p) {  // at places below p
    int sum = 0;
#pragma unroll
    for (int y = 0; y < kXcds; ++y) sum += count[y] < p ? count[y] : p;
    return sum;
  };
  // the last place with at most t entries before it: at least t / 8, at most t; 64 candidates at a time
  const int lane = threadIdx.x & 63;
  for (int span = t - place + 1; span > 1;) {
    const int step = (span + 63) / 64;
    place += (__builtin_popcountll(__builtin_amdgcn_ballot_w64(lane * step < span && entries_before(place + lane * step) <= t)) - 1) * step;
    span = step;
  }
  uint32_t open = (uint32_t)__builtin_amdgcn_ballot_w64(n > place) & 0xff;
  for (int skip = t - entries_before(place); skip > 0; --skip) open &= open - 1;
  die = __builtin_ctz(open);
  return true;
}

// The unit of this workgroup in a batch whose sequence of length L has units(L) units per KV head: its KV head, its
// sequence and its number there; false for workgroups past the last one.  The order is that of the work list
// (worklist.hpp): sequences ranked by length, longest first, their (sequence, KV head) pairs dealt to the dies in
// serpentine order, and the units of a die's pairs handed out by take_entry.
template <typename Units>
__device__ __forceinline__ bool find_unit(const int32_t* cu, int batch, int n_kv_heads, Units units, int& seq_start, int& seq_len, int& kv_head, int& unit) {
  const int lane = threadIdx.x & 63;
  int start = 0, len = 0;
  if (lane < batch) {
    start = cu[lane];
    len = cu[lane + 1] - start;
  }
  const int pairs = batch * n_kv_heads;
  const float per_kv = 1.0f / n_kv_heads;
  // the pair in a row of one pair per die, and its sequence
  auto pair_of = [&](int row, int column) { return row * kXcds + ((row & 1) ? kXcds - 1 - column : column); };
  auto seq_of = [&](int pair) { return (int)((pair + 0.5f) * per_kv); };  // pair / n_kv_heads (exact: fewer than 2^20 pairs)
  int die = (int)blockIdx.x % kXcds, place = (int)blockIdx.x / kXcds;
  const int first_len = __builtin_amdgcn_readfirstlane(len);
  if (__builtin_amdgcn_ballot_w64(lane < batch && len != first_len) == 0) {
    // Sequences of one length (images of one resolution, a request alone): every pair has as many units, and the place says
    // which it is, without lanes that ask each other (us, through the scan below and so: one image of 577 tokens with 16 heads of
    // 64 9.71 -> 9.49, 12 of them 28.0 -> 27.6; one request of 558 tokens, 28 / 4 heads of 128, 12.58 -> 12.28, of 2000 39.9 -> 39.7).
    const int n = __builtin_amdgcn_readfirstlane(units(first_len));
    if (n <= 0) return false;
    if (batch == 1 && pairs < kXcds && (pairs & (pairs - 1)) == 0 && n > kDieUnits) {
      // one request of 1, 2 or 4 KV heads: its pairs in turn, which gives each die one pair, or a part of one (through take_entry, whose counts take
      // a workgroup half a microsecond: 28 / 4 heads of 128, 700 tokens 14.3 us, 13.8 so; in halved items 400 tokens 9.1 and 8.7)
      kv_head = (int)blockIdx.x % pairs;
      unit = (int)blockIdx.x / pairs;
      seq_start = __builtin_amdgcn_readfirstlane(start);
      seq_len = first_len;
      return unit < n;
    }
    if (n_kv_heads % kXcds != 0 && (pairs > kXcds || n > kDieUnits)) {
      const int rows = pairs / kXcds;
      if (!take_entry(n * (rows + (pair_of(rows, lane % kXcds) < pairs ? 1 : 0)), (int)blockIdx.x, die, place)) return false;
    }
    const int row = (int)((place + 0.5f) * __builtin_amdgcn_rcpf((float)n));  // place / n (exact: fewer than 2^20 places)
    const int pair = pair_of(row, die), seq = seq_of(pair);
    if (pair >= pairs) return false;
    kv_head = pair - seq * n_kv_heads;
    unit = place - row * n;
    seq_start = __builtin_amdgcn_readlane(start, seq);
    seq_len = first_len;
    return true;
  }
  // lane r gets the sequence of rank r (ranks are distinct; lanes without a sequence come last)
  int rank = lane < batch ? 0 : lane;
  for (int o = 0; o < batch; o += 4) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {  // (lanes past the batch hold length 0 and a larger number: they precede nobody)
      const int other = __builtin_amdgcn_readlane(len, o + e);
      if (lane < batch) rank += (other > len || (other == len && o + e < lane)) ? 1 : 0;
    }
  }
  start = __builtin_amdgcn_ds_permute(rank * 4, start);
  len = __builtin_amdgcn_ds_permute(rank * 4, len);
  const int n = units(len);
  // the units of a pair (0 past the last one)
  auto units_of = [&](int pair) {
    const int seq = seq_of(pair);
    const int u = __builtin_amdgcn_ds_bpermute((seq < 63 ? seq : 63) * 4, n);
    return pair < pairs ? u : 0;
  };
  // (not where every die has the same pairs of every sequence, nor where no queue can be longer than take_entry asks for)
  if (n_kv_heads % kXcds != 0 && (pairs > kXcds || __builtin_amdgcn_ballot_w64(n > kDieUnits) != 0)) {
    int queue = 0;  // units of the pairs of column lane % 8
    for (int row0 = 0; row0 * kXcds < pairs; row0 += 64 / kXcds) queue += units_of(pair_of(row0 + lane / kXcds, lane % kXcds));
    queue = sum_of_columns(queue);
    if (!take_entry(queue, (int)blockIdx.x, die, place)) return false;
  }
  // rows of the die's column, 64 at a time: units of each row's pair and, by a scan, of the rows before it
  int before = 0;
  for (int row0 = 0; row0 * kXcds < pairs; row0 += 64) {
    const int pair = pair_of(row0 + lane, die), seq = seq_of(pair);
    const int mine = units_of(pair);
    const int incl = wave_scan_add(mine);
    const int here = __builtin_amdgcn_readlane(incl, 63);
    if (place < before + here) {
      const int at = place - before;
      const int r = __builtin_ctzll(__builtin_amdgcn_ballot_w64(incl > at));
      const int pair_r = __builtin_amdgcn_readlane(pair, r), seq_r = __builtin_amdgcn_readlane(seq, r);
      kv_head = pair_r - seq_r * n_kv_heads;
      unit = at - __builtin_amdgcn_readlane(incl - mine, r);
      seq_start = __builtin_amdgcn_readlane(start, seq_r);
      seq_len = __builtin_amdgcn_readlane(len, seq_r);
      return true;
    }
    before += here;
  }
  return false;
}
#endif  // __HIP_DEVICE_COMPILE__

}  // namespace hydra
