// Attention of decode steps over the paged KV cache (gfx950): few rows, long contexts, HBM-bound.
//
// All (new token, query head) pairs of one (request, KV head) form ONE tile of at most 16 rows, so the context
// is read once per KV head.  The waves of a workgroup split the keys: wave w takes the blocks of 32 keys
// w, w + W, w + 2 W, ... of the workgroup's share, and the partial results (row maximum, row sum, unnormalised
// output) are merged through LDS at the end.
//
// The contractions are
//   S^T[key, row] = K Q^T        v_mfma_f32_16x16x32_bf16, A = K, B = Q
//   O^T[c, row]  += V^T P^T      the same instruction, A = V^T, B = P^T
// and both K and V come from memory in load instructions that cover whole rows (4 rows of 256 bytes at head_dim 128):
//   - K goes through a stage of the wave's own in LDS, where it is read back in the layout of the A operand, lane
//     (m, h) = (lane % 16, lane / 16) holding 16-byte piece 4 s + h of key m in step s.
//   - V stays in registers.  Lane (m, h) loads, for each of the eight keys it contributes to a block of 32, its D / 16
//     columns m D/16 .., and one v_perm_b32 per register turns that 8 x (D / 16) block of bf16 into the
//     eight-keys-per-column order of the A operand.  The matrix instruction that takes column u of every lane's block
//     yields output columns m D/16 + u.
// In the result layout of the first contraction lane (m, h) has row m and keys 4 h .. 4 h + 3 of both halves of 16; as
// the B operand of the second a lane owns eight keys of its row, and which eight is free as long as V uses the same:
// so P stays where it is.
//
// What bounds it: memory.  Reading rows of 256 bytes, scattered in pages of 16, this chip gives 6.4 TB/s with
// non-temporal loads and 5.7 without; 16 rows x 64 bytes per instruction (K straight in the operand layout, no LDS)
// gave 5.5 and 4.9, and was built first.  A compute unit gets at most 48 GB/s of a stream that comes from HBM, four
// waves with one block of 32 keys (16 KB) in flight each are enough for that, and a second block in flight per wave
// made the whole chip slower (5.2 - 5.7 TB/s).  So a wave keeps one block in flight: the K registers are refilled as soon as
// they are staged, the V registers as soon as the product is out.
// Against the form for up to 32 rows (32 x 32 tiles, in attn_paged.hpp), us: 96 requests of 128 .. 1782 tokens, 28 / 4
// heads of 128, 41.5 -> 35.7 (150 MB); 33 requests of 600 .. 1100 tokens, 32 / 32 heads, 83.8 -> 79.7 (475 MB, 5.9 TB/s);
// 4 requests of 300 .. 1200 tokens 12.3 -> 5.5, in 16 shares instead of 2.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_tiles.hpp"
#include "paged_args.hpp"

namespace hydra {
namespace paged {

constexpr int kDecodeRows = 16;  // rows (new tokens x grouped heads) of a decode tile
constexpr int kDecodeKeys = 32;  // keys per step
constexpr int kUnits = 256;      // compute units

// Floats of LDS per wave and row of partial output (padded: the rows of a wave start in different banks).
template <int D>
constexpr int kDecodeRowFloats = D + 4;

// A wave's slot in LDS: its stage of 32 rows of K during the loop, its partial output for the merge.
template <int D>
constexpr int kDecodeSlotFloats = kDecodeRows * kDecodeRowFloats<D> > kDecodeKeys * D / 2 ? kDecodeRows * kDecodeRowFloats<D> : kDecodeKeys * D / 2;
template <int D>
constexpr size_t kDecodeLdsPerWave = (kDecodeSlotFloats<D> + 2 * kDecodeRows) * sizeof(float);

// (see attn_decode_kernel)
constexpr int kOrderedKeys = 256;      // a batch without a context of more keys is not ordered by them
constexpr int kDecodeShortKeys = 512;  // a batch without a context of as many does with four waves per workgroup

#if defined(__HIP_DEVICE_COMPILE__)

typedef const __attribute__((address_space(4))) int32_t* const_table_t;

// The same value of all four lanes l, l ^ 16, l ^ 32, l ^ 48 combined with `op`.
template <typename Op>
__device__ __forceinline__ float over_row_lanes(float x, Op op) {
  float r0, r1;
  own_and_other_half(x, r0, r1);
  x = op(r0, r1);
  // (as own_and_other_half, between the odd and the even rows of 16 lanes)
  float a = x, b = x;
  asm volatile("s_nop 3\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 3" : "+v"(a), "+v"(b));
  return op(a, b);
}

// A wave's state for one tile of up to 16 rows, and its walk over keys.
template <int D>
struct DecodeWave {
  static constexpr int KS = D / 32;          // 32-wide steps of the QK contraction
  static constexpr int CW = D / 16;          // columns of V per lane, units of the PV contraction
  static constexpr int VW = CW / 2;          // registers per V row of a lane
  static constexpr int RL = D / 8;           // lanes per K row (16 bytes each)
  static constexpr int KL = 16 * RL / 64;    // load instructions per 16 rows of K
  static constexpr int ROWB = D * 2;
  typedef __attribute__((ext_vector_type(VW))) uint32_t vrow_t;

  bf16x8_t q[KS];
  f32x4_t o[CW];
  float row_max, row_sum;  // maximum over all lanes of the row, this lane's part of the sum
  u32x4_t kreg[2][KL];     // [half of 16 keys]: rows lane / RL + u 64 / RL, piece lane % RL
  vrow_t vreg[2][4];       // [half of 16 keys][key 4 h + j]
  uint64_t k_base, v_base; // this KV head's part of cache row 0
  uint32_t row_bytes, k_off, v_off;
  int k_chunk, k_row;
  uint32_t k_put, k_get[KS]; // LDS addresses of this lane's pieces of the wave's K stage
  int kv_len, block_shift, last_block;

  __device__ __forceinline__ void init(const uint16_t* k_cache, const uint16_t* v_cache, int n_kv_heads, int kv_head, int kv_len_, int block_shift_,
                                       int num_blocks, const uint16_t* q_row, float scale_log2, uint32_t stage, int lane) {
    const int m = lane & 15, h = lane >> 4;
    k_base = (uint64_t)(uintptr_t)(k_cache + (int64_t)kv_head * D);
    v_base = (uint64_t)(uintptr_t)(v_cache + (int64_t)kv_head * D);
    row_bytes = (uint32_t)n_kv_heads * (D * 2);
    const int kr = lane / RL, kc = lane % RL;
    k_off = (uint32_t)kr * row_bytes + kc * 16;
    k_put = stage + kr * ROWB;
    k_chunk = kc;
    k_row = kr;
#pragma unroll
    for (int s = 0; s < KS; ++s) k_get[s] = stage + m * ROWB + k_swizzle<D>(m, 4 * s + h) * 16;
    v_off = (uint32_t)(4 * h) * row_bytes + m * (CW * 2);
    kv_len = kv_len_;
    block_shift = block_shift_;
    last_block = num_blocks - 1;
#pragma unroll
    for (int s = 0; s < KS; ++s) q[s] = *reinterpret_cast<const bf16x8_t*>(q_row + (4 * s + h) * 8);
    restart();
  }
  __device__ __forceinline__ void restart() {  // before the first key of a stream
    row_max = kLowest;
    row_sum = 0.f;
#pragma unroll
    for (int u = 0; u < CW; ++u) o[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  // Descriptor of the 16 rows that start at key `key` (a multiple of 16), which lie in cache block `block`: it ends
  // with the last row of the context, so rows past it (and whole groups past it) arrive as zeros.
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rows16(uint64_t base, int block, int key) const {
    const uint32_t slot = ((uint32_t)block << block_shift) + ((uint32_t)key & ((1u << block_shift) - 1u));
    int valid = kv_len - key;
    valid = valid > 16 ? 16 : valid;
    const uint32_t bytes = valid > 0 ? (uint32_t)(valid - 1) * row_bytes + D * 2 : 0u;
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(base + (uint64_t)slot * row_bytes), 0, (int)bytes, 0x00020000);
  }
  // (nt: every key of a context is read by one wave only)
  __device__ __forceinline__ void load_k(int half, int block, int key) {
    const __amdgpu_buffer_rsrc_t r = rows16(k_base, block, key);
#pragma unroll
    for (int u = 0; u < KL; ++u) kreg[half][u] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)k_off, u * (64 / RL) * (int)row_bytes, 2);
  }
  __device__ __forceinline__ void stage_k() const {
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int u = 0; u < KL; ++u) {
        const int row = 16 * half + u * (64 / RL);
        *reinterpret_cast<u32x4_t*>(HYDRA_LDS_BYTE(k_put + row * ROWB + k_swizzle<D>(row + k_row, k_chunk) * 16)) = kreg[half][u];
      }
  }
  __device__ __forceinline__ void load_v(int half, int block, int key) {
    const __amdgpu_buffer_rsrc_t r = rows16(v_base, block, key);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (VW == 4) vreg[half][j] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)v_off, j * (int)row_bytes, 2);
      else vreg[half][j] = __builtin_amdgcn_raw_buffer_load_b64(r, (int)v_off, j * (int)row_bytes, 2);
    }
  }

  // S^T of the block of 32 keys in kreg: s[half], keys 16 half + 4 h + r of row m
  __device__ __forceinline__ void scores(f32x4_t (&s)[2]) const {
#pragma unroll
    for (int half = 0; half < 2; ++half) s[half] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < KS; ++st)
#pragma unroll
      for (int half = 0; half < 2; ++half)
        {
        const bf16x8_t kf = *reinterpret_cast<const bf16x8_t*>(HYDRA_LDS_BYTE(k_get[st] + half * 16 * ROWB));
        s[half] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, q[st], s[half], 0, 0, 0);
      }
  }
  // Online softmax of the block whose first key is key0: P in bf16, O and the sums rescaled.
  __device__ __forceinline__ bf16x8_t softmax(f32x4_t (&s)[2], int key0, int lim, float c, int h) {
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (key0 + 16 * half + 4 * h + r > lim) s[half][r] = -__builtin_inff();
    float top = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])), fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
    top = over_row_lanes(top, [](float x, float y) { return fmaxf(x, y); });
    // (a row whose keys are all masked so far keeps the initial, very negative maximum: its exponentials are 0)
    const float m_new = fmaxf(row_max, top);
    const float alpha = fast_exp2((row_max - m_new) * c);
    row_max = m_new;
    const float mc = reference_exponent(m_new, c);
    bf16x8_t p;
    float sum = 0.f;
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        const f32x2_t e = {fast_exp2(__builtin_fmaf(s[half][r], c, -mc)), fast_exp2(__builtin_fmaf(s[half][r + 1], c, -mc))};
        sum += e[0];
        sum += e[1];
        const bf16x2_t b = __builtin_convertvector(e, bf16x2_t);
        p[4 * half + r] = b[0];
        p[4 * half + r + 1] = b[1];
      }
    row_sum = row_sum * alpha + sum;
#pragma unroll
    for (int u = 0; u < CW; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) o[u][r] *= alpha;
    return p;
  }
  // O^T += V^T P^T for the block in vreg
  __device__ __forceinline__ void product(const bf16x8_t& p) {
#pragma unroll
    for (int u = 0; u < CW; ++u) {
      // column u of the lane's block: low or high halves of register u / 2 of the eight rows, two rows per register
      const uint32_t sel = u % 2 ? 0x07060302u : 0x05040100u;
      u32x4_t a;
#pragma unroll
      for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int j = 0; j < 4; j += 2) a[2 * half + j / 2] = __builtin_amdgcn_perm(vreg[half][j + 1][u / 2], vreg[half][j][u / 2], sel);
      o[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), p, o[u], 0, 0, 0);
    }
  }
};

// One workgroup's share of one (request, KV head): all of it, its output included, when the context fits one share,
// otherwise a partial result for the combine kernel.  Called by all n_waves waves; lds: kDecodeLdsPerWave<D> bytes per wave
// (PER_WAVE 2: twice as many), 16-byte aligned.  Does nothing for a request that has no new tokens or more than kDecodeRows rows.
// The keys of a share are dealt out to n_streams streams, block by block, each with a running maximum, a sum and an output of
// its own until the merge: so the number of streams is part of the result.  It is n_waves, or with PER_WAVE 2 also twice that:
// a wave then walks its first stream and goes on with its second one, whose first block is in flight by then.
// thread: number among the threads of the n_waves waves.  Returns whether the waves met at a workgroup barrier (once) on the way.
template <int D, int PER_WAVE = 1>
__device__ __forceinline__ bool run_decode(const PagedArgs& a, float* lds, int n_waves, int n_streams, int b, int kv_head, int q_start, int q_len, int kv_len,
                                           int split, int thread) {
  const int lane = thread & 63;
  const int wave = __builtin_amdgcn_readfirstlane(thread >> 6);
  const int m = lane & 15, h = lane >> 4;
  float* s_max = lds;
  float* s_sum = s_max + PER_WAVE * n_waves * kDecodeRows;
  float* s_slots = s_sum + PER_WAVE * n_waves * kDecodeRows;
  const bool two = PER_WAVE == 2 && n_streams > n_waves;  // (else as with PER_WAVE 1)

  if (kv_len <= 0) return false;
  const int n_halves = (kv_len + kDecodeKeys - 1) / kDecodeKeys;
  int begin, end, per_share, n_shares;
  share_plan(n_halves, a.n_splits, a.least_log2, per_share, n_shares);
  split_range(n_halves, per_share, split, begin, end);
  if (begin >= end) return false;  // past the context's last share: the combine kernel knows and skips it

  // Block-table entries of the wave's next 32 steps: lane 2 i + half has the entry of that half of step i
  // (one load; the loop takes them from there lane by lane).  Ids are clamped to the cache, so that a corrupt
  // table cannot make the loads leave it; entries past the context are not read.
  const int32_t* table = a.block_tables + (int64_t)b * a.max_blocks_per_seq;
  const int last_entry = (kv_len - 1) >> a.block_shift;
  auto steps_of = [&](int stream) { return begin + stream < end ? (end - begin - stream + n_streams - 1) / n_streams : 0; };
  const int steps0 = steps_of(wave), steps = two ? steps0 + steps_of(wave + n_waves) : steps0;  // of the first stream, of all
  auto key_of = [&](int i) {
    int block = wave + n_streams * i;
    if (PER_WAVE == 2 && two && i >= steps0) block = wave + n_waves + n_streams * (i - steps0);
    return (begin + block) * kDecodeKeys;
  };
  auto entries = [&](int first_step) {
    const int key = key_of(first_step + (lane >> 1)) + 16 * (lane & 1);
    int e = key >> a.block_shift;
    return table[e < last_entry ? e : last_entry];
  };
  // (the first ones are asked for together with the request's rows)
  int ids = entries(0);
  if (q_len <= 0 || kv_len < q_len || q_len * a.group > kDecodeRows) return false;
  const int n_rows = q_len * a.group;

  // this lane's row
  const int row = m < n_rows ? m : n_rows - 1;
  const int token = quotient(row, a.group);
  const int head = kv_head * a.group + (row - token * a.group);
  const int lim = kv_len - q_len + token;  // largest visible key
  const float c = a.scale_log2;

  DecodeWave<D> w;
  w.init(a.k_cache, a.v_cache, a.n_kv_heads, kv_head, kv_len, a.block_shift, a.num_blocks, a.q + (int64_t)(q_start + token) * a.q_stride + head * D, c,
         (uint32_t)(uintptr_t)HYDRA_LDS_PTR(s_slots + (wave + (PER_WAVE - 1) * n_waves) * kDecodeSlotFloats<D>), lane);
  // A stream's rows' maximum, sum and unnormalised output, for the merge.  (The wave's stage of K is the last slot it writes.)
  constexpr int RF = kDecodeRowFloats<D>;
  constexpr int CW = DecodeWave<D>::CW;
  auto leave = [&](int stream) {
    const float total_own = over_row_lanes(w.row_sum, [](float x, float y) { return x + y; });
    if (h == 0) {
      s_max[stream * kDecodeRows + m] = w.row_max;
      s_sum[stream * kDecodeRows + m] = total_own;
    }
    if (m < n_rows) {
      float* mine = s_slots + stream * kDecodeSlotFloats<D> + m * RF;
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < CW; u += 4)  // columns (4 h + r) CW + u ..
          *reinterpret_cast<f32x4_t*>(mine + (4 * h + r) * CW + u) = f32x4_t{w.o[u][r], w.o[u + 1][r], w.o[u + 2][r], w.o[u + 3][r]};
    }
  };
  if (PER_WAVE == 2 && two && steps0 == 0) leave(wave);
  if (steps > 0) {
    auto in_cache = [&](int id) { return id < 0 ? 0 : (id > w.last_block ? w.last_block : id); };
    auto id_of = [&](int i, int half) { return __builtin_amdgcn_readlane(ids, 2 * (i & 31) + half); };
    ids = in_cache(ids);
#pragma unroll
    for (int half = 0; half < 2; ++half) w.load_k(half, id_of(0, half), key_of(0) + 16 * half);
#pragma unroll
    for (int half = 0; half < 2; ++half) w.load_v(half, id_of(0, half), key_of(0) + 16 * half);
    for (int i = 0; i < steps; ++i) {
      f32x4_t s[2];
      w.stage_k();
      // (the loads of a step that does not exist are issued all the same, with nothing in range: a branch around
      // them would make the compiler wait for everything in flight where the paths meet again)
      if ((i & 31) == 31) ids = in_cache(entries(i + 1));
      const int b0 = id_of(i + 1, 0), b1 = id_of(i + 1, 1), next = i + 1 < steps ? key_of(i + 1) : kv_len;
      w.load_k(0, b0, next);
      w.load_k(1, b1, next + 16);
      __builtin_amdgcn_sched_barrier(0);
      w.scores(s);
      const bf16x8_t p = w.softmax(s, key_of(i), lim, c, h);
      __builtin_amdgcn_sched_barrier(0);
      w.product(p);
      __builtin_amdgcn_sched_barrier(0);
      w.load_v(0, b0, next);
      w.load_v(1, b1, next + 16);
      if (PER_WAVE == 2 && two && i + 1 == steps0) {
        __builtin_amdgcn_sched_barrier(0);
        leave(wave);
        w.restart();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ---- merge ----
  __builtin_amdgcn_sched_barrier(0);
  leave(two ? wave + n_waves : wave);
  __syncthreads();
  const bool whole = n_shares == 1;  // the context is one share: this workgroup writes the output
  constexpr int kCols = D / 4;
  for (int i = thread; i < n_rows * kCols; i += 64 * n_waves) {
    const int r = i / kCols, col = (i - r * kCols) * 4;
    // (four streams at a time, so that their reads are in flight together; there are four or eight)
    float top = s_max[r];
    for (int o = 0; o < n_streams; o += 4)
#pragma unroll
      for (int e = o; e < o + 4; ++e) top = fmaxf(top, s_max[e * kDecodeRows + r]);
    float total = 0.f;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int o = 0; o < n_streams; o += 4) {
      float own_top[4], own_sum[4];
      f32x4_t v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        own_top[e] = s_max[(o + e) * kDecodeRows + r];
        own_sum[e] = s_sum[(o + e) * kDecodeRows + r];
        v[e] = *reinterpret_cast<const f32x4_t*>(s_slots + (o + e) * kDecodeSlotFloats<D> + r * RF + col);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // (a stream that saw no key of this row still holds the initial maximum: weight 0)
        const float weight = fast_exp2((own_top[e] - top) * c);
        total += weight * own_sum[e];
#pragma unroll
        for (int x = 0; x < 4; ++x) acc[x] += weight * v[e][x];
      }
    }
    if (whole) {
      const int tok = quotient(r, a.group), hd = kv_head * a.group + (r - tok * a.group);
      const float inv = 1.0f / total;
      const f32x2_t a0 = {acc[0] * inv, acc[1] * inv}, a1 = {acc[2] * inv, acc[3] * inv};
      const u32x2_t pk = {__builtin_bit_cast(uint32_t, __builtin_convertvector(a0, bf16x2_t)),
                          __builtin_bit_cast(uint32_t, __builtin_convertvector(a1, bf16x2_t))};
      *reinterpret_cast<u32x2_t*>(a.out + ((int64_t)(q_start + tok) * a.n_q_heads + hd) * D + col) = pk;
    } else {
      float* rec = a.partials + (((int64_t)b * a.n_kv_heads + kv_head) * a.n_splits + split) * kPartialFloats<D>;
      if (col == 0) {
        rec[r] = top;
        rec[kRows + r] = total;
      }
      *reinterpret_cast<f32x4_t*>(rec + 2 * kRows + r * D + col) = acc;
    }
  }
  return true;
}

// The lane of the set bit number n of a mask that has more than n.
__device__ __forceinline__ int nth_lane(uint64_t mask, int n) {
  const int lane = threadIdx.x & 63;
  const int lower = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
  return __builtin_ctzll(__builtin_amdgcn_ballot_w64((mask >> lane & 1) != 0 && lower == n));
}

// The request of rank `rank` (register x 64 + lane), longest first and equal ones by number, of those whose length steps[]
// holds; -1 in the other lanes.  A search over the bits of a length, highest first: ballots count how many requests reach it.
template <int REGS>
__device__ __forceinline__ int search_rank(const int (&steps)[REGS], int rank, int table_keys) {
  // the largest number of steps that more than `rank` requests reach: that of the request asked for
  int v = 0;
  for (int bit = 1 << (31 - __builtin_clz((table_keys + kDecodeKeys - 1) / kDecodeKeys)); bit > 0; bit >>= 1) {
    int reach = 0;
#pragma unroll
    for (int r = 0; r < REGS; ++r) reach += __builtin_popcountll(__builtin_amdgcn_ballot_w64(steps[r] >= (v | bit)));
    v = reach > rank ? v | bit : v;
  }
  int skip = rank;  // requests of as many steps that come before it
#pragma unroll
  for (int r = 0; r < REGS; ++r) skip -= __builtin_popcountll(__builtin_amdgcn_ballot_w64(steps[r] > v));
  int found = -1;
#pragma unroll
  for (int r = 0; r < REGS; ++r) {
    const uint64_t here = __builtin_amdgcn_ballot_w64(steps[r] == v);
    const int n = __builtin_popcountll(here);
    if (skip >= 0 && skip < n) found = r * 64 + nth_lane(here, skip);
    skip -= n;
  }
  return found;
}

// The request of rank `rank` when the batch is ordered by context, longest first (in steps of kDecodeKeys; equal ones by
// number), and its context.  Called by whole waves; every wave finds it for itself, without LDS or a barrier: the lengths
// lie in REGS registers of its lanes, and a search over the bits of a length, highest first, counts with ballots how many
// requests reach it (0.3 us; a search over single keys, with branches around the registers that a batch does not fill, 0.9).
// A request without new tokens ranks by the context it has left, and its workgroups leave at once (96 slots, a third of them idle with
// 1500 .. 1800 old tokens, 20.4 us in the order of the batch, 18.0 so).
// False where the order would not matter: contexts within a quarter of each other, or none of kOrderedKeys.
// any_long: some context has kDecodeShortKeys.
template <int REGS>
__device__ __forceinline__ bool request_of_rank(const PagedArgs& a, int rank, int table_keys, int& b, int& kv_len, bool& any_long) {
  const int lane = threadIdx.x & 63;
  int len[REGS], steps[REGS];
#pragma unroll
  for (int r = 0; r < REGS; ++r) len[r] = a.kv_lens[r * 64 + lane < a.batch ? r * 64 + lane : a.batch - 1];
  bool ragged = false, far = false, longer = false;
#pragma unroll
  for (int r = 0; r < REGS; ++r) {
    const bool real = r * 64 + lane < a.batch;
    len[r] = len[r] < table_keys ? len[r] : table_keys;
    steps[r] = real ? (len[r] > 0 ? (len[r] + kDecodeKeys - 1) / kDecodeKeys : 0) : -1;
    const int64_t first = __builtin_amdgcn_readfirstlane(steps[0]);
    far = far || steps[r] > kOrderedKeys / kDecodeKeys;
    longer = longer || len[r] >= kDecodeShortKeys;
    ragged = ragged || (real && (steps[r] * 5 < first * 4 || steps[r] * 4 > first * 5));
  }
  any_long = __builtin_amdgcn_ballot_w64(longer) != 0;
  if (__builtin_amdgcn_ballot_w64(far) == 0 || __builtin_amdgcn_ballot_w64(ragged) == 0) return false;
  const int at = search_rank(steps, rank, table_keys);
  if (at < 0) return true;  // (not for a rank that a request has)
  b = at;
#pragma unroll
  for (int r = 0; r < REGS; ++r)
    if (at / 64 == r) kv_len = __builtin_amdgcn_readlane(len[r], at % 64);
  return true;
}

#endif  // __HIP_DEVICE_COMPILE__

// Whether requests of `rows` rows take this form (the 16 keys of half a step lie in one cache block).
template <int D>
constexpr bool kDecodeForm = D == 64 || D == 128;
constexpr int kDecodeMinBlock = 16;

// Waves per SIMD the kernel is built for (168 registers each).
constexpr int kDecodeWavesPerSimd = 3;
constexpr int kDecodeWaves = 4;        // waves of a workgroup: enough to keep a compute unit's memory path full
constexpr int kDecodeMaxStreams = 8;   // as many waves: a unit then holds one workgroup at a time
constexpr int kDecodeWideTable = 4096; // keys in a row of the block table from which on the kernel looks for that

// Batches of more pairs than compute units are taken in the order of their contexts: units are then level, whatever the order
// of the requests in the batch, and no long context starts behind another one.  The first 256 workgroups, which the hardware
// deals out one to a unit, take the 256 longest pairs from the shortest of them up, the ones behind them the others from the
// longest down: so the second pair of a unit is the longer the shorter its first one is, and the very longest have a unit
// for themselves.  us, in the order of the batch and so (the same bits), 28 / 4 heads of 128: 96 requests of 128 .. 1800 tokens
// 39.4 -> 31.8, 125 43.4 -> 33.6, 80 31.6 -> 28.2, 70 of 900 .. 1800 44.3 -> 37.4, 200 of 128 .. 1800 60.9 -> 46.9, 100 of 40 .. 407
// 12.8 -> 10.3; 32 / 32 heads: 14 of 300 .. 2000 43.7 -> 36.4, 33 of 600 .. 1100 equal, 9 of 300 .. 3000, which the longest context
// holds up either way, 34.5 -> 35.0.
// Not where no context has more than kOrderedKeys (the search costs what the order gains: 300 of 30 .. 200 tokens 14.4 -> 15.5),
// and the batch has to fit four registers of a wave's lanes (eight: 500 of 20 .. 100 under a wide table 15.7 -> 17.0, without a search).
constexpr int kOrderedMost = 256;  // requests
inline bool decode_ordered(int64_t pairs, int n_splits, int batch, int64_t table_keys) {
  return pairs > kUnits && n_splits == 1 && batch <= kOrderedMost && table_keys > kOrderedKeys;
}
// Long contexts of one to two pairs per unit are dealt out to eight streams, others to four.  The number says how the sums are
// put together (run_decode), so it follows from the batch alone and not from the order it is taken in.
constexpr int kDecodeLongKeys = 768;   // a block table from which on contexts count as long
inline int decode_streams(int64_t pairs, int n_splits, int64_t table_keys) {
  return pairs > kUnits && pairs <= 2 * kUnits && n_splits == 1 && table_keys >= kDecodeLongKeys ? kDecodeMaxStreams : kDecodeWaves;
}
// Eight streams are eight waves where a unit should hold one pair at a time, so that one that is done early takes one of the
// remaining pairs.  In the order of the batch that is everywhere (96 requests of 128 .. 1782 tokens 35.7 us, 39.7 with four waves
// and four streams), in the order of the contexts where the second pairs are nearly as many as the first ones.  Otherwise four
// waves have two streams each, and two pairs share a unit.  us, eight waves and four, 28 / 4 heads of 128: 96 of 360 .. 900 23.0 and
// 21.4, 80 of 1000 .. 1099 36.3 and 34.8, 70 of 900 .. 1800 38.6 and 37.4, 96 of 128 .. 1800 31.5 and 31.8; from 464 pairs on: 116 of
// 90 .. 900 16.5 and 17.4, 128 of 200 .. 2000 36.1 and 38.8, of 630 .. 900 33.9 and 32.9.
constexpr int kDecodeManyPairs = 464;
inline int decode_waves(int64_t pairs, int streams, bool ordered) { return ordered && pairs < kDecodeManyPairs ? kDecodeWaves : streams; }

#if defined(__HIP_DEVICE_COMPILE__)
// All arguments in one trip to memory.  (Left to itself the compiler asks for each group of them where it is first used and waits there.)
// us of the decode kernel and the merge so, and then without integer divisions on the way to the first load (`quotient`, and a grid that
// says which request and head), 28 / 4 heads of 128: 4 requests of 300 .. 1500 tokens 6.86 -> 6.62 -> 6.39, 16 of 400 .. 800 9.5 -> 9.3 -> 8.9,
// 4 of 150 .. 300 (not cut) 5.40 -> 5.34 -> 5.05, one of 16 384 11.3 -> 11.1 -> 10.7, 8 of 16 384 45.3 -> 45.2 -> 44.9.  (The block table
// asked for together with the lengths, where a context is not cut: no faster.)
__device__ __forceinline__ void ask_for_arguments(const PagedArgs& a) {
  asm volatile("" : : "s"(a.q), "s"(a.out), "s"(a.q_stride), "s"(a.k_cache), "s"(a.v_cache), "s"(a.block_tables), "s"(a.cu_seqlens_q), "s"(a.kv_lens),
               "s"(a.max_blocks_per_seq), "s"(a.num_blocks), "s"(a.block_shift), "s"(a.n_q_heads), "s"(a.n_kv_heads), "s"(a.group), "s"(a.scale_log2),
               "s"(a.n_splits), "s"(a.least_log2), "s"(a.partials), "s"(a.batch));
}
#endif

// grid = (n_kv_heads, batch, n_splits) workgroups: share-major (the first shares of all pairs, which every request
// has, then the second shares, ...).  Ordered: batch * n_kv_heads.  Dynamic LDS: STREAMS * kDecodeLdsPerWave<D> bytes.
template <int D, bool ORDERED, int WAVES, int STREAMS>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(kDecodeWavesPerSimd, kDecodeWavesPerSimd))) void attn_decode_kernel(
    const PagedArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  extern __shared__ __attribute__((aligned(16))) float s_decode[];
  ask_for_arguments(a);
  const int64_t table_keys = (int64_t)a.max_blocks_per_seq << a.block_shift;  // (at most 2^30)
  const const_table_t cu = (const_table_t)(uintptr_t)a.cu_seqlens_q, lens = (const_table_t)(uintptr_t)a.kv_lens;
  int split = 0, b, kv_head;
  if constexpr (ORDERED) {
    const int id = (int)blockIdx.x, pair = id < kUnits ? kUnits - 1 - id : id;
    b = quotient(pair, a.n_kv_heads);
    kv_head = pair - b * a.n_kv_heads;
  } else {
    split = (int)blockIdx.z;
    b = (int)blockIdx.y;
    kv_head = (int)blockIdx.x;
  }
  int q_start = cu[b], q_end = cu[b + 1], kv_len = lens[b];
  if constexpr (!ORDERED) asm volatile("" : "+s"(q_start), "+s"(q_end), "+s"(kv_len));  // (asked for together)
  bool any_long = true;
  if constexpr (ORDERED) {
    const int keys = (int)table_keys;
    const bool found = a.batch <= 64    ? request_of_rank<1>(a, b, keys, b, kv_len, any_long)
                       : a.batch <= 128 ? request_of_rank<2>(a, b, keys, b, kv_len, any_long)
                                        : request_of_rank<4>(a, b, keys, b, kv_len, any_long);
    if (found) {
      q_start = cu[b];
      q_end = cu[b + 1];
    }
    any_long = any_long || keys < kDecodeWideTable;
  } else if (STREAMS > kDecodeWaves && kv_len < kDecodeShortKeys && table_keys >= kDecodeWideTable) {
    any_long = false;
    for (int r = (int)threadIdx.x & 63; r < a.batch; r += 64) any_long = any_long || a.kv_lens[r] >= kDecodeShortKeys;
    any_long = __builtin_amdgcn_ballot_w64(any_long) != 0;
  }
  // Eight streams are for long contexts, and the host knows only that the table allows them: a batch without one has four, and
  // where there are eight waves half of them leave, and the unit has room for a second workgroup (300 requests of at most 407
  // tokens under a table of 32 768 keys, one KV head).  In the order of the batch only workgroups of short contexts look for a
  // long one, and in either order only a table that could be wider than the contexts counts for nothing (125 of 128 .. 1800
  // tokens under a tight one 42.4 us, looking 43.2).
  const int streams = STREAMS > kDecodeWaves && !any_long ? kDecodeWaves : STREAMS;
  if (WAVES > streams && __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) >= streams) return;
  if (kv_len > table_keys) kv_len = (int)table_keys;
  run_decode<D, STREAMS / WAVES>(a, s_decode, WAVES < streams ? WAVES : streams, streams, b, kv_head, q_start, q_end - q_start, kv_len, split, (int)threadIdx.x);
#else
  (void)a;
#endif
}

}  // namespace paged
}  // namespace hydra
