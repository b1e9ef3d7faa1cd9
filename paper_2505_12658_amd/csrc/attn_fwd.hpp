// Fused packed variable-length attention forward for gfx950 (MI355X).
//
// One workgroup (4 wavefronts of 256 registers each) runs one work-list item: up to four "wave
// tiles" that share a sequence and a KV head.  A wave tile is 32 consecutive query tokens of one
// query head.  K/V tiles of 64 keys stream global -> LDS with direct-to-LDS 128-bit loads into
// rings of two tiles (a tile is loaded while the previous one is consumed) and are shared by the
// four waves.
//
// The kernel is persistent: two workgroups per compute unit (two waves per SIMD, half of the
// LDS each), each pulling items from the queue of the accelerator die (XCD) it runs on.  The
// prepass puts all items of one (sequence, KV head) into the same queue, next to each other, so
// the workgroups that stream the same K/V rows run on the same die at about the same time and
// share them through that die's L2.  The two workgroups of a compute unit work on different
// items: while one loads Q, stores O or waits at a barrier, the other one's matrix instructions
// fill the SIMDs.
//
// Each wave walks its keys in blocks of 32 and software-pipelines three stages, so that the
// matrix pipe and the vector ALU work side by side also within the wave: while the VALU does the
// softmax of block j, the MFMAs issued between its instructions compute S(j+1) = K(j+1) Q^T and
// O += V(j-1)^T P(j-1).
//
// Per wave and key block (scores kept transposed so that no cross-lane movement is needed between
// the two contractions):
//   S^T[key, query] = K_tile * Q^T        v_mfma_f32_32x32x16_bf16, A = K from LDS, B = Q in registers
//   online softmax over keys: each lane owns one query column and 16 keys per 32-key block, the
//   other 16 live in lane ^ 32 (one v_permlane32_swap per row maximum; row sums are merged once,
//   in the epilogue)
//   O^T[c, query] += V_tile^T * P^T       A = V^T via ds_read_b64_tr_b16 from the row-major V tile,
//                                         B = P, which is exactly the register layout S^T came out in
// The operation is scaled-dot-product attention as costed in the paper's Table 2
// (Attention/encode, Attention/prefill); causal tiles above the diagonal are never loaded.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "attn_careful.hpp"
#include "attn_tiles.hpp"
#include "wave_ops.hpp"

#include "find_unit.hpp"

namespace hydra {

// TEAMS: sets of rings, one for each team of waves that works on a part of an item's keys.
template <int D, int TEAMS = 1, int STAGE_ROWS = 0>
struct TileGeom : RowGeom<D> {
  using RowGeom<D>::kTileBytes;
  // K tiles and V tiles each live in a ring of kRing LDS tiles; loads run kRing - 1 tiles ahead of use
  // (a tile's slot is free again after the barrier that ends the iteration consuming it)
  static constexpr int kRing = 2;
  static constexpr int kPrefetch = kRing - 1;
  // D = 80: the third 32-column block of P V has 16 columns to spare.  The lanes that feed them read bf16 ones
  // from a constant area instead of the V tile, so the matrix unit delivers the softmax row sums in output
  // columns 80..95 and the vector unit does not have to add them up (16 additions per key block and wave).
  // The area covers every offset a V fragment read adds to its lane address (key block, step); the two ring slots have an
  // address register each for that block, so that the area is one tile long and three workgroups fit a compute unit's LDS.
  static constexpr bool kSumsFromMatrixUnit = D == 80;
  static constexpr int kOnesBytes = kSumsFromMatrixUnit ? 9 * 1024 : 0;
  static constexpr int kTeamBytes = 2 * kRing * kTileBytes;         // K ring, V ring
  static constexpr int kOnesAt = TEAMS * kTeamBytes + 64;           // (+ slack behind the last V tile)
  static constexpr int kSumsAt = kOnesAt + kOnesBytes;              // the teams' references and sums, 512 bytes per wave tile
  static constexpr int kTeamSums = kWavesPerItem / TEAMS * 512;
  static constexpr int kSumsBytes = TEAMS > 1 ? TEAMS * kTeamSums : 0;
  static constexpr int kQueriesAt = (kSumsAt + kSumsBytes + 1023) / 1024 * 1024;  // STAGE_ROWS rows of Q
  static constexpr int kLdsBytes = STAGE_ROWS > 0 ? kQueriesAt + STAGE_ROWS * RowGeom<D>::kRowBytes : kSumsAt + kSumsBytes;
};

// Everything below uses gfx950-only types and builtins, so the host pass of hipcc only sees the
// kernel's declaration (it still emits the launch stub).
#if defined(__HIP_DEVICE_COMPILE__)
// Loads of one 64-row K or V tile, global -> LDS, 16 bytes per lane, through a buffer resource
// that covers exactly the rows of this sequence and KV head: rows past the end of the sequence are out
// of range and arrive as zeros (they are masked later; zeros keep V finite).  The descriptor and the
// per-lane offset are fixed for the whole item; the tile advances through the instruction's scalar
// offset, which the hardware's range check takes into account (a scalar offset beyond the end of the
// buffer puts every lane out of range).
//
// The load is issued from inline assembly on purpose: when the compiler knows that vector-memory
// loads write LDS, it makes every later LDS read wait for ALL outstanding loads (vmcnt 0), which
// would serialise the prefetch ring with the compute.  Completion is tracked by hand instead:
// every wave waits for ALL of its outstanding loads (wait_all_loads) at the end of the iteration
// before the one that reads them, followed by the workgroup barrier.  Nothing relies on the order
// in which direct-to-LDS loads complete: a load that misses to HBM was observed to land after a
// younger one that hit in L2.
// WAVES: how many waves share a tile's loads; wave w of them issues loads w, w + WAVES, ...
template <int D, int WAVES = kWavesPerItem>
struct TileLoader {
  using G = TileGeom<D>;
  static constexpr int kPerWave = (G::kLoadInstr + WAVES - 1) / WAVES;
  // Where kPeriod of a wave's loads cover a whole multiple of 16 rows, lane offsets of loads kPeriod apart
  // differ by a constant (the swizzle repeats), which also goes into the scalar offset:
  // kPeriod offset registers instead of kPerWave.
  static constexpr int repeats_after(int loads) { return (loads * WAVES * 64) % (16 * G::kChunks) == 0 || loads >= kPerWave ? loads : repeats_after(loads + 1); }
  static constexpr int kPeriod = repeats_after(1);
  static constexpr bool kUniformStep = kPeriod == 1;
  static constexpr int kOffsets = kPeriod;
  u32x4_t rsrc;                 // the sequence's rows of this KV head, from the first row to the end of the last
  uint32_t tile_off;            // bytes from the first row of the sequence to the first row of the next tile
  uint32_t tile_stride;         // bytes between first rows of consecutive tiles
  uint32_t lane_off[kOffsets];  // bytes from the first row of a tile
  uint32_t step_bytes;          // bytes between the rows of loads of this wave that are kPeriod apart
  int wave;

  template <bool IS_V>
  __device__ __forceinline__ void init(const uint16_t* base, int64_t stride, int64_t seq_start, int seq_len, int kv_head, int wave_, int lane) {
    wave = wave_;
    __builtin_assume(wave >= 0 && wave < WAVES);
    const uint32_t row_bytes = (uint32_t)(stride * 2);
    const uint64_t first_row = (uint64_t)(uintptr_t)(base + seq_start * stride + kv_head * D);
    rsrc[0] = __builtin_amdgcn_readfirstlane((uint32_t)first_row);
    rsrc[1] = __builtin_amdgcn_readfirstlane((uint32_t)(first_row >> 32) & 0xffffu);
    rsrc[2] = __builtin_amdgcn_readfirstlane((uint32_t)(((int64_t)(seq_len - 1) * stride + D) * 2));
    rsrc[3] = 0x00020000u;
    tile_off = 0;
    tile_stride = __builtin_amdgcn_readfirstlane((uint32_t)kKvTileRows * row_bytes);
    step_bytes = __builtin_amdgcn_readfirstlane((uint32_t)(kPeriod * WAVES * 64 / G::kChunks) * row_bytes);
#pragma unroll
    for (int u = 0; u < kOffsets; ++u) {
      const int flat = (wave + WAVES * u) * 64 + lane;
      const int row = flat / G::kChunks, phys = flat % G::kChunks;
      const int chunk = IS_V ? v_swizzle<D>(row, phys) : k_swizzle<D>(row, phys);
      lane_off[u] = (uint32_t)row * row_bytes + chunk * 16;
    }
  }
  // Issues load u (0 .. kPerWave - 1) of this wave's share of the next tile; lds_dst: LDS byte address
  // of the tile's ring slot.
  __device__ __forceinline__ void issue_piece(int u, uint32_t lds_dst) const {
    const int instr = wave + WAVES * u;
    if (instr < G::kLoadInstr) {
      // (m0 is reserved: the compiler only ever sets it immediately before an instruction of its own that reads it)
      const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_dst + instr * 1024);
      const uint32_t soff = __builtin_amdgcn_readfirstlane(tile_off + (uint32_t)(u / kPeriod) * step_bytes);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                   :
                   : "s"(m0), "v"(lane_off[u % kPeriod]), "s"(rsrc), "s"(soff));
    }
  }
  // Issues all of this wave's loads of the next tile at once and moves on to the tile after it.
  __device__ __forceinline__ void issue_next(uint32_t lds_dst) {
#pragma unroll
    for (int u = 0; u < kPerWave; ++u) issue_piece(u, lds_dst);
    tile_off += tile_stride;
  }
};

// Waits until none of this wave's vector-memory operations is in flight.
__device__ __forceinline__ void wait_all_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }


// ---- matrix instructions -------------------------------------------------------------------
// With 256 registers per wave the kernel uses no accumulation registers at all (the compiler
// splits the budget in two halves as soon as one is needed), so scores and output accumulators
// live in ordinary registers, where the softmax and the epilogue read them directly.
// O += V^T P goes through the compiler's builtin, which inserts the wait states the readers of the
// result need.  S = K Q^T is written as inline assembly: measured faster at head_dim 128 (the
// compiler pads every builtin with its own wait states and is freer to move it).  The compiler does
// not see these as matrix instructions, so
//   - s_results_to_valu() supplies the wait states between the last of them and the first reader of
//     S where no other matrix instruction follows (inside the pipeline steps the trailing PV
//     instructions cover them);
//   - an output that nobody reads must still be kept reserved until the instruction has retired
//     (the compiler takes an assembly statement's outputs as written the moment it issues).
typedef __attribute__((ext_vector_type(4))) uint32_t qreg_t;

// O += A(vf) * B(pf)
__device__ __forceinline__ void mfma_pv(f32x16_t& O, const bf16x8_t& vf, const bf16x8_t& pf) {
  O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf, O, 0, 0, 0);
}
// S = A(kf) * B(q), then S += A(kf) * B(q)
__device__ __forceinline__ void mfma_qk_zero(f32x16_t& S, const bf16x8_t& kf, const qreg_t& q) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(S) : "v"(kf), "v"(q));
}
__device__ __forceinline__ void mfma_qk_acc(f32x16_t& S, const bf16x8_t& kf, const qreg_t& q) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(S) : "v"(kf), "v"(q));
}
// Wait states after the last QK matrix instruction, before anything else touches S.
__device__ __forceinline__ void s_results_to_valu(f32x16_t (&S)[1]) { asm volatile("s_nop 15\n\ts_nop 3" : "+v"(S[0])); }
__device__ __forceinline__ void s_results_to_valu(f32x16_t (&S)[2]) { asm volatile("s_nop 15\n\ts_nop 3" : "+v"(S[0]), "+v"(S[1])); }

#endif  // __HIP_DEVICE_COMPILE__

// Scheduling hints: keep the listed instruction classes in this order inside the current region.
#define HYDRA_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// How the items of a call are shared out.  Workgroup id w belongs to die w % 8 (the hardware deals ids to the dies
// round-robin: measured, always; nothing but locality depends on it) and is number w / 8 there.  The first entries of a
// queue go to the die's workgroups by their number, without an atomic; the rest are claimed one by one from the queue's
// head.  When a die's queue has run out, its workgroups look at the other dies' heads, all at once, and claim from one
// that has entries left.
// What this avoids: a few hundred atomics on one address take tens of microseconds, from all dies together, and the end
// of a kernel is where all workgroups would meet.  (It was: every workgroup made one failing claim on every queue, one
// round trip after the other, and the last failing claim on a queue put its head back to zero.  For one image of 577
// tokens that was 6 - 8 us of 18.7; polling all heads with claims at once made every batch 10 - 30 us longer.)
//
// Before the kernel ends the heads have to be zero again for the next call on the same work list (the next layer of
// the same batch).  The last workgroup of a die to leave is known from a count per die, and the last die from a count of
// dies, so no address sees more than a die's workgroups; the last of all clears everything.  Where no queue is longer
// than its die's workgroups are many, no head is ever touched and nothing is counted.

// Workgroups of die y in a grid of n.
__device__ __forceinline__ int queue_wgs(int y, int n) { return (n - y + kXcds - 1) / kXcds; }

// The claimed part of queue y: entries past those that belong to the die's workgroups.
__device__ __forceinline__ int claimable(const WorkControl* ctrl, int y) {
  return ctrl->xcd_start[y + 1] - ctrl->xcd_start[y] - queue_wgs(y, (int)gridDim.x);
}

// An item of another die's queue, for a workgroup whose own has run out.  Called by all lanes of ONE wave.  Returns the
// list index, or -1 when all queues are empty.  Heads only grow, so a queue seen empty stays so: every round either
// returns an item or leaves fewer queues to look at.
__device__ __forceinline__ int steal_item(WorkControl* ctrl, int own, int first) {
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));  // (keeps what follows from the lane number out of the hot loop's registers)
  uint32_t open = 0xffu & ~(1u << own);
  while (open != 0) {
    bool left = false;
    if (lane < kXcds && (open >> lane & 1)) {
      const int n = claimable(ctrl, lane);
      left = n > 0 && __hip_atomic_load(&ctrl->queue_head[lane * kHeadStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n;
    }
    open = (uint32_t)__builtin_amdgcn_ballot_w64(left);
    if (open == 0) break;
    int y = own;
    for (int k = 0; k < kXcds - 1; ++k) {  // (a different neighbour first for different workgroups)
      y = (own + 1 + (first + k) % (kXcds - 1)) & (kXcds - 1);
      if (open >> y & 1) break;
    }
    const int n = claimable(ctrl, y);
    int pos = 0;
    if (lane == 0) pos = atomicAdd(&ctrl->queue_head[y * kHeadStride], 1);
    pos = __builtin_amdgcn_readfirstlane(pos);
    if (pos < n) return ctrl->xcd_start[y + 1] - n + pos;
    open &= ~(1u << y);
  }
  return -1;
}

// The last thing a workgroup does in a call that claims (one thread; its claims have returned).
__device__ __forceinline__ void leave(WorkControl* ctrl) {
  const int n = (int)gridDim.x, die = (int)blockIdx.x % kXcds, dies = n < kXcds ? n : kXcds;
  if (atomicAdd(&ctrl->queue_head[die * kHeadStride + kLeftAt], 1) != queue_wgs(die, n) - 1) return;
  if (atomicAdd(&ctrl->queues_left, 1) != dies - 1) return;
  for (int y = 0; y < kXcds; ++y) {
    atomicExch(&ctrl->queue_head[y * kHeadStride], 0);
    atomicExch(&ctrl->queue_head[y * kHeadStride + kLeftAt], 0);
  }
  atomicExch(&ctrl->queues_left, 0);
}

constexpr int kKeyBlock = 32;         // keys per pipeline step

template <int N>
using NextRB = std::integral_constant<int, N>;  // key block the following step reads in the same tiles (-1: none)

// LDS fragments are requested this many work units (one K or V^T fragment and the matrix instructions it feeds)
// ahead of their use.  Each unit of distance keeps one more K and one more V^T fragment (8 registers) in flight.
// Two in kernels built for two waves per SIMD (three: no faster; one: head_dim 128, 558 tokens 14.8 -> 15.1 us, larger batches level;
// head_dim 80 with one workgroup per compute unit asked for, 48 requests with 28 / 4 heads 210.8 -> 213.9, 65 536 tokens in images of
// 256 .. 4096 with 16 heads 1059 -> 1064; head_dim 64 from cache pages level).  One in kernels built for three, whose waves cover the
// LDS latency for each other: the same images with a workgroup per item 796 -> 791, 32 images of 577 tokens with 16 heads of 64
// 62.6 -> 62.3, one image equal (but 180.4 instead of 178.8 where one workgroup per unit is asked for, 48 requests with 28 / 4 heads of 64).
template <int WAVES_PER_SIMD>
constexpr int kFragsAhead = WAVES_PER_SIMD >= 3 ? 1 : 2;

#if defined(__HIP_DEVICE_COMPILE__)
// LDS fragments of the first PF QK units and the first PF PV units of a pipeline step.
template <int PF>
struct StepFrags {
  bf16x8_t k[PF], v[PF];
};
#endif
constexpr float kMaxRowSum = 1.0995116e12f;  // 2^40: largest row sum (relative to the reference) the fast kernel accepts


// Where a workgroup's items and their K/V rows come from.  The packed kernel (below) takes items from the work
// list's queues and K/V rows from the packed batch; for small batches a workgroup works its one item out for itself
// (attn_fwd_direct_kernel) and hands it over in its source object; the paged kernel does so as well, with K/V rows
// gathered from cache pages and queries that are the LAST q_len positions of a context of kv_len keys (see
// attn_paged.hpp for that source).
struct PackedSource {
  static constexpr bool kPaged = false, kOneItem = false;
  template <int D, int WAVES>
  using Loader = int;  // (of its loading waves: none)
  static constexpr int kTeams = 1, kTiles = kWavesPerItem;
  static constexpr int kLoaders = 0, kStageRows = 0;
  template <int D>
  static constexpr int kWavesPerSimd = kWorkgroupsPerCu<D>;  // that the kernel is built for
  template <int D>
  struct Gather {};  // (the paged source's K/V gatherer; the packed rows use two TileLoaders)
};
// TEAMS: 2 where the keys of an item are divided between two teams of waves; LOADERS: waves of each team that do nothing but load
// tiles (see attn_fwd_direct_kernel).
template <int TEAMS, int LOADERS>
struct DirectSource {
  static constexpr bool kPaged = false, kOneItem = true;
#if defined(__HIP_DEVICE_COMPILE__)
  template <int D, int WAVES>
  using Loader = TileLoader<D, WAVES>;
#endif
  static constexpr int kTeams = TEAMS, kTiles = kWavesPerItem / TEAMS, kLoaders = LOADERS;
  static constexpr int kStageRows = LOADERS > 0 && kTiles > 2 ? kTiles * kWaveTileRows : 0;
  static constexpr int kThreads = 64 * TEAMS * (kTiles + LOADERS);
  // (what the compiler is told: two teams without loading waves are for calls that leave half of the registers to others)
  static constexpr int kBound = TEAMS == 2 ? 512 : kThreads;
  template <int D>
  static constexpr int kWavesPerSimd = TEAMS == 1 && LOADERS == 0 ? kDirectPerCu<D> : 2;
  template <int D>
  struct Gather {};
  int64_t q_start;   // first token of the sequence
  int q_len;         // its length
  int f0, kv_head;   // first flattened wave tile of the item, KV head
};

#if defined(__HIP_DEVICE_COMPILE__)
// The item loop of a workgroup (4 waves).  smem: TileGeom<D>::kLdsBytes bytes of LDS, 1024-aligned; s_claim: 4
// ints, s_redo: 8 ints of LDS.  Packed source: runs until the queues are empty.  One-item sources: runs the source's
// item and returns whether its row sums left the fast path's range (same value in every thread; the caller then
// recomputes the item with its own careful routine).
template <int D, bool CAUSAL, class Src>
__device__ __forceinline__ bool attn_item_loop(const AttnArgs& a, const Src& src, unsigned char* smem, int* s_claim, int* s_redo) {
  constexpr int TEAMS = Src::kTeams, WT = Src::kTiles;  // teams of WT waves, one per wave tile of the item
  constexpr int kLoaders = Src::kLoaders;               // more waves per team that load its K (one half) and its V tiles (the other)
  using G = TileGeom<D, TEAMS, Src::kStageRows>;
  constexpr int KS = G::kQkSteps;
  constexpr int CC = G::kPvChunks;
  constexpr int ROWB = G::kRowBytes;
  constexpr int NQ = KS;      // QK work units per key block: step s = one K fragment read + 2 MFMAs (qs = 0, 1)
  constexpr int NP = 2 * CC;  // PV work units per key block: (s2, cc) = one V^T fragment + 2 MFMAs
  constexpr int PF = kFragsAhead<Src::template kWavesPerSimd<D>>;
  // LDS: K ring then V ring; tile t of either lives in ring slot t % kRing.
  constexpr int R = G::kRing, PD = G::kPrefetch;
  const int lane_id = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool loader_wave = kLoaders > 0 && wave >= TEAMS * WT;
  const int team = TEAMS == 1 ? 0 : loader_wave ? (wave - TEAMS * WT) / (kLoaders > 0 ? kLoaders : 1) : wave / WT, wave_tile = TEAMS == 1 ? wave : wave % WT;
  const uint32_t lds0 = (uint32_t)(uintptr_t)HYDRA_LDS_PTR(smem);  // LDS byte addresses
  const uint32_t k_ring = lds0 + team * G::kTeamBytes;
  const uint32_t v_ring = k_ring + R * G::kTileBytes;

  const int die = (int)blockIdx.x % kXcds;  // the die this workgroup runs on, whose queue is its own
  // s_redo: an item whose exponentials left the fast path's range: {flag, first token, length, first wave tile, KV
  // head}, posted by the waves that noticed, acted upon by the whole workgroup at the top of its next round.
  if (threadIdx.x == 0) s_redo[0] = 0;
  if constexpr (G::kSumsFromMatrixUnit) {
    static_assert(kKvTileRows * ROWB - 8 * ROWB + 8 <= G::kOnesBytes, "a V fragment read stays inside the ones");
    for (int i = threadIdx.x * 16; i < G::kOnesBytes; i += 64 * TEAMS * (WT + kLoaders) * 16)
      *reinterpret_cast<u32x4_t*>(HYDRA_LDS_BYTE(lds0 + G::kOnesAt + i)) = u32x4_t{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
  }

  // Wave 0 claims the items for the whole workgroup, one round ahead: the claim for the next
  // round is issued at the top of a round, resolved (and the item read) before the hot loop, and
  // posted in LDS after it, so that none of its latency shows.
  auto post_claim = [&](int idx) {  // wave 0: read the item and post it for the next round
    WorkItem it = make_int4(0, 0, 0, 0);
    if (idx >= 0) it = a.items[idx];
    // (used by the whole wave right here, so that the load has completed on every code path that
    // goes on to the hot loop; see the note at pending_claim)
    it.x = __builtin_amdgcn_readfirstlane(it.x);
    it.y = __builtin_amdgcn_readfirstlane(it.y);
    it.z = __builtin_amdgcn_readfirstlane(it.z);
    it.w = __builtin_amdgcn_readfirstlane(it.w);
    if (lane_id == 0) {
      s_claim[0] = it.x;
      s_claim[1] = it.y;
      s_claim[2] = it.z;
      s_claim[3] = it.w;
    }
  };
  int own_claimed_at = 0, own_count = 0;  // the claimed part of the own queue: first entry, entries
  if constexpr (!Src::kOneItem) {
    own_count = claimable(a.ctrl, die);
    own_claimed_at = a.ctrl->xcd_start[die + 1] - own_count;
  }
  // Q: a wave's 32 rows come in with direct-to-LDS loads that cover whole rows (loaded straight
  // into the B-operand register layout, one instruction would touch 32 different rows: one address
  // cycle per row in the memory pipeline), into a private staging area in K-tile layout, and are
  // read back with the lane pattern of the K reads.  Staging area: the V ring, which is idle from
  // an item's last iteration until the barrier before the next item's first key block.  The loads
  // of the NEXT item are issued as soon as the current item's last iteration is over, ahead of the
  // epilogue, so that their latency hides behind it.
  static_assert(WT * kWaveTileRows * ROWB <= R * G::kTileBytes, "the Q tiles of a team's waves fit its V ring");
  constexpr int kRowInstr = kWaveTileRows * G::kChunks / 64;  // 64-lane instructions that cover a 32-row tile
  static_assert(kWaveTileRows * G::kChunks % 64 == 0, "whole instructions");
  // (with waves of their own for the loads the first V tile is on its way at the same time, into slot 0)
  const uint32_t q_stage = (Src::kStageRows > 0 ? lds0 + G::kQueriesAt : lds0 + R * G::kTileBytes + (kLoaders > 0 ? G::kTileBytes : 0)) + wave_tile * (kWaveTileRows * ROWB);
  static_assert(kLoaders == 0 || WT * kWaveTileRows * ROWB <= G::kTileBytes || Src::kStageRows == WT * kWaveTileRows, "... and slot 1");
  auto issue_q_loads = [&](int64_t seq_start, int seq_len, int q0, int head, int lane) {
    const uint64_t base = (uint64_t)(uintptr_t)(a.q + (seq_start + q0) * a.q_stride + head * D);
    const uint32_t q_row_bytes = (uint32_t)(a.q_stride * 2);
    const int rows = seq_len - q0 < kWaveTileRows ? seq_len - q0 : kWaveTileRows;
    u32x4_t rsrc;
    rsrc[0] = __builtin_amdgcn_readfirstlane((uint32_t)base);
    rsrc[1] = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
    rsrc[2] = __builtin_amdgcn_readfirstlane((uint32_t)(rows - 1) * q_row_bytes + D * 2);  // rows past the end arrive as zeros
    rsrc[3] = 0x00020000u;
#pragma unroll
    for (int i = 0; i < (kRowInstr + TEAMS - 1) / TEAMS; ++i) {
      const int instr = i * TEAMS + team;  // (teams share the loads of the rows that they share)
      if (TEAMS > 1 && instr >= kRowInstr) break;
      const int flat = instr * 64 + lane;
      const int row = flat / G::kChunks, phys = flat % G::kChunks;
      const uint32_t off = (uint32_t)row * q_row_bytes + k_swizzle<D>(row, phys) * 16;
      const uint32_t m0 = __builtin_amdgcn_readfirstlane(q_stage + instr * 1024);
      // (nt: Q is read once; marking its lines for early replacement leaves the L2 to the K/V rows that are re-read)
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds" : : "s"(m0), "v"(off), "s"(rsrc));
    }
  };
  bool q_ahead = false;      // the current item's Q loads were issued at the end of the previous round
  bool own_empty = own_count <= 0;  // nothing is left to claim from this die's queue (same value in all waves)
  if constexpr (!Src::kOneItem) {
    if (wave == 0) {
      const int idx = a.ctrl->xcd_start[die] + (int)blockIdx.x / kXcds;
      post_claim(idx < a.ctrl->xcd_start[die + 1] ? idx : -1);
    }
  }

  for (;;) {  // one work item per round
  __syncthreads();
  if constexpr (!Src::kOneItem)
  if (__builtin_expect(__builtin_amdgcn_readfirstlane(s_redo[0]) != 0, 0)) {
    // The previous round's item has to be redone carefully.  Its (wrong) output rows are already stored and are
    // overwritten by the same waves; the loads of the next item's Q, in flight into the V ring, are waited for
    // first (the routine takes both rings as its stages) and issued again afterwards.
    const int64_t r_start = __builtin_amdgcn_readfirstlane(s_redo[1]);
    const int r_len = __builtin_amdgcn_readfirstlane(s_redo[2]);
    const int r_f0 = __builtin_amdgcn_readfirstlane(s_redo[3]);
    const int r_kv = __builtin_amdgcn_readfirstlane(s_redo[4]);
    wait_all_loads();
    __syncthreads();
    if (threadIdx.x == 0) s_redo[0] = 0;
    careful::run_item<D, CAUSAL>(a, r_start, r_len, r_f0, r_kv, k_ring);
    q_ahead = false;
  }
  // Everything derived from the lane number is recomputed in every round (the empty statement hides
  // the value from the optimiser): kept across rounds, dozens of such lane constants would sit in
  // registers through the hot loop, which has none to spare.
  int lane = lane_id;
  asm volatile("" : "+v"(lane));
  __builtin_assume(lane >= 0 && lane < 64);  // (divisions of lane-derived indices by constants become shifts)
  const int m = lane & 31, hf = lane >> 5, sl = lane & 15, grp = (lane >> 4) & 1;
  if constexpr (!Src::kOneItem)
  if (__builtin_amdgcn_readfirstlane(s_claim[1]) == 0) {
    // Nothing left in this die's queue: take an item from another die's queue.  This is done here, with
    // the workgroup idle, and synchronously (two memory round trips), not ahead of time like the claims
    // from the own queue.  Every wave has seen the empty claim before wave 0 overwrites it.
    own_empty = true;
    __syncthreads();
    if (wave == 0) post_claim(steal_item(a.ctrl, die, (int)(blockIdx.x / kXcds)));
    __syncthreads();
  }
  // The item: `seq_len` query rows that start at packed token `seq_start`, and `kv_len` keys; query row i sees
  // keys 0 .. shift + i (causal).  Packed batch: the keys are the sequence's own rows, shift = 0.
  int64_t seq_start;
  int seq_len, f0, kv_head;
  if constexpr (Src::kOneItem) {
    seq_start = src.q_start;
    seq_len = src.q_len;
    f0 = src.f0;
    kv_head = src.kv_head;
  } else {
    seq_start = __builtin_amdgcn_readfirstlane(s_claim[0]);
    seq_len = __builtin_amdgcn_readfirstlane(s_claim[1]);
    f0 = __builtin_amdgcn_readfirstlane(s_claim[2]);
    kv_head = __builtin_amdgcn_readfirstlane(s_claim[3]);
    if (seq_len == 0) break;
  }
  int kv_len_, shift_;
  if constexpr (Src::kPaged) {
    kv_len_ = src.kv_len;
    shift_ = src.kv_len - src.q_len;
  } else {
    kv_len_ = seq_len;
    shift_ = 0;
  }
  const int kv_len = kv_len_, shift = shift_;
  // Thread 0: position claimed in this die's queue for the next round.  (Written as a per-thread
  // condition, and read below by every wave, on purpose: the compiler tracks outstanding memory
  // operations per code path, and an atomic that is "maybe still in flight" on some path into
  // the hot loop makes it wait for ALL loads there, which would undo the tile prefetch.)
  int pending_claim = 0x7fffffff;
  if constexpr (!Src::kOneItem) {
    if (threadIdx.x == 0 && !own_empty) pending_claim = atomicAdd(&a.ctrl->queue_head[die * kHeadStride], 1);
  }
  const int n_tok_tiles = (seq_len + kWaveTileRows - 1) / kWaveTileRows;
  const int n_wave_tiles = n_tok_tiles * a.group;

  // this wave's tile
  int f = f0 + wave_tile;
  const bool active = f < n_wave_tiles;
  if (!active) f = n_wave_tiles - 1;
  // (head_dim 64 and a reciprocal: 32 images of 577 tokens with 16 heads 59.4 -> 59.0 us in a run of its own, within the spread of others; two teams: causal requests of 200 tokens
  // 6.83 -> 6.68, but one image 6.53 -> 6.59; head_dim 128 with four wave tiles, a request of 1000 tokens 16.0 -> 16.3.  One item per
  // workgroup only: over many items the causal kernel of head_dim 64 would spill vector registers for it)
  constexpr bool kByReciprocal = Src::kOneItem && !Src::kPaged && (TEAMS > 1 ? CAUSAL : D == 64);
  auto token_tile = [&](int flat) { return kByReciprocal ? quotient(flat, a.group) : flat / a.group; };
  const int tok_tile = token_tile(f);
  const int head = kv_head * a.group + (f - tok_tile * a.group);
  const int q0 = tok_tile * kWaveTileRows;
  const int f_last = (f0 + WT - 1 < n_wave_tiles ? f0 + WT - 1 : n_wave_tiles - 1);
  // KV tiles (of 64 keys) the workgroup streams
  const int n_kv_tiles = (kv_len + kKvTileRows - 1) / kKvTileRows;
  const int causal_keys = shift + (token_tile(f_last) + 1) * kWaveTileRows;  // keys visible to the item's last query tile
  const int W_all = CAUSAL && causal_keys < kv_len ? (causal_keys + kKvTileRows - 1) / kKvTileRows : n_kv_tiles;
  // ... of which this team takes tiles [first_tile, first_tile + W_own); W: the most that a team takes
  const int W = (W_all + TEAMS - 1) / TEAMS, first_tile = team * W;
  const int W_own = TEAMS == 1 || first_tile + W <= W_all ? W : (first_tile < W_all ? W_all - first_tile : 0);
  const int key_base = first_tile * kKvTileRows;  // blocks, masks and limits count from here
  // key blocks this wave consumes: of the keys [0, kv_end) those of its team's tiles
  const int kv_end = CAUSAL ? (shift + q0 + kWaveTileRows < kv_len ? shift + q0 + kWaveTileRows : kv_len) : kv_len;
  int blocks = (kv_end - key_base + kKeyBlock - 1) / kKeyBlock;
  if constexpr (TEAMS > 1) blocks = blocks < 0 ? 0 : blocks < 2 * W_own ? blocks : 2 * W_own;
  const int NB = active ? blocks : 0;

  // Workgroup iterations: iteration 0 is the prologue (needs K(0)); iteration t >= 1 needs K tile t
  // and V tile t - 1 and runs, per wave, key-block steps 2t - 1 and 2t.  There are W + 1 of them.
  // Load order of the whole item: K(0) V(0) K(1) V(1) ..., each tile issued PD = 1 iteration ahead of
  // its use into the ring slot freed by the barrier that ended the previous iteration; everything
  // issued in iteration t is needed in iteration t + 1, so each iteration ends with a wait for all
  // of the wave's loads and a barrier.
  static_assert(PD == 1 && R == 2, "the iteration-end wait is for everything in flight");
  if constexpr (kLoaders > 0) {
    if (loader_wave) {
      // K tile 0 is the computing waves' own; these start with K tile 1 and V tile 0, ahead of the item's first barrier.
      constexpr int kEach = kLoaders / 2;
      const int number = (wave - TEAMS * WT) % kLoaders;
      const bool is_v = number >= kEach;
      const int ahead = is_v ? 0 : 1;  // iteration t loads K tile t + 1, V tile t
      const uint32_t ring = is_v ? v_ring : k_ring;
      typename Src::template Loader<D, kEach> loader;
      if constexpr (Src::kPaged) {  // (K tile 0 as well)
        loader.init(src, is_v, kv_head, number % kEach, lane);
        if (!is_v) {
          loader.issue_next(ring);
          wait_all_loads();
        }
      } else {
        if (is_v) loader.template init<true>(a.v, a.v_stride, seq_start, seq_len, kv_head, number % kEach, lane);
        else loader.template init<false>(a.k, a.k_stride, seq_start, seq_len, kv_head, number % kEach, lane);
        loader.tile_off = (first_tile + ahead) * loader.tile_stride;
      }
      if (ahead < W_own) loader.issue_next(ring + ahead * G::kTileBytes);
      __syncthreads();  // (the one behind K tile 0 and Q)
      wait_all_loads();
      __syncthreads();
      for (int t = 1; t <= W; ++t) {
        if (t + ahead < W_own) loader.issue_next(ring + ((t + ahead) % R) * G::kTileBytes);
        wait_all_loads();
        __syncthreads();
      }
      if constexpr (TEAMS > 1) __syncthreads();  // (the one between the teams' results and their sum)
      break;
    }
  }
  // The loaders of the two sources have different shapes: two independent tile loaders for the packed rows, one
  // gatherer for the pages (a V tile comes from the pages its K tile came from one iteration earlier).
  std::conditional_t<Src::kPaged, int, TileLoader<D, WT>> k_loader, v_loader;
  typename Src::template Gather<D> gather;
  if constexpr (Src::kPaged) {
    if constexpr (kLoaders == 0) gather.init(src, kv_head, wave, lane);
  } else {
    k_loader.template init<false>(a.k, a.k_stride, seq_start, seq_len, kv_head, wave_tile, lane);
    v_loader.template init<true>(a.v, a.v_stride, seq_start, seq_len, kv_head, wave_tile, lane);
    if constexpr (TEAMS > 1) {
      k_loader.tile_off = first_tile * k_loader.tile_stride;
      v_loader.tile_off = first_tile * v_loader.tile_stride;
    }
  }
  // after the issue of iteration t, tile loads 0 .. 2(t+PD) are out; iteration t needs 0 .. 2t
  auto issue_loads = [&](int t) {
    if constexpr (Src::kPaged) {
      if constexpr (kLoaders == 0) gather.issue(t - 1 + PD < W, v_ring + ((t - 1 + PD) % R) * G::kTileBytes, t + PD < W, k_ring + ((t + PD) % R) * G::kTileBytes);
    } else {
      if constexpr (kLoaders > 0) return;
      if (t - 1 + PD < W_own) v_loader.issue_next(v_ring + ((t - 1 + PD) % R) * G::kTileBytes);
      if (t + PD < W_own) k_loader.issue_next(k_ring + ((t + PD) % R) * G::kTileBytes);
    }
  };
  if constexpr (Src::kPaged) {
    if constexpr (kLoaders == 0) gather.issue_first(k_ring);
  } else {
    k_loader.issue_next(k_ring);
  }

  if (!q_ahead) issue_q_loads(seq_start, seq_len, q0, head, lane);
  // Q fragments (B operand): lane (m, hf) holds query row q0 + 32*qs + m, columns hf*D/2 + 8*s .. +7, as
  // they come from memory.  The softmax scale is applied to the scores in fp32 (see softmax_half).
  const float c = a.scale_log2;
  qreg_t qf[QS][KS];
  int q_lim[QS];  // largest visible key index for this lane's query of sub-tile qs
  wait_all_loads();  // Q (and this wave's part of K(0)) has landed
  if constexpr (TEAMS > 1) __syncthreads();  // ... and the other waves' parts
#pragma unroll
  for (int qs = 0; qs < QS; ++qs) {
    int row = q0 + 32 * qs + m;
    row = row < seq_len ? row : seq_len - 1;
    q_lim[qs] = (CAUSAL ? shift + row : kv_len - 1) - key_base;
#pragma unroll
    for (int s = 0; s < KS; ++s)
      qf[qs][s] = *reinterpret_cast<const qreg_t*>(HYDRA_LDS_BYTE(q_stage + (32 * qs + m) * ROWB + k_swizzle<D>(32 * qs + m, KS * hf + s) * 16));
  }

  // LDS read addresses: lane part + ring slot of the iteration's K tile / V tile; the key block
  // inside the tile and the step are immediates.  Advanced once per iteration.
  uint32_t k_addr[KS], v_addr[CC];
  uint32_t v_last1 = 0;  // kSumsFromMatrixUnit: the last block's address for ring slot 1 (v_addr: slot 0)
  const uint32_t lds_base = k_ring;
#pragma unroll
  for (int s = 0; s < KS; ++s) k_addr[s] = lds_base + m * ROWB + k_swizzle<D>(m, KS * hf + s) * 16;  // K tile 0
  {
    const int r = 4 * hf + (sl >> 2);
#pragma unroll
    for (int cc = 0; cc < CC; ++cc) {
      const int chunk = 4 * cc + 2 * grp + ((sl & 3) >> 1);
      v_addr[cc] = lds_base + R * G::kTileBytes + r * ROWB + v_swizzle<D>(r, chunk) * 16 + 8 * (sl & 1);  // V ring, slot 0
    }
    if constexpr (G::kSumsFromMatrixUnit) {
      // columns 80..95 (the upper 16 of the last block): ones, whichever ring slot is read
      v_last1 = grp == 1 ? lds0 + G::kOnesAt : v_addr[CC - 1] + G::kTileBytes;
      if (grp == 1) v_addr[CC - 1] = lds0 + G::kOnesAt;
    }
  }
  // The address registers point at slot 0 of both rings from here through the hot loop, whose reads name
  // their ring slot in the instruction offset (two iterations per trip: the slots are constants there).  The
  // iterations after the hot loop move the registers instead (position_addresses) and read at offset 0.
  int k_pos = 0, v_pos = 0;  // where the registers point: bytes from slot 0
  auto position_addresses = [&](int t) {  // to K tile t, V tile t - 1 (t >= 1)
    const int k_new = (t % R) * G::kTileBytes, v_new = ((t - 1) % R) * G::kTileBytes;
    const int dk = k_new - k_pos, dv = v_new - v_pos;
#pragma unroll
    for (int s = 0; s < KS; ++s) k_addr[s] += dk;
#pragma unroll
    for (int cc = 0; cc < CC; ++cc) v_addr[cc] += G::kSumsFromMatrixUnit && cc == CC - 1 && grp == 1 ? 0 : dv;
    k_pos = k_new;
    v_pos = v_new;
  };

  f32x16_t o_acc[QS][CC];
#pragma unroll
  for (int qs = 0; qs < QS; ++qs)
#pragma unroll
    for (int cc = 0; cc < CC; ++cc)
#pragma unroll
      for (int r = 0; r < 16; ++r) o_acc[qs][cc][r] = 0.f;
  // Softmax reference: the row maximum over key block 0, kept for the whole row, so O never has to be
  // rescaled inside the loop.  The matrix unit returns raw scores <q, k>; scale and reference go in with
  // one fused multiply-add per score, p = exp2(score * c - reference * c), c = softmax_scale * log2 e.
  // That is exact as long as the exponentials stay far from the end of the fp32
  // range: a wave whose row sums (which bound every single exponential) exceed kMaxRowSum, or are
  // not finite, posts its work item for the careful routine (attn_careful.hpp), which rescales at every tile
  // and which the workgroup runs at the top of its next round.  (bf16 activations lead the first block's maximum by a few
  // powers of two at most.  Below the limit the unnormalised output is bounded by 2^40 times the sum
  // of |V| over the keys, so it cannot overflow for |V| up to 10^20.)
  float nref[QS];        // -reference * c of this lane's query row
  float row_sum[QS];     // this lane's half of the row sum
#pragma unroll
  for (int qs = 0; qs < QS; ++qs) {
    row_sum[qs] = 0.f;
    if constexpr (TEAMS > 1) nref[qs] = -kLowest;  // (a wave tile none of whose keys are this team's)
  }

  // LDS fragment reads; rb = key block inside the tile the address registers point at.
  // (koff / voff: ring slot of the tile, in bytes; constants where it matters, so they end up in the instruction)
  auto load_k_frag = [&](int rb, int s, int koff) -> bf16x8_t {
    return *reinterpret_cast<const bf16x8_t*>(HYDRA_LDS_BYTE(k_addr[s] + koff + rb * kKeyBlock * ROWB));
  };
  // PV unit u = (s2, cc): the V^T fragment of 16 keys x 32 columns
  auto load_v_frag = [&](int rb, int u, int voff) -> bf16x8_t {
    const int cc = u % CC, s2 = u / CC;
    const uint32_t tile = G::kSumsFromMatrixUnit && cc == CC - 1 ? (voff == 0 ? v_addr[cc] : v_last1) : v_addr[cc] + voff;
    const uint32_t at = tile + rb * kKeyBlock * ROWB + s2 * 16 * ROWB;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)HYDRA_LDS_BYTE(at));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)HYDRA_LDS_BYTE(at + 8 * ROWB));
    typedef __attribute__((ext_vector_type(8))) short s16x8_t;
    const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, both);
  };

  // Mask of key block j (only blocks that reach past a query's limit need it).
  auto apply_mask = [&](int j, f32x16_t(&S)[QS]) {
    const int key0 = j * kKeyBlock;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = key0 + 8 * (r >> 2) + 4 * hf + (r & 3);
#pragma unroll
      for (int qs = 0; qs < QS; ++qs)
        if (key > q_lim[qs]) S[qs][r] = -__builtin_inff();
    }
  };
  const int min_lim = (CAUSAL ? shift + q0 : kv_len - 1) - key_base;
  auto needs_mask = [&](int j) { return j * kKeyBlock + kKeyBlock - 1 > min_lim; };

  // Softmax of a key block whose S holds the raw scores, in 16 * QS halves of an element pair (pair = half / 2:
  // sub-tile pair / 8, registers 2 * (pair % 8), +1): scale and reference, exponentials, row sum, rounding to
  // bf16.  A half is one exponential (a quarter-rate instruction) and two or three full-rate ones, about as long
  // as one matrix instruction takes, so that a wave alone on its SIMD can put one behind every matrix
  // instruction and keep the matrix pipe fed; whole pairs behind every other instruction left it idle a third
  // of the time.  The first half leaves its results in the two S registers.
  // (The sum is two plain adds on purpose: the 2-element dot-product instruction would halve them,
  // but it runs in the matrix pipe and stalls behind the matrix instructions it is meant to hide in.)
  auto softmax_half = [&](int half, f32x16_t(&Sc)[QS], bf16x8_t(&Pc)[QS][2], float(&psum)[QS]) __attribute__((always_inline)) {
    const int pair = half / 2, qs = pair / 8, r = 2 * (pair % 8);
    if (half % 2 == 0) {
      float e0 = fast_exp2(__builtin_fmaf(Sc[qs][r], c, nref[qs]));
      float x1 = __builtin_fmaf(Sc[qs][r + 1], c, nref[qs]);
      asm volatile("" : "+v"(e0), "+v"(x1));  // keeps this half's work where it is written
      Sc[qs][r] = e0;
      Sc[qs][r + 1] = x1;
    } else {
      float x1 = Sc[qs][r + 1];
      asm volatile("" : "+v"(x1));  // the second exponential stays behind the matrix instruction it is meant to follow
      f32x2_t pr = {Sc[qs][r], fast_exp2(x1)};
      if constexpr (!G::kSumsFromMatrixUnit) {
        psum[qs] += pr[0];
        psum[qs] += pr[1];
      }
      uint32_t packed = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2_t));
      asm volatile("" : "+v"(packed), "+v"(psum[qs]));
      const bf16x2_t pk = __builtin_bit_cast(bf16x2_t, packed);
      Pc[qs][r / 8][r % 8] = pk[0];
      Pc[qs][r / 8][r % 8 + 1] = pk[1];
    }
  };

  // One pipeline step for key block j >= 1 of this wave.  KRB / VRB: key block of K(j+1) and of
  // V(j-1) inside the tiles the address registers point at.
  //   VALU : softmax of S(j) (in Sc) -> P(j) (into Pc)
  //   MFMA : O += V(j-1)^T P(j-1) (P in Pp) and S(j+1) = K(j+1) Q^T (into Sn)
  // One matrix instruction, then the share of vector work that fits in its shadow, and so on:
  // the wave issues in order, so this is what lets the two pipes run side by side.
  constexpr int NM = QS * (NQ + NP);  // matrix instructions per step
  constexpr int NV = 16 * QS;         // vector work pieces per step: the halves of 8 element pairs per sub-tile
  // qk_tag: false for a wave's last step, which has no S(j+1) to compute.
  // The LDS fragments of a step's first PF QK units and first PF PV units are fetched ahead of the
  // step (the LDS answers after several matrix instructions; fetched at the top of the step that
  // latency would be exposed once per step): `fr` holds them on entry.  next_tag >= 0: the step that
  // follows reads key block next_tag of the SAME tiles, and this step's last units fetch its first
  // fragments into `fr` (next_qk_tag: whether it has QK units).  next_tag < 0: nothing is fetched ahead
  // (the next tiles are only complete after the iteration's barrier; the caller fetches them then).
  auto block_step = [&](auto rb_tag, auto qk_tag, auto next_tag, auto next_qk_tag, int j, f32x16_t(&Sc)[QS], f32x16_t(&Sn)[QS],
                        const bf16x8_t(&Pp)[QS][2], bf16x8_t(&Pc)[QS][2], StepFrags<PF>& fr, int koff, int voff) __attribute__((always_inline)) {
    constexpr int RB = decltype(rb_tag)::value;  // step 2t-1: K(2t), V(2t-2) -> 0; step 2t: K(2t+1), V(2t-1) -> 1
    constexpr bool QK = decltype(qk_tag)::value;
    constexpr int NEXT_RB = decltype(next_tag)::value;
    constexpr bool NEXT_QK = decltype(next_qk_tag)::value;
    constexpr int NMS = QK ? NM : QS * NP;       // matrix instructions of this step
    if (needs_mask(j)) apply_mask(j, Sc);
    // vector work piece i of this step: half a softmax pair
    auto valu_piece = [&](int i) __attribute__((always_inline)) { softmax_half(i, Sc, Pc, row_sum); };
    // kq[i] / vq[i]: fragment of the QK / PV unit i places ahead of the one that runs next
    bf16x8_t kq[PF], vq[PF], k_new, v_new;
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      kq[i] = fr.k[i];
      vq[i] = fr.v[i];
    }
    int ms = 0;  // matrix-instruction index inside the step
    auto shadow = [&](int ms_done) __attribute__((always_inline)) {
      // vector pieces [ms*NV/NMS, (ms+1)*NV/NMS) run behind matrix instruction ms
#pragma unroll
      for (int i = ms_done * NV / NMS; i < (ms_done + 1) * NV / NMS; ++i) valu_piece(i);
      HYDRA_SCHED_FENCE();
    };
    // Order: QK unit 0, then alternately QK unit u and PV unit u - 1; the step ends with (at least)
    // two PV units, whose matrix instructions cover the wait states of the last QK result.
    static_assert(NP >= NQ && NP >= 2, "the step must end with two PV units");
    static_assert(NQ >= PF && NP >= PF, "a step's last units fetch the next step's first fragments");
#pragma unroll
    for (int u = 0; u <= NP; ++u) {
      if (QK && u < NQ) {
        const bool k_more = u + PF < NQ || (NEXT_RB >= 0 && NEXT_QK);
        if (u + PF < NQ) k_new = load_k_frag(RB, u + PF, koff);
        else if (NEXT_RB >= 0 && NEXT_QK) k_new = load_k_frag(NEXT_RB, u + PF - NQ, koff);
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) {
          if (u == 0) mfma_qk_zero(Sn[qs], kq[0], qf[qs][u]); else mfma_qk_acc(Sn[qs], kq[0], qf[qs][u]);
          shadow(ms++);
        }
#pragma unroll
        for (int i = 0; i + 1 < PF; ++i) kq[i] = kq[i + 1];
        if (k_more) kq[PF - 1] = k_new;
      }
      if (u >= 1) {
        const int pu = u - 1;
        const bool v_more = pu + PF < NP || NEXT_RB >= 0;
        if (pu + PF < NP) v_new = load_v_frag(RB, pu + PF, voff);
        else if (NEXT_RB >= 0) v_new = load_v_frag(NEXT_RB, pu + PF - NP, voff);
        const int cc = pu % CC, s2 = pu / CC;
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) {
          mfma_pv(o_acc[qs][cc], vq[0], Pp[qs][s2]);
          shadow(ms++);
        }
#pragma unroll
        for (int i = 0; i + 1 < PF; ++i) vq[i] = vq[i + 1];
        if (v_more) vq[PF - 1] = v_new;
      }
    }
    if constexpr (NEXT_RB >= 0) {
#pragma unroll
      for (int i = 0; i < PF; ++i) {
        fr.k[i] = kq[i];
        fr.v[i] = vq[i];
      }
    }
  };
  // first fragments of a step that reads key block rb of the tiles the address registers point at
  auto fetch_step_frags = [&](int rb, bool with_qk, StepFrags<PF>& fr, int koff, int voff) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      fr.v[i] = load_v_frag(rb, i, voff);
      if (with_qk) fr.k[i] = load_k_frag(rb, i, koff);
    }
  };

  // PV only (after this wave's last softmax): O += V^T P for key block rb of the V tile in reach
  auto pv_only = [&](int rb, const bf16x8_t(&Pp)[QS][2]) __attribute__((always_inline)) {
    // (all fragments are requested before the first matrix instruction: left to itself the compiler
    // fetches each one right before its use and the wave sits through the LDS latency NP times)
    bf16x8_t vf[NP];
#pragma unroll
    for (int u = 0; u < NP; ++u) vf[u] = load_v_frag(rb, u, 0);
    HYDRA_SCHED_FENCE();
#pragma unroll
    for (int u = 0; u < NP; ++u) {
#pragma unroll
      for (int qs = 0; qs < QS; ++qs) mfma_pv(o_acc[qs][u % CC], vf[u], Pp[qs][u / CC]);
    }
  };

  f32x16_t s_a[QS], s_b[QS];        // S of even / odd key blocks
  bf16x8_t p_a[QS][2], p_b[QS][2];  // P of even / odd key blocks
  using RB0 = std::integral_constant<int, 0>;
  using RB1 = std::integral_constant<int, 1>;
  using WithQK = std::integral_constant<bool, true>;
  using LastStep = std::integral_constant<bool, false>;

  if constexpr (TEAMS == 1 || kLoaders == 0) __syncthreads();  // K(0) is complete; every wave has taken its Q out of the V ring
  // the rest of the prologue loads: V(0) K(1) V(1) ... K(PD)
  if constexpr (Src::kPaged) {
    if constexpr (kLoaders == 0) gather.issue(0 < W, v_ring, 1 < W, k_ring + G::kTileBytes);
  } else {
#pragma unroll
    for (int n = 0; n < (kLoaders > 0 ? 0 : PD); ++n) {
      if (n < W_own) v_loader.issue_next(v_ring + n * G::kTileBytes);
      if (n + 1 < W_own) k_loader.issue_next(k_ring + (n + 1) * G::kTileBytes);
    }
  }

  // iteration 0: S(0) = K(0) Q^T alone, then S(1) = K(1) Q^T with the vector work of block 0 in its
  // shadow (reference = row maximum of block 0, softmax of block 0)
  if (NB > 0) {
    // (the K fragments of both blocks are requested ahead of the matrix instructions that use them,
    // with scheduling fences in between: see pv_only)
    bf16x8_t kf0[NQ], kf1[NQ];
#pragma unroll
    for (int s = 0; s < NQ; ++s) kf0[s] = load_k_frag(0, s, 0);
    HYDRA_SCHED_FENCE();
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
#pragma unroll
      for (int qs = 0; qs < QS; ++qs) {
        if (s == 0) mfma_qk_zero(s_a[qs], kf0[s], qf[qs][s]); else mfma_qk_acc(s_a[qs], kf0[s], qf[qs][s]);
      }
    }
    HYDRA_SCHED_FENCE();
#pragma unroll
    for (int s = 0; s < NQ; ++s) kf1[s] = load_k_frag(1, s, 0);
    HYDRA_SCHED_FENCE();
    // (S(1) is computed even when NB == 1: harmless, never read.)  Its first two matrix instructions cover
    // the wait states of S(0); the vector work follows behind the others.
    static_assert(NQ * QS >= 4, "two matrix instructions ahead of the first read of S(0), at least two to hide the vector work behind");
    constexpr int kLead = 2;
    int mi = 0;
    auto block0_valu = [&](int piece, int pieces) __attribute__((always_inline)) {
      // piece 0: mask and row maximum; the 16 * QS softmax halves are spread over the others
      if (piece == 0) {
        if (needs_mask(0)) apply_mask(0, s_a);
#pragma unroll
        for (int qs = 0; qs < QS; ++qs) {
          float t = fmaxf(s_a[qs][0], s_a[qs][1]);
#pragma unroll
          for (int r = 2; r < 16; ++r) t = fmaxf(t, s_a[qs][r]);
          t = max_with_other_half(t);
          nref[qs] = -t * c;
        }
      } else {
        const int n = 16 * QS, per = (n + pieces - 2) / (pieces - 1);
#pragma unroll
        for (int half = (piece - 1) * per; half < piece * per && half < n; ++half) softmax_half(half, s_a, p_a, row_sum);
      }
      HYDRA_SCHED_FENCE();
    };
    constexpr int kPieces = NQ * QS - kLead;
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
#pragma unroll
      for (int qs = 0; qs < QS; ++qs) {
        if (s == 0) mfma_qk_zero(s_b[qs], kf1[s], qf[qs][s]); else mfma_qk_acc(s_b[qs], kf1[s], qf[qs][s]);
        HYDRA_SCHED_FENCE();
        if (mi >= kLead) block0_valu(mi - kLead, kPieces);
        ++mi;
      }
    }
    s_results_to_valu(s_b);
  }
  wait_all_loads();
  __syncthreads();
  const int pos = __builtin_amdgcn_readfirstlane(pending_claim);  // every wave: the claim has returned (see above)
  if constexpr (!Src::kOneItem)
  if (wave == 0) {
    // (own queue empty: an empty claim is posted, and the top of the next round goes stealing)
    const int idx = pos < own_count ? own_claimed_at + pos : -1;
    // The item itself travels memory -> LDS on its own (one more direct-to-LDS load, lane 0 only):
    // it is complete when this wave's last wait of the round (for zero loads in flight) has
    // passed, and the barrier after that wait makes it visible to the other waves.  Every wave
    // has read this round's claim before the two barriers above, so the slot is free.
    if (lane == 0) {
      if (idx >= 0) {
        const uint64_t base = (uint64_t)(uintptr_t)a.items;
        u32x4_t rsrc;
        rsrc[0] = __builtin_amdgcn_readfirstlane((uint32_t)base);
        rsrc[1] = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
        rsrc[2] = 0xffffffffu;
        rsrc[3] = 0x00020000u;
        const uint32_t off = (uint32_t)idx * (uint32_t)sizeof(WorkItem);
        const uint32_t m0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)HYDRA_LDS_PTR(&s_claim[0]));
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(m0), "v"(off), "s"(rsrc));
      } else {
        s_claim[0] = 0;
        s_claim[1] = 0;
        s_claim[2] = 0;
        s_claim[3] = 0;
      }
    }
  }

  // Per wave: steps 1 .. NB-1.  Iterations 1 .. F run two steps each (the hot loop), iteration
  // F + 1 runs the odd step left over (if any) and the last P V product, later iterations only
  // keep the workgroup's loads and barriers going.
  const int F = NB > 0 ? (NB - 1) / 2 : 0;
  // The wave's last step (block NB - 1) has no further scores to compute.  With an odd number of
  // steps it is the single step of iteration F + 1; with an even number it is the second step of
  // iteration F, which is therefore run apart from the loop.
  const bool odd_steps = ((NB - 1) & 1) != 0;
  const int F_loop = odd_steps ? F : (F > 0 ? F - 1 : 0);
  int t = 1;
  StepFrags<PF> fr;
  // Inside its pipeline steps a wave goes ahead of the SIMD's other wave when that one is between items
  // (Q scaling, epilogue: long runs of vector instructions that would otherwise take every other issue slot).
  __builtin_amdgcn_s_setprio(1);
  // Iteration t reads K tile t (ring slot t % 2) and V tile t - 1 (slot (t - 1) % 2); t is odd at the top of a trip.
  static_assert(R == 2, "two iterations per trip cover the ring");
  auto hot_iteration = [&](int tt, int koff, int voff) __attribute__((always_inline)) {
    fetch_step_frags(0, true, fr, koff, voff);
    HYDRA_SCHED_FENCE();
    issue_loads(tt);
    block_step(RB0{}, WithQK{}, NextRB<1>{}, WithQK{}, 2 * tt - 1, s_b, s_a, p_a, p_b, fr, koff, voff);
    block_step(RB1{}, WithQK{}, NextRB<-1>{}, WithQK{}, 2 * tt, s_a, s_b, p_b, p_a, fr, koff, voff);
    wait_all_loads();
    __syncthreads();
  };
  for (; t + 1 <= F_loop; t += 2) {
    hot_iteration(t, G::kTileBytes, 0);
    hot_iteration(t + 1, 0, G::kTileBytes);
  }
  if (t <= F_loop) {
    hot_iteration(t, G::kTileBytes, 0);
    ++t;
  }
  if (!odd_steps && F > 0) {
    position_addresses(t);
    fetch_step_frags(0, true, fr, 0, 0);
    HYDRA_SCHED_FENCE();
    issue_loads(t);
    block_step(RB0{}, WithQK{}, NextRB<1>{}, LastStep{}, 2 * t - 1, s_b, s_a, p_a, p_b, fr, 0, 0);
    block_step(RB1{}, LastStep{}, NextRB<-1>{}, LastStep{}, 2 * t, s_a, s_b, p_b, p_a, fr, 0, 0);
    wait_all_loads();
    __syncthreads();
    ++t;
  }
  if (NB > 0 && t <= W) {
    position_addresses(t);
    if (odd_steps) {
      fetch_step_frags(0, false, fr, 0, 0);
      HYDRA_SCHED_FENCE();
    }
    issue_loads(t);
    if (odd_steps) {
      block_step(RB0{}, LastStep{}, NextRB<-1>{}, LastStep{}, NB - 1, s_b, s_a, p_a, p_b, fr, 0, 0);  // NB - 1 = 2t - 1
      pv_only(1, p_b);                                            // V block NB - 1 = 2t - 1: second block of V tile t - 1
    } else {
      pv_only(0, p_a);  // V block NB - 1 = 2t - 2: first block of V tile t - 1
    }
    wait_all_loads();
    __syncthreads();
    ++t;
  }
  for (; t <= W; ++t) {
    issue_loads(t);
    wait_all_loads();
    __syncthreads();
  }
  __builtin_amdgcn_s_setprio(0);
  // a row sum out of the safe range somewhere in this wave's rows: have the item recomputed (top of the next round)
  if (NB > 0) {
    bool too_far = false;
#pragma unroll
    for (int qs = 0; qs < QS; ++qs) {
      // (with the sums from the matrix unit: output column 80 + 4 hf of this lane's row)
      if constexpr (G::kSumsFromMatrixUnit) row_sum[qs] = o_acc[qs][CC - 1][8];
      too_far = too_far || !(row_sum[qs] <= kMaxRowSum);
    }
    if (__builtin_amdgcn_ballot_w64(too_far) != 0 && lane == 0) {
      s_redo[1] = (int)seq_start;
      s_redo[2] = seq_len;
      s_redo[3] = f0;
      s_redo[4] = kv_head;
      s_redo[0] = 1;
    }
  }
  // The next item (posted during this round; the last iteration's wait and barrier made it visible):
  // start its Q loads now.  (When the die's queue has run out the posted claim is empty, and the
  // item stolen at the top of the next round loads its Q there.)
  q_ahead = false;
  if constexpr (!Src::kOneItem) {
    const int next_len = __builtin_amdgcn_readfirstlane(s_claim[1]);
    if (next_len != 0) {
      const int64_t next_start = __builtin_amdgcn_readfirstlane(s_claim[0]);
      const int next_f0 = __builtin_amdgcn_readfirstlane(s_claim[2]);
      const int next_kv = __builtin_amdgcn_readfirstlane(s_claim[3]);
      const int wave_tiles = ((next_len + kWaveTileRows - 1) / kWaveTileRows) * a.group;
      const int nf = next_f0 + wave < wave_tiles ? next_f0 + wave : wave_tiles - 1;
      const int tile = token_tile(nf);
      issue_q_loads(next_start, next_len, tile * kWaveTileRows, next_kv * a.group + (nf - tile * a.group), lane);
      q_ahead = true;
    }
  }
  // ---- epilogue: normalise, round to bf16, transpose through LDS, store whole rows ----
  // In the accumulators a lane owns one query row and scattered groups of 4 columns; stored from
  // there, one store instruction would touch 32 different rows.  So each wave writes its 32 x D
  // tile to a private LDS staging area in K-tile layout and reads it back with one row per 16
  // (D = 128) lanes.  Staging area: the K ring, which is idle between an item's last iteration and the
  // next item's first load (issued after the barrier at the top of the next round).  The stores go
  // through a buffer descriptor that ends with the tile's last valid row (rows past it are dropped
  // by the hardware).
  static_assert(WT * kWaveTileRows * ROWB <= R * G::kTileBytes, "the output tiles of a team's waves fit its K ring");
  // Two teams: each has the references, sums and unnormalised outputs of its keys.  They exchange halves of the columns through
  // their rings, in the order of the registers, and each finishes its half.
  constexpr int kOut = G::kChunks / TEAMS;  // 16-byte pieces of an output row that a wave finishes
  float o_mine[kOut][4];                    // (eight columns of a row are with lanes m and m + 32)
  float total = row_sum[0];
  if constexpr (TEAMS > 1) {
    static_assert(QS == 1 && TEAMS == 2 && G::kChunks % 2 == 0, "one row per lane, halves of columns");
    constexpr int kSlotBytes = kOut * 1024;
    static_assert(WT * kSlotBytes <= R * G::kTileBytes, "what a team hands over fits its K ring");
    const uint32_t slot = wave_tile * kSlotBytes + lane * 16, sums = lds0 + G::kSumsAt + wave_tile * 512 + lane * 8;
    const uint32_t k_other = lds0 + (1 - team) * G::kTeamBytes;
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
      f32x4_t theirs;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float lower = o_acc[0][i / 4][4 * (i % 4) + e], upper = o_acc[0][(i + kOut) / 4][4 * ((i + kOut) % 4) + e];
        o_mine[i][e] = team == 0 ? lower : upper;
        theirs[e] = team == 0 ? upper : lower;
      }
      *reinterpret_cast<f32x4_t*>(HYDRA_LDS_BYTE(k_ring + slot + i * 1024)) = theirs;
    }
    *reinterpret_cast<f32x2_t*>(HYDRA_LDS_BYTE(sums + team * G::kTeamSums)) = f32x2_t{-nref[0], row_sum[0]};
    __syncthreads();
    const f32x2_t rs = *reinterpret_cast<const f32x2_t*>(HYDRA_LDS_BYTE(sums + (1 - team) * G::kTeamSums));
    const float both = fmaxf(-nref[0], rs[0]), w_mine = fast_exp2(-nref[0] - both), w_theirs = fast_exp2(rs[0] - both);
    total = row_sum[0] * w_mine + rs[1] * w_theirs;
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
      const f32x4_t x = *reinterpret_cast<const f32x4_t*>(HYDRA_LDS_BYTE(k_other + slot + i * 1024));
#pragma unroll
      for (int e = 0; e < 4; ++e) o_mine[i][e] = o_mine[i][e] * w_mine + x[e] * w_theirs;
    }
    // (each wave's staging area below lies in its own team's V ring: the other team may still be reading the K ring)
  } else {
#pragma unroll
    for (int i = 0; i < kOut; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) o_mine[i][e] = o_acc[0][i / 4][4 * (i % 4) + e];
  }
  if (active) {
    const uint32_t o_stage = (TEAMS > 1 ? v_ring : k_ring) + wave_tile * (kWaveTileRows * ROWB);
    if constexpr (!G::kSumsFromMatrixUnit) total = sum_with_other_half(total);
    const float inv = 1.0f / total;
#pragma unroll
    for (int i = 0; i < kOut; ++i) {  // columns 8 i .. 8 i + 7 of the wave's; this lane has 4 hf .. 4 hf + 3 of them
      f32x2_t x0 = {o_mine[i][0] * inv, o_mine[i][1] * inv};
      f32x2_t x1 = {o_mine[i][2] * inv, o_mine[i][3] * inv};
      u32x2_t pk = {__builtin_bit_cast(uint32_t, __builtin_convertvector(x0, bf16x2_t)),
                    __builtin_bit_cast(uint32_t, __builtin_convertvector(x1, bf16x2_t))};
      *reinterpret_cast<u32x2_t*>(HYDRA_LDS_BYTE(o_stage + m * ROWB + k_swizzle<D>(m, i) * 16 + 8 * hf)) = pk;
    }
    const uint64_t base = (uint64_t)(uintptr_t)(a.out + ((seq_start + q0) * a.n_q_heads + head) * D);
    const uint32_t out_row_bytes = (uint32_t)a.n_q_heads * (D * 2);
    const int rows = seq_len - q0 < kWaveTileRows ? seq_len - q0 : kWaveTileRows;
    u32x4_t rsrc;
    rsrc[0] = __builtin_amdgcn_readfirstlane((uint32_t)base);
    rsrc[1] = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32) & 0xffffu);
    rsrc[2] = __builtin_amdgcn_readfirstlane((uint32_t)(rows - 1) * out_row_bytes + D * 2);
    rsrc[3] = 0x00020000u;
#pragma unroll
    for (int i = 0; i < (kRowInstr + TEAMS - 1) / TEAMS; ++i) {
      const int flat = i * 64 + lane;
      const int r = flat / kOut, chunk = flat % kOut;
      const u32x4_t piece = *reinterpret_cast<const u32x4_t*>(HYDRA_LDS_BYTE(o_stage + r * ROWB + k_swizzle<D>(r, chunk) * 16));
      const uint32_t off = (uint32_t)r * out_row_bytes + (team * kOut + chunk) * 16;  // (r past the tile: out of the descriptor's range)
      // (a store of more than 8 bytes reads its data registers a little after it issues; the wait
      // states keep the next instruction from overwriting them: the compiler does not see this store)
      // (nt: the output is not read again by this kernel)
      asm volatile("buffer_store_dwordx4 %0, %1, %2, 0 offen nt\n\ts_nop 1" : : "v"(piece), "v"(off), "s"(rsrc) : "memory");
    }
  }
  if constexpr (Src::kOneItem) break;
  }  // next work item
  if constexpr (Src::kOneItem) {
    __syncthreads();
    return s_redo[0] != 0;
  }
  if constexpr (!Src::kOneItem) {
    if (wave == 0) {
      int y = threadIdx.x & (kXcds - 1);
      asm volatile("" : "+v"(y));
      if (__builtin_amdgcn_ballot_w64(claimable(a.ctrl, y) > 0) != 0 && threadIdx.x == 0) leave(a.ctrl);
    }
  }
  return false;
}
#endif  // __HIP_DEVICE_COMPILE__

template <int D, bool CAUSAL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PackedSource::kWavesPerSimd<D>, PackedSource::kWavesPerSimd<D>))) void attn_fwd_kernel(const AttnArgs a) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(1024))) unsigned char smem[TileGeom<D>::kLdsBytes];
  __shared__ __attribute__((aligned(16))) int s_claim[4];
  __shared__ __attribute__((aligned(16))) int s_redo[8];
  attn_item_loop<D, CAUSAL>(a, PackedSource{}, smem, s_claim, s_redo);
#else
  (void)a;
#endif
}

// ---- one workgroup per item ------------------------------------------------------------------------------------
// Batches of a few items per workgroup slot run with one workgroup per item, dealt out by the hardware as slots fall
// free, instead of persistent workgroups that claim: at so few rounds the claims, their start and their end cost more
// than loading the next item's Q ahead wins (7 LLaVA requests, 3 rounds: 85.0 -> 78.3 us; at 6 rounds the two are
// level, at 13 persistent workgroups win by 2 %).  At head_dim 80, where three of these workgroups fit a compute unit and only
// two persistent ones, this form is the faster one at every size measured (200 000 tokens in images of 256 .. 4096, 16 heads, 2265 -> 2102 us).
// The item comes from the work list when there is one.  Without one (the call that would have to build it first), and
// for at most kDirectSeqs sequences, every wave works its workgroup's item out from cu_seqlens, one round trip to memory
// and some 300 instructions, about 1.3 us per workgroup against a prepass of 4 - 5 us.
// Forms.  TEAMS = 1, LOADERS = 0: as the persistent kernel, but one item.  Where the batch has a compute unit for every item, an item's
// chain of key tiles is the kernel's length, and a wave alone on its SIMD spends half of an iteration issuing its share of the tile loads
// (16 cycles of the compute unit per kilobyte, during which a wave issues nothing else) and in the LDS and matrix latencies that no
// other wave covers.  LOADERS > 0: that many more waves per team issue the loads, half of them K tiles and half V tiles, the first of
// them while Q is on its way: an iteration of 64 keys at head_dim 128 takes 0.8 us instead of 1.0.  TEAMS = 2: the workgroup has two
// wave tiles instead of four, and each of two teams of two waves half of the key tiles, in rings of its own; the teams share the
// loads of Q and merge their results through LDS, half of the columns by each (all by one: 0.3 to 0.6 us longer).  us with 4, 8 and 8
// waves so: one image of 577 tokens with 16 heads of 64 9.45, 8.58, 6.58; a request of 558 tokens with 28 / 4 heads of 128 12.4, 11.3,
// 8.9.  TEAMS = 2, LOADERS = 0 is the same split for calls that leave registers to others (10.5 us).  It leaves
// less of the LDS, at head_dim 128 too little for a decode workgroup of the same head_dim.  us per call alone, and of it and of a stream
// of decode steps beside it, as persistent workgroups and so: 200 tokens with 28 / 4 heads of 128 beside 64 of 128 .. 1800 tokens 8.4,
// 15.6 + 26.2 and 6.6, 9.0 + 29.5; 558 tokens beside 32 of 400 .. 1200 13.1, 15.5 + 18.6 and 10.1, 13.3 + 17.0; 577 with 16 heads of 64 beside
// 33 of 600 .. 1100 with 32 / 32 heads of 128 10.7, 37.3 + 79.8 and 7.4, 42.5 + 78.2.  Both streams together are done earlier, or 1 % later,
// in eleven of twelve such pairs, in the last one named 4 % later.
// LOADERS change no bit of the result; two teams' P is rounded relative to a reference of each team (the relative error against 64 bits
// goes down by 0.3 to 3 %).
// Not kept: one copy of the iteration's code instead of two plus the last one's, 0.1 to 0.5 us longer; two teams of four waves without
// loading waves, equal to one team with; two loading waves per team of four waves, three waves per SIMD, equal at head_dim 64, 4 to 7 %
// faster at 80; two waves per wave tile that take the scores of every other key block each, exchange P through LDS and multiply half
// of the columns each, 9.0 and 10.8 us: an iteration per key tile again, and 0.4 us of an iteration are latencies.
template <int D, bool CAUSAL, int TEAMS, int LOADERS>
__global__ __launch_bounds__((DirectSource<TEAMS, LOADERS>::kBound)) __attribute__((amdgpu_waves_per_eu(DirectSource<TEAMS, LOADERS>::template kWavesPerSimd<D>, DirectSource<TEAMS, LOADERS>::template kWavesPerSimd<D>))) void attn_fwd_direct_kernel(
    const AttnArgs a, const int batch, const int n_kv_heads) {  // batch 0: the item comes from the work list
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ __attribute__((aligned(1024))) unsigned char smem[TileGeom<D, TEAMS, DirectSource<TEAMS, LOADERS>::kStageRows>::kLdsBytes];
  __shared__ __attribute__((aligned(16))) int s_claim[4];
  __shared__ __attribute__((aligned(16))) int s_redo[8];
  // (all arguments in one trip to memory: one image of 577 tokens with 16 heads of 64 6.63 -> 6.53 us, a request of 1500 tokens with 28 / 4
  // heads of 128 22.4 -> 22.1)
  asm volatile("" : : "s"(a.q), "s"(a.k), "s"(a.v), "s"(a.out), "s"(a.q_stride), "s"(a.k_stride), "s"(a.v_stride), "s"(a.cu_seqlens), "s"(a.items), "s"(a.ctrl),
               "s"(a.n_q_heads), "s"(a.group), "s"(a.scale_log2), "s"(batch), "s"(n_kv_heads));
  DirectSource<TEAMS, LOADERS> src;
  constexpr int TILES = src.kTiles, kShare = kWavesPerItem / TILES;  // wave tiles per workgroup, workgroups per entry of the list
  if (batch == 0) {  // (an entry of the list is shared by kShare workgroups)
    const int lane = threadIdx.x & 63;
    const int first = a.ctrl->xcd_start[lane % kXcds];
    int die, place;
    if (!take_entry((a.ctrl->xcd_start[lane % kXcds + 1] - first) * kShare, (int)blockIdx.x, die, place)) return;
    const WorkItem it = a.items[__builtin_amdgcn_readlane(first, die) + place / kShare];
    src.q_start = __builtin_amdgcn_readfirstlane(it.x);
    src.q_len = __builtin_amdgcn_readfirstlane(it.y);
    src.f0 = __builtin_amdgcn_readfirstlane(it.z) + place % kShare * TILES;
    src.kv_head = __builtin_amdgcn_readfirstlane(it.w);
    if (kShare > 1 && src.f0 >= (src.q_len + kWaveTileRows - 1) / kWaveTileRows * a.group) return;
  } else {
    int start, item;
    if (!find_unit(a.cu_seqlens, batch, n_kv_heads, [&](int len) { return items_of_sequence<TILES>(len, a.group); }, start, src.q_len, src.kv_head, item)) return;
    if (CAUSAL) item = items_of_sequence<TILES>(src.q_len, a.group) - 1 - item;  // most expensive first
    src.q_start = start;
    src.f0 = item * TILES;
  }
  if (attn_item_loop<D, CAUSAL>(a, src, smem, s_claim, s_redo)) {
    if constexpr (TEAMS > 1) {  // (the other team's waves have stored parts of the rows that are stored again)
      wait_all_loads();
      __syncthreads();
    }
    const uint32_t lds = (uint32_t)(uintptr_t)HYDRA_LDS_PTR(smem);
    careful::run_item<D, CAUSAL, TILES, DirectSource<TEAMS, LOADERS>::kThreads / 64>(a, src.q_start, src.q_len, src.f0, src.kv_head, lds);
  }
#else
  (void)a;
  (void)batch;
  (void)n_kv_heads;
#endif
}

}  // namespace hydra
