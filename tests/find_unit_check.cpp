// Walks find_unit (paper_2505_12658_amd/csrc/find_unit.hpp) on the host, for every workgroup of many batches: each (sequence, KV head,
// item) has to come out exactly once, and nothing else.
// The 64 lanes of a wave are 64 contexts; each runs up to its next operation over the wave's lanes, and when all have got there,
// all go on.  An operation that not all lanes reach, or a uniform operand that differs, ends the program.
#include <setjmp.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <random>
#include <vector>

#define __device__
#define __forceinline__ inline
#define __HIP_DEVICE_COMPILE__ 1

struct Index {
  int x;
};
static Index threadIdx, blockIdx;

static void fail(const char* what) {
  printf("FAILED: %s\n", what);
  exit(1);
}

namespace wave {
constexpr int kLanes = 64;
constexpr size_t kStack = 64 * 1024;
enum Kind { kBallot, kReadLane, kReadFirst, kPermute, kBpermute, kScan, kColumns, kEnd };
static ucontext_t first_entry[kLanes], main_context;
static jmp_buf lane_at[kLanes], scheduler;
static std::vector<char> stacks(kLanes * kStack);
static int value[kLanes], operand[kLanes], result[kLanes];  // of the lanes' current operation
static uint64_t mask;
static Kind kind[kLanes];
static void (*body)();

// hands over this lane's value and goes on when all lanes have done so and `result` or `mask` is there
static int meet(Kind what, int v, int other = 0) {
  const int lane = threadIdx.x;
  value[lane] = v;
  operand[lane] = other;
  kind[lane] = what;
  if (_setjmp(lane_at[lane]) == 0) _longjmp(scheduler, 1);
  return result[threadIdx.x];
}
static void entry() {
  for (;;) {
    body();
    meet(kEnd, 0);
  }
}
static void resume(int lane, bool fresh) {
  threadIdx.x = lane;
  if (_setjmp(scheduler) != 0) return;
  if (fresh) setcontext(&first_entry[lane]);
  _longjmp(lane_at[lane], 1);
}
static void init(void (*b)()) {
  body = b;
  for (int l = 0; l < kLanes; ++l) {
    getcontext(&first_entry[l]);
    first_entry[l].uc_stack.ss_sp = &stacks[l * kStack];
    first_entry[l].uc_stack.ss_size = kStack;
    first_entry[l].uc_link = &main_context;
    makecontext(&first_entry[l], entry, 0);
  }
}
static void do_operation() {
  for (int l = 1; l < kLanes; ++l)
    if (kind[l] != kind[0]) fail("lanes are at different operations of the wave");
  int sum = 0, columns[8] = {};
  mask = 0;
  for (int l = 0; l < kLanes; ++l) {
    if (kind[0] == kReadLane && (operand[l] != operand[0] || operand[l] < 0 || operand[l] >= kLanes)) fail("a lane number that is not one");
    mask |= (uint64_t)(value[l] != 0) << l;
    columns[l % 8] += value[l];
  }
  for (int l = 0; l < kLanes; ++l) {
    sum += value[l];
    switch (kind[0]) {
      case kReadLane: result[l] = value[operand[0]]; break;
      case kReadFirst: result[l] = value[0]; break;
      case kPermute: result[operand[l] >> 2 & 63] = value[l]; break;
      case kBpermute: result[l] = value[operand[l] >> 2 & 63]; break;
      case kScan: result[l] = sum; break;
      case kColumns: result[l] = columns[l % 8]; break;
      default: break;
    }
  }
}
static bool started = false;
static void run() {  // one pass of all lanes through the body
  do {
    for (volatile int l = 0; l < kLanes; l = l + 1) resume(l, !started);
    started = true;
    do_operation();
  } while (kind[0] != kEnd);
}
}  // namespace wave

static uint64_t __builtin_amdgcn_ballot_w64(bool x) {
  wave::meet(wave::kBallot, x);
  return wave::mask;
}
static int __builtin_amdgcn_readlane(int x, int lane) { return wave::meet(wave::kReadLane, x, lane); }
static int __builtin_amdgcn_readfirstlane(int x) { return wave::meet(wave::kReadFirst, x); }
static int __builtin_amdgcn_ds_permute(int address, int x) { return wave::meet(wave::kPermute, x, address); }
static int __builtin_amdgcn_ds_bpermute(int address, int x) { return wave::meet(wave::kBpermute, x, address); }
static float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }

namespace hydra {
constexpr int kXcds = 8;
static int wave_scan_add(int x) { return wave::meet(wave::kScan, x); }
static int sum_of_columns(int x) { return wave::meet(wave::kColumns, x); }
}  // namespace hydra

#include "../paper_2505_12658_amd/csrc/find_unit.hpp"

static struct {
  std::vector<int32_t> cu;
  int batch, n_kv_heads, group, tiles;
} job;
static struct Found {
  bool found;
  int seq_start, seq_len, kv_head, unit;
} found[64];

static int items(int len) { return ((len + 31) / 32 * job.group + job.tiles - 1) / job.tiles; }

static void one_lane() {
  const int lane = threadIdx.x;
  Found f = {};
  f.found = hydra::find_unit(job.cu.data(), job.batch, job.n_kv_heads, items, f.seq_start, f.seq_len, f.kv_head, f.unit);
  found[lane] = f;
}

static long batches = 0, units = 0;

static void check(const std::vector<int>& lengths, int n_kv_heads, int group, int tiles) {
  job.batch = (int)lengths.size();
  job.n_kv_heads = n_kv_heads;
  job.group = group;
  job.tiles = tiles;
  job.cu.assign(1, 0);
  for (int n : lengths) job.cu.push_back(job.cu.back() + n);
  char what[256];
  std::vector<std::vector<char>> done(lengths.size() * n_kv_heads);
  for (size_t b = 0; b < lengths.size(); ++b)
    for (int h = 0; h < n_kv_heads; ++h) done[b * n_kv_heads + h].assign(items(lengths[b]), 0);
  const int64_t grid = hydra::direct_workgroups(tiles, tiles, job.batch, job.cu.back(), group, n_kv_heads);
  auto say = [&](const char* why, int64_t id) {
    snprintf(what, sizeof what, "%s: workgroup %ld of %ld, %zu sequences of %d, %d .. %d, %d KV heads, group %d, %d wave tiles per item", why, (long)id, (long)grid, lengths.size(),
             lengths[0], lengths.size() > 1 ? lengths[1] : lengths[0], lengths.back(), n_kv_heads, group, tiles);
    fail(what);
  };
  for (int64_t id = 0; id < grid; ++id) {
    blockIdx.x = (int)id;
    wave::run();
    const Found f = found[0];
    for (int l = 1; l < 64; ++l)
      if (found[l].found != f.found || (f.found && (found[l].seq_start != f.seq_start || found[l].seq_len != f.seq_len || found[l].kv_head != f.kv_head || found[l].unit != f.unit)))
        say("lanes differ", id);
    if (!f.found) continue;
    size_t b = 0;
    while (b < lengths.size() && (job.cu[b] != f.seq_start || lengths[b] == 0)) ++b;
    if (b == lengths.size() || f.seq_len != lengths[b]) say("no such sequence", id);
    if (f.kv_head < 0 || f.kv_head >= n_kv_heads) say("no such KV head", id);
    std::vector<char>& d = done[b * n_kv_heads + f.kv_head];
    if (f.unit < 0 || f.unit >= (int)d.size()) say("no such item", id);
    if (d[f.unit]++) say("an item twice", id);
  }
  for (size_t i = 0; i < done.size(); ++i)
    for (size_t u = 0; u < done[i].size(); ++u)
      if (!done[i][u]) say("an item is left out", (int64_t)u);
  ++batches;
  units += grid;
}

int main(int argc, char** argv) {
  const int part = argc > 1 ? atoi(argv[1]) : 0, parts = argc > 2 ? atoi(argv[2]) : 1;
  wave::init(one_lane);
  std::mt19937 gen(part);
  auto pick = [&](int lo, int hi) { return lo + (int)(gen() % (unsigned)(hi - lo + 1)); };
  int number = 0;
  // sequences of one length, and of many
  for (int batch : {1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 23, 32, 33, 48, 63, 64})
    for (int heads : {1, 2, 3, 4, 5, 7, 8, 12, 16}) {
      if (number++ % parts != part) continue;
      const int pairs = batch * heads, tiles = pick(0, 1) ? 2 : 4, group = pick(1, 16);
      const int most = pairs < 600 ? 600 / pairs : 1;  // items per pair
      for (int n : {pick(1, most), most}) {
        const int wave_tiles = n * tiles / group > 0 ? n * tiles / group : 1, len = 32 * (wave_tiles - 1) + pick(1, 32);
        check(std::vector<int>(batch, len), heads, group, tiles);
        if (n == most) continue;
        std::vector<int> lens(batch);
        for (int& l : lens) l = pick(0, 4) == 0 ? 0 : pick(1, 2 * len);
        lens[pick(0, batch - 1)] = len;
        check(lens, heads, group, tiles);
      }
    }
  // few pairs, more than 32 items for each
  for (int batch : {1, 2, 3, 4, 7})
    for (int heads : {1, 2, 3, 4}) {
      if (batch * heads > 8 || number++ % parts != part) continue;
      for (int tiles : {2, 4})
        for (int group : {7, 8, 16})
          for (int len : {300, 600, 1100}) check(std::vector<int>(batch, len), heads, group, tiles);
    }
  printf("%ld batches, %ld workgroups: ok\n", batches, units);
  return 0;
}
