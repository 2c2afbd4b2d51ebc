// The inner loop of an epoch (Alg. 1 steps 5-11; Alg. 2 steps 5-15) on CSR data in one launch (one per 128 iterations):
// P = 256 workgroups, each the owner of the columns c = p mod P for all vectors, with its slice of the iterate in LDS.
//
// As separate launches an iteration of n = d = 2^20, N = 16, B = 256, 40 entries a row is 36 us of kernels (worker pass 11.2,
// statistics 10.6, quantizer 7.3, receiver and update of all d coordinates 6.3), although it samples 1.3 MB.  Here the update
// of the coordinates that no row touches never leaves a workgroup, u^i is formed where its column lives, and what crosses
// between workgroups, as tagged words, is
//   1. the iterate at the columns that the next iteration's rows hold, from their owners to the rows' wavefronts,
//   2. a row's slope difference, from its wavefront to the owners of its columns,
//   3. the statistics of u^i, from every owner to all of them, by way of a wavefront per vector and die; each derives the scale
//      factors.
// The draws do not depend on the iterates, so what an owner has to add up is known ahead: list_build_kernel leaves, for every
// iteration, vector and owner, the sampled entries with their columns together and in batch-position order.  Wavefront i
// of an owner takes vector i's list: slope times value, sums, eq. (3), rules (1) and (2); the codes meet in LDS, a field per
// vector and column, and a lane per touched column takes eq. (4) and the update.
// Margins and sums are added up in the order of the separate launches (a column's entries in blocks of batch positions, the
// blocks in order: a list is cut in pieces of one column and block), so an epoch's bits do not depend on the route, but for
// three sums of another order: what a row holds past its 64th entry or a second time, which the sparse worker pass adds by
// itself, and with clipping by c*sigma the sums over the coordinates.  A segmented scan over the lanes would be 0.3 us per
// iteration less (16 vectors), and another rounding now and then.
// Neighbouring columns belong to different owners because text-like data has its frequent columns side by side.
// Reuse of words: a column's x word is kept once, written again when its owner has the slopes of every row that holds the
// column, hence after those rows' wavefronts read it.  Slopes and statistics have two sets: set t is written again at t + 2 by
// somebody who has seen words of t + 1 from every owner (by way of the iterate of t + 2, in a slope's case), and an owner
// writes those after it has done with the slopes and statistics of t.
// The launch is cooperative; waits are bounded as in lpc_columns.hip, and a launch that gave up leaves the caller's vectors alone.
//
// Bound by the four trips of words (store to load about 1.2 us each) and by the owner of the most frequent column, whose lists
// are six times as long as the others'.  Measured on MI355X, separate launches -> these kernels, us per iteration, the lists
// (1.7 there) included: n = d = 2^20, N = 16, B = 256, b = 2: 35.5 -> 11.7; d = 150001, N = 8 + J, B = 100, b = 4: 30.6 -> 11.0.
// Steps that paid, us per iteration of the first: registers loaded ahead without a join that waits for them and waits for
// them before the next store, not behind it, together with priority for rows and sums over what only fills the waits, 1.0;
// columns found by the builder instead of here and words stored as soon as they are known, 1.9; half of the trips' time went
// where words of several dies shared a line: a line belongs to one workgroup, or to one die.  Steps that did not: copies of the
// frequent columns' words per die (+ 1.1), the lists requested while the statistics travel (+ 1.2), pauses between polls (0),
// P = 128 (+ 1.8).
#include <hip/hip_runtime.h>

#include "lpc_device.h"
#include "lpc_internal.h"

namespace lpc {

namespace {

constexpr int kLiThreads = 1024, kLiWaves = kLiThreads / 64;
constexpr int kLiRows = 2;      // sampled rows of a wavefront
constexpr int kLiChunks = 5;    // 64-entry chunks of a vector's list that a wavefront holds in registers
constexpr int kLiPairs = 2;     // ... and 64-column chunks of its columns
constexpr int kLiLds = 156 * 1024;
constexpr int kOwnerBits = 8, kOwners = 1 << kOwnerBits;
constexpr int kOwnBins = 4;     // an owner's first columns, with a map of batch positions each; the others: bins of a quarter
constexpr int kMaxBatch = 512;
constexpr int kKeyChunks = 100; // 64-entry chunks of the others' keys that a workgroup of the builder sorts at once
constexpr int kKeyCap = 64 * kKeyChunks;
constexpr int kRecord = 5;      // words of a list's record: first entry, entries, columns, pieces, longest piece
constexpr int kSortChunks = (kKeyChunks + kLiWaves - 1) / kLiWaves;
constexpr int kHeld = 16;       // rows whose columns a wavefront of the builder holds
constexpr int kDies = 8;
constexpr int kLine = 16;       // words of a 128-byte line
constexpr uint32_t kNoEntry = 0xffffffffu, kLast = 0x80000000u;

// ---------------------------------------------------------------------------------------------------------------------
// The lists.  A workgroup takes one vector's batch of one iteration; entry (column c, batch position pos, k-th of its row)
// has the key lc << (pos_bits + k_bits) | pos << k_bits | k, lc = c / P, unique in an owner's list.
struct ListBuildArgs {
  const int32_t *col_idx;
  const float *vals;
  RowPlan *plan;        // of the first iteration of the launch; its margins become slopes
  uint32_t *rec;        // [iterations][nvec][P][kRecord]
  uint2 *ent;           // [iterations][nvec][cap]: batch position, value
  uint32_t *cols;       // [iterations][nvec][cap]: a list's columns lc + 1, from its first entry's place on
  uint32_t *pieces;     // [iterations][nvec][cap]: likewise its pieces' first entries (kLast: its column's last one); with the
                        // piece's length from bit 12 on if the list has no more entries than a wavefront takes in registers
  int64_t cap;
  int32_t B, pos_bits, k_bits, map_words, map_space, key_space, loss, block;
};

// A buffer of its own for a row or list: loads past its end are 0, without a branch.
__device__ __forceinline__ auto buffer(const void *from, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(from), 0, (int)bytes, 0x00027000);
}

// An owner's first four columns (text-like data has more than half of its entries there, hundreds in a column) have a map of
// the batch positions each: an entry's rank is a count of bits, the pieces are counts of bits of a block.  The other entries'
// keys are put in the owner's four bins in any order, counted against the five or so others of their bin, written back in order,
// and walked in that order: heads of columns and pieces are votes of 64 neighbours, and counts of votes place them.  No sum or
// place depends on timing.
// Entries go to memory by way of LDS: stored from where they are read, one line each, the address units were busy throughout
// and lines left the L2 half full (0.77 GB written for 0.24; now 0.35).  Registers must not spill: 30 of them are as many bytes as the lists.
// Bound by instructions (2360 of the vector units per wavefront and batch: these are busy 58 % of the time) and LDS (73 %).  Two workgroups to a CU: 80 KB for B = 256.
// Measured on MI355X, lists of 128 iterations of n = d = 2^20, 16 vectors, B = 256, 40 entries a row: 214 us; 64 iterations of
// d = 150001, 9 vectors, B = 100, 24 entries: 40 (each entry placed by itself, a wavefront per list to find heads: 362, 63).
__global__ __launch_bounds__(kLiThreads, 8) void list_build_kernel(ListBuildArgs a) {
  extern __shared__ uint32_t build_lds[];
  __shared__ uint32_t cursor[kOwnBins * kOwners];     // key slots of a bin: the next one
  __shared__ uint32_t single_at[kOwnBins * kOwners];  // a mapped column's first entry, of the mapped ones
  __shared__ uint32_t first[kOwners + 1], slot0[kOwners + 1];  // an owner's first entry, first key slot
  __shared__ uint32_t singles[kOwners], longest[kOwners];      // pieces << 16 | columns of the mapped ones; longest piece
  __shared__ uint64_t votes_mem[2 * (kKeyChunks + 1)];
  __shared__ uint32_t before[kKeyChunks + 1];  // pieces << 16 | columns of the chunks before
  __shared__ uint32_t total_a[kLiWaves], total_b[kLiWaves], twice;
  int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Between the phases: what is derived from these is not to be kept in registers, let alone in memory, from one to the next.
  auto part = [&] {
    asm volatile("" : "+v"(tid));
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  };
  constexpr int P = kOwners, kBins = kOwnBins * P;  // bin: column mod kBins
  // first maps [map_words][4 P], for every other of their words the bits before it, and staged entries; then keys with owners and values
  uint32_t *maps = build_lds, *key_values = build_lds, *keys = build_lds + a.map_space;
  uint8_t *owner = reinterpret_cast<uint8_t *>(keys + kKeyCap);
  uint16_t *ranks = reinterpret_cast<uint16_t *>(keys);
  const int n_ranks = kBins * ((a.map_words + 1) / 2), n_stage = (a.key_space - n_ranks / 2) * 4 / 6;
  uint32_t *stage_value = keys + n_ranks / 2;
  uint16_t *stage_pos = reinterpret_cast<uint16_t *>(stage_value + n_stage);
  uint64_t *col_heads = votes_mem, *heads = votes_mem + kKeyChunks + 1;
  uint32_t *one0 = reinterpret_cast<uint32_t *>(votes_mem);  // before there are heads: an owner's first entry of the mapped ones
  int32_t *lo_sh = reinterpret_cast<int32_t *>(keys + a.key_space), *len_sh = lo_sh + a.B;
  RowPlan *rows = a.plan + (int64_t)blockIdx.x * a.B;
  uint2 *out = a.ent + (int64_t)blockIdx.x * a.cap;
  uint32_t *cols = a.cols + (int64_t)blockIdx.x * a.cap, *pieces = a.pieces + (int64_t)blockIdx.x * a.cap;
  for (int r = tid; r < a.B; r += kLiThreads) {
    const RowPlan row = rows[r];
    lo_sh[r] = row.lo;
    len_sh[r] = row.hi - row.lo;
    rows[r].z = loss_slope(a.loss, row.z, row.y);
  }
  if (tid == 0) twice = 0u;
  const int held = kHeld * kLiWaves, groups = (a.B + held - 1) / held;
  int32_t c[kHeld];
  bool far = false;  // a row of the wavefront's has more than 64 entries
  uint32_t row_lo, row_len;  // lane q's: row g * held + q * kLiWaves + wave
  auto take_rows = [&](int g) {
    const int r = g * held + lane * kLiWaves + wave;
    const bool has = lane < kHeld && r < a.B;
    row_lo = has ? (uint32_t)lo_sh[r] : 0u;
    row_len = has ? (uint32_t)len_sh[r] : 0u;
    far = __ballot(row_len > 64u) != 0ull;
  };
  // lane l's of a row's first 64 words (0 past its end)
  auto row_words = [&](const void *from, int q) {
    return __builtin_amdgcn_raw_buffer_load_b32(
        buffer(static_cast<const uint32_t *>(from) + read_lane(row_lo, q), 4u * read_lane(row_len, q)), 4 * lane, 0, 0);
  };
  auto load = [&](int g) {
    take_rows(g);
#pragma unroll
    for (int q = 0; q < kHeld; ++q) {
      const uint32_t col = row_words(a.col_idx, q);
      c[q] = (uint32_t)lane < read_lane(row_len, q) ? (int32_t)col : -1;
    }
  };
  // f(column, row, index in the row, value) for the entries past a row's first 64
  auto walk_far = [&](int g, auto f) {
    if (!far) return;
    for (int r = g * held + wave; r < a.B && r < (g + 1) * held; r += kLiWaves) {
      const int32_t lo = __builtin_amdgcn_readfirstlane(lo_sh[r]), len = __builtin_amdgcn_readfirstlane(len_sh[r]);
      for (int32_t k = 64 + lane; k < len; k += 64) f((uint32_t)a.col_idx[lo + k], r, (uint32_t)k, lo + k);
    }
  };
  auto map_word = [&](uint32_t bin, int w) -> uint32_t & { return maps[w * kBins + (int)bin]; };
  auto rank_of = [&](uint32_t bin, int r) -> uint32_t {  // bits of a map before position r
    uint32_t n = ranks[(r >> 6) * kBins + (int)bin] + __popc(map_word(bin, r >> 5) & ((1u << (r & 31)) - 1u));
    if (r & 32) n += __popc(map_word(bin, (r >> 5) - 1));  // uniform
    return n;
  };
  bool mapped = true;  // false: a row holds a column twice, all entries have keys
  for (;;) {
    cursor[tid] = 0u;
    for (int w = tid; w < kBins * a.map_words; w += kLiThreads) maps[w] = 0u;
    __syncthreads();
    uint32_t again = 0u;
    // One atomic per entry, without a branch: a bit of a map, set by adding it (a sum that carries is not used), or a count.
    auto enter = [&](uint32_t col, int r, bool in) {
      const uint32_t bin = col & (uint32_t)(kBins - 1);
      const bool one = mapped && col < (uint32_t)kBins;
      const uint32_t bit = 1u << (r & 31);
      const uint32_t old = atomicAdd(one ? &map_word(bin, r >> 5) : &cursor[in ? bin : tid], one ? bit : in ? 1u : 0u);
      return one ? old & bit : 0u;
    };
    for (int g = 0; g < groups; ++g) {
      load(g);
#pragma unroll
      for (int q = 0; q < kHeld; ++q) again |= enter((uint32_t)c[q], g * held + q * kLiWaves + wave, c[q] >= 0);
      walk_far(g, [&](uint32_t col, int r, uint32_t, int32_t) { again |= enter(col, r, true); });
    }
    if (again != 0u) twice = 1u;
    __syncthreads();
    if (!mapped || twice == 0u) break;  // uniform: nobody writes it behind the barrier
    mapped = false;
  }
  part();
  // ---- first places and key slots: exclusive scans over the bins, one per thread (owner tid / 4); the mapped columns' pieces
  uint32_t all_keys = 0;
  {
    const int p = tid / kOwnBins, b = tid & (kOwnBins - 1), bin = b * P + p;
    const uint32_t n_key = cursor[bin];
    uint32_t n_one = 0, n_pieces = 0, most = n_key != 0u ? 1u : 0u;
    if (mapped)
      for (int w = 0; w < a.map_words; ++w) {
        if ((w & 1) == 0) ranks[w / 2 * kBins + bin] = (uint16_t)n_one;
        n_one += __popc(map_word(bin, w));
      }
    // A map's blocks: their numbers of bits.
    auto blocks = [&](auto f) {
      uint32_t prior = 0;
      for (int x = a.block; x < a.B; x += a.block) {  // uniform
        const uint32_t upto = rank_of(bin, x);
        f(upto - prior);
        prior = upto;
      }
      f(n_one - prior);
    };
    if (mapped)
      blocks([&](uint32_t n) {
        n_pieces += n != 0u ? 1u : 0u;
        most = max(most, n);
      });
    uint32_t sa = n_one + n_key, sb = n_key;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t ua = __shfl_up(sa, o, 64), ub = __shfl_up(sb, o, 64);
      if (lane >= o) { sa += ua; sb += ub; }
    }
    if (lane == 63) { total_a[wave] = sa; total_b[wave] = sb; }
    __syncthreads();
    uint32_t all = 0;
#pragma unroll 4
    for (int w = 0; w < kLiWaves; ++w) {
      if (w < wave) { sa += total_a[w]; sb += total_b[w]; }
      all += total_a[w];
      all_keys += total_b[w];
    }
    sa -= n_one + n_key;
    sb -= n_key;
    auto quad_sum = [&](uint32_t x) {  // of an owner's bins up to this one
      const uint32_t x1 = __shfl_up(x, 1, kOwnBins);
      x += b >= 1 ? x1 : 0u;
      const uint32_t x2 = __shfl_up(x, 2, kOwnBins);
      return x + (b >= 2 ? x2 : 0u);
    };
    const uint32_t list = __shfl(sa, 0, kOwnBins), one_at = quad_sum(n_one) - n_one;
    const uint32_t n_list = __shfl(sa + n_one + n_key, kOwnBins - 1, kOwnBins) - list;
    const uint32_t mine = n_pieces << 16 | (n_one != 0u ? 1u : 0u), upto = quad_sum(mine);
    most = max(most, __shfl_xor(most, 1, kOwnBins));
    most = max(most, __shfl_xor(most, 2, kOwnBins));
    cursor[bin] = sb;
    single_at[bin] = sa - sb;
    if (b == 0) {
      first[p] = list;
      slot0[p] = sb;
      one0[p] = sa - sb;
      longest[p] = most;
    }
    if (b == kOwnBins - 1) singles[p] = upto;
    if (n_one != 0u) {
      const uint32_t at = upto - mine;
      cols[list + (at & 0xffffu)] = (uint32_t)b + 1u;
      uint32_t k = list + (at >> 16), from = one_at;
      blocks([&](uint32_t n) {
        if (n == 0u) return;
        const uint32_t size = n_list <= 64u * kLiChunks ? n << 12 : 0u;
        pieces[k++] = from | size | (from + n == one_at + n_one ? kLast : 0u);
        from += n;
      });
    }
    if (tid == 0) { first[P] = all; slot0[P] = all_keys; one0[P] = all - all_keys; }
  }
  __syncthreads();
  auto bin_of = [&](uint32_t col) { return col & (uint32_t)(kBins - 1); };
  part();
  // ---- the mapped columns' entries, as many owners' at a time as there is room for (one's always: 4 B of them at most)
  for (int p0 = 0; mapped && p0 < P;) {
    const uint32_t base = one0[p0];
    int p1 = P;
    if (one0[P] - base > (uint32_t)n_stage) {
      int lo = p0 + 1, hi = P;
      while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (one0[mid] - base <= (uint32_t)n_stage) lo = mid; else hi = mid - 1;
      }
      p1 = lo;
    }
    part();
    const uint32_t room = one0[p1] - base;
    auto put = [&](uint32_t col, int r, uint32_t value) {
      if (col >= (uint32_t)kBins) return;  // (no entry: column 2^32 - 1)
      const uint32_t at = single_at[col] + rank_of(col, r) - base;
      if (at >= room) return;
      stage_value[at] = value;
      stage_pos[at] = (uint16_t)r;
    };
    for (int g = 0; g < groups; ++g) {
      if (groups > 1) load(g);
#pragma unroll
      for (int q0 = 0; q0 < kHeld; q0 += 8) {
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = row_words(a.vals, q0 + i);
#pragma unroll
        for (int i = 0; i < 8; ++i) put((uint32_t)c[q0 + i], g * held + (q0 + i) * kLiWaves + wave, v[i]);
      }
      walk_far(g, [&](uint32_t col, int r, uint32_t, int32_t e) { put(col, r, __float_as_uint(a.vals[e])); });
    }
    __syncthreads();
    part();
    for (int p = p0 + (tid >> 4); p < p1; p += kLiThreads / 16) {  // sixteen lanes a list
      const uint32_t from = one0[p] - base, n = one0[p + 1] - base - from;
      for (uint32_t i = tid & 15; i < n; i += 16) out[first[p] + i] = make_uint2(stage_pos[from + i], stage_value[from + i]);
    }
    __syncthreads();
    p0 = p1;
  }
  const uint32_t pos_mask = (1u << a.pos_bits) - 1u;
  const uint32_t per_block = a.block < a.B ? 65536u / (uint32_t)a.block + 1u : 0u;  // pos / block = pos * this >> 16, pos < 512
  auto place_of = [&](uint32_t pair) { return (pair >> a.pos_bits) << 4 | ((pair & pos_mask) * per_block) >> 16; };  // column, block
  // ---- as many owners at a time as the keys have room for (all of them unless rows are long)
  for (int p0 = 0; p0 < P;) {
    const uint32_t base = slot0[p0];
    int p1 = P;
    if (all_keys - base > (uint32_t)kKeyCap) {
      int lo = p0 + 1, hi = P;
      while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (slot0[mid] - base <= (uint32_t)kKeyCap) lo = mid; else hi = mid - 1;
      }
      p1 = lo;
    }
    const int n_keys = (int)(slot0[p1] - base), chunks = (n_keys + 63) / 64;
    __syncthreads();
    part();
    auto put_key = [&](uint32_t col, int r, uint32_t k, uint32_t slot, uint32_t value) {
      key_values[slot] = value;
      keys[slot] = ((col >> kOwnerBits) << a.pos_bits | (uint32_t)r) << a.k_bits | k;
      owner[slot] = (uint8_t)col;
    };
    const int32_t keyed = mapped ? kBins : 0;  // columns from there on
    auto mine = [&](uint32_t col) {  // (no entry: -1)
      return (int32_t)col >= keyed && (col & (uint32_t)(P - 1)) - (uint32_t)p0 < (uint32_t)(p1 - p0);
    };
    for (int g = 0; g < groups; ++g) {
      if (groups > 1 || p0 > 0) load(g);
#pragma unroll
      for (int q0 = 0; q0 < kHeld; q0 += 8) {
        uint32_t slot[8], v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = row_words(a.vals, q0 + i);
#pragma unroll
        for (int i = 0; i < 8; ++i) {  // (the others add nothing, each to a word of its own)
          const uint32_t col = (uint32_t)c[q0 + i];
          const bool has = mine(col);
          slot[i] = atomicAdd(&cursor[has ? bin_of(col) : (uint32_t)tid], has ? 1u : 0u) - base;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const uint32_t col = (uint32_t)c[q0 + i];
          if (mine(col)) put_key(col, g * held + (q0 + i) * kLiWaves + wave, (uint32_t)lane, slot[i], v[i]);
        }
      }
      walk_far(g, [&](uint32_t col, int r, uint32_t k, int32_t e) {
        if (mine(col)) put_key(col, r, k, atomicAdd(&cursor[bin_of(col)], 1u) - base, __float_as_uint(a.vals[e]));
      });
    }
#pragma unroll
    for (int q = 0; q < kHeld; ++q) c[q] = -1;  // (not kept for another turn)
    __syncthreads();
    part();
    // ---- the keys in order
    uint32_t key[kSortChunks], val[kSortChunks], to[kSortChunks];
#pragma unroll
    for (int i = 0; i < kSortChunks; ++i) {
      const int slot = 64 * (wave + i * kLiWaves) + lane;
      key[i] = val[i] = to[i] = 0u;
      if (slot < n_keys) {
        key[i] = keys[slot];
        val[i] = key_values[slot];
        const uint32_t p = owner[slot], b = (key[i] >> (a.pos_bits + a.k_bits)) & (uint32_t)(kOwnBins - 1);
        const uint32_t hi = cursor[b * P + p] - base, lo = b != 0u ? cursor[b * P + p - P] - base : slot0[p] - base;
        uint32_t n = lo;
        for (uint32_t k = lo; k < hi; k += 4) {  // (what lies behind the keys is LDS of this kernel)
          const uint32_t k0 = keys[k], k1 = keys[k + 1], k2 = keys[k + 2], k3 = keys[k + 3];
          n += k0 < key[i] ? 1u : 0u;
          n += k + 1 < hi && k1 < key[i] ? 1u : 0u;
          n += k + 2 < hi && k2 < key[i] ? 1u : 0u;
          n += k + 3 < hi && k3 < key[i] ? 1u : 0u;
        }
        to[i] = n;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortChunks; ++i)
      if (64 * (wave + i * kLiWaves) + lane < n_keys) {
        keys[to[i]] = key[i];
        key_values[to[i]] = val[i];
      }
    __syncthreads();
    part();
    // ---- entries, heads of columns and pieces
#pragma unroll
    for (int i = 0; i < kSortChunks; ++i) {
      const int chunk = wave + i * kLiWaves, slot = 64 * chunk + lane;
      if (chunk >= chunks) break;  // uniform
      bool col = false, piece = false;
      if (slot < n_keys) {
        key[i] = keys[slot];
        const uint32_t at = place_of(key[i] >> a.k_bits);
        const uint32_t prev = slot > 0 ? place_of(keys[slot - 1] >> a.k_bits) : 0u;
        col = slot == 0 || owner[slot] != owner[slot - 1] || at >> 4 != prev >> 4;
        piece = col || at != prev;
      }
      const uint64_t col_votes = __ballot(col), votes = __ballot(piece);
      if (lane == 0) { col_heads[chunk] = col_votes; heads[chunk] = votes; }
    }
    if (tid == 0) { col_heads[chunks] = 0u; heads[chunks] = 0u; }
    __syncthreads();
    if (wave == 0) {
      uint32_t sum = 0;
      for (int k = 0; k <= chunks; k += 64) {
        const uint32_t n = k + lane < chunks ? (uint32_t)__popcll(heads[k + lane]) << 16 | (uint32_t)__popcll(col_heads[k + lane]) : 0u;
        uint32_t s = n;
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t below = __shfl_up(s, o, 64);
          if (lane >= o) s += below;
        }
        if (k + lane <= chunks) before[k + lane] = sum + s - n;
        sum += read_lane(s, 63);
      }
    }
    __syncthreads();
    auto count = [&](int slot) {  // of heads below a slot: pieces << 16 | columns
      const uint64_t below = (1ull << (slot & 63)) - 1ull;
      return before[slot >> 6] + ((uint32_t)__popcll(heads[slot >> 6] & below) << 16 | (uint32_t)__popcll(col_heads[slot >> 6] & below));
    };
    part();
    for (int p = p0 + tid; p < p1; p += kLiThreads)  // (of the owner's heads before its first slot)
      singles[p] -= count((int)(slot0[p] - base));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kSortChunks; ++i) {
      const int slot = 64 * (wave + i * kLiWaves) + lane;
      if (slot < n_keys) {
        const uint32_t p = owner[slot], list = first[p], n_list = first[p + 1] - list;
        const int s1 = (int)(slot0[p + 1] - base);
        const uint32_t at = n_list - (uint32_t)(s1 - slot);  // in the list
        out[list + at] = make_uint2((key[i] >> a.k_bits) & pos_mask, key_values[slot]);
        const uint64_t votes = heads[slot >> 6], bit = 1ull << lane;
        if (votes & bit) {
          const uint32_t k = singles[p] + count(slot);
          if (col_heads[slot >> 6] & bit) cols[list + (k & 0xffffu)] = (key[i] >> (a.pos_bits + a.k_bits)) + 1u;
          int chunk = slot >> 6;
          uint64_t next = votes & ~bit & ~(bit - 1ull);
          while (next == 0ull && chunk + 1 < chunks) next = heads[++chunk];
          int end = next != 0ull ? 64 * chunk + __builtin_ctzll(next) : n_keys;  // (the next owner's first key is a head)
          const bool last = end >= s1 || ((col_heads[end >> 6] >> (end & 63)) & 1ull);
          const uint32_t size = (uint32_t)(end - slot);
          pieces[list + (k >> 16)] = at | (n_list <= 64u * kLiChunks ? size << 12 : 0u) | (last ? kLast : 0u);
          if (size > 1u) atomicMax(&longest[p], size);
        }
      }
    }
    __syncthreads();
    for (int p = p0 + tid; p < p1; p += kLiThreads) {
      const uint32_t k = singles[p] + count((int)(slot0[p + 1] - base));
      uint32_t *rec = a.rec + ((int64_t)blockIdx.x * P + p) * kRecord;
      rec[0] = first[p];
      rec[1] = first[p + 1] - first[p];
      rec[2] = k & 0xffffu;
      rec[3] = k >> 16;
      rec[4] = longest[p];
    }
    __syncthreads();
    p0 = p1;
  }
}

// Snapshot margins of the planned rows where the snapshot pass did not visit every row: sixteen lanes per row, in the order
// of the worker pass (lpc_csr.hip).
__global__ __launch_bounds__(256) void plan_margins_kernel(const int32_t *__restrict__ col_idx, const float *__restrict__ vals,
                                                           const float *__restrict__ w_snap, int64_t rows,
                                                           RowPlan *__restrict__ plan) {
  const int64_t r = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  if (r >= rows) return;  // whole rows of sixteen lanes
  const RowPlan p = plan[r];
  float s = 0.0f;
  for (int32_t e = p.lo + (int32_t)(threadIdx.x & 15); e < p.hi; e += 16) s = __builtin_fmaf(vals[e], w_snap[col_idx[e]], s);
  s = row16_sum(s);
  if ((threadIdx.x & 15) == 0) plan[r].z = s;
}

// out[0]: entries of the longest row; out[1]: the most entries of a row that belong to one owner.  A wavefront per row and turn.
__global__ __launch_bounds__(256) void row_extents_kernel(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx,
                                                          int64_t n, int32_t *__restrict__ out) {
  __shared__ uint32_t entries[4][kOwners];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t *mine = entries[wave];
  for (int i = lane; i < kOwners; i += 64) mine[i] = 0u;
  __syncthreads();
  int32_t longest = 0, most = 0;
  for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < n; r += (int64_t)gridDim.x * 4) {
    const int32_t lo = row_ptr[r], hi = row_ptr[r + 1];
    longest = hi - lo > longest ? hi - lo : longest;
    for (int32_t e = lo + lane; e < hi; e += 64) most = max(most, (int32_t)atomicAdd(&mine[col_idx[e] & (kOwners - 1)], 1u) + 1);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int32_t e = lo + lane; e < hi; e += 64) mine[col_idx[e] & (kOwners - 1)] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
  if (lane == 0) {
    atomicMax(&out[0], longest);
    atomicMax(&out[1], most);
  }
}

// ---------------------------------------------------------------------------------------------------------------------
// A vector between the caller's order and the owners' (element lc of owner p = coordinate lc P + p), a tile of 32 lc by 64 p.
struct DealArgs {
  const float *from[4];
  float *to[4];
  float scale[4];
  const uint32_t *ctl;  // dealt back: not where a launch with this tag gave up
  uint32_t launch_tag;
  int32_t d, S, pshift, back;
};

__global__ __launch_bounds__(256) void deal_kernel(DealArgs a) {
  if (a.back && a.ctl[0] == a.launch_tag) return;
  __shared__ float tile[32][65];
  const float *from = a.from[blockIdx.z];
  float *to = a.to[blockIdx.z];
  const int l0 = blockIdx.x * 32, p0 = blockIdx.y * 64, P = 1 << a.pshift;
  if (!a.back) {
    for (int e = threadIdx.x; e < 32 * 64; e += 256) {
      const int l = e >> 6, p = e & 63;
      const int64_t c = (int64_t)(l0 + l) * P + p0 + p;
      tile[l][p] = c < a.d ? from[c] : 0.0f;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * 64; e += 256) {
      const int p = e >> 5, l = e & 31;
      if (l0 + l < a.S) to[(int64_t)(p0 + p) * a.S + l0 + l] = tile[l][p];
    }
  } else {
    const float scale = a.scale[blockIdx.z];
    for (int e = threadIdx.x; e < 32 * 64; e += 256) {
      const int p = e >> 5, l = e & 31;
      tile[l][p] = l0 + l < a.S ? from[(int64_t)(p0 + p) * a.S + l0 + l] : 0.0f;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 32 * 64; e += 256) {
      const int l = e >> 6, p = e & 63;
      const int64_t c = (int64_t)(l0 + l) * P + p0 + p;
      if (c < a.d) to[c] = tile[l][p] * scale;
    }
  }
}

// ---------------------------------------------------------------------------------------------------------------------
struct ListArgs {
  const int32_t *col_idx;
  const float *vals;
  const RowPlan *plan;     // [iterations][nvec * B] of this launch
  const uint32_t *rec;     // of this launch
  uint2 *ent;
  const uint32_t *cols;
  uint32_t *pieces;
  int64_t cap;
  const float *mu, *ws;    // the owners' order, here and below
  float *x, *y, *z, *ysum;
  // [P][S]; [2][nvec * B]; [2][N][5][P]; [2][N][dies][kLine]
  u64 *xw, *slope, *stat, *stat2;
  uint32_t *flags, *ctl;
  int32_t d, S, pshift, block, N, nvec, B, it0, it1, bits, fields, words, scheme, loss;
  uint32_t tag0, spin_limit;
  QuantSpec qs;
  StreamKey key;
  float scale, step, thr, shrink;
  float step_y, thr_y, shrink_y, alpha, thr_z, shrink_z, t1, t2, t3;
  double theta, weight;
};

// PLAIN: lambda clipping and scale factors of the workers' own (scheme (a)), the paper's way in all its experiments.
// Everything that is requested ahead goes through buffers, whose lanes past the end read 0: a load under a condition is joined
// with the other case's value, and the join waits for it.
template <bool ALPC, bool PLAIN>
__global__ __launch_bounds__(kLiThreads) void list_epoch_kernel(ListArgs a) {
  touch_kernel_arguments<(int)(sizeof(ListArgs))>();
  extern __shared__ __attribute__((aligned(16))) float lds[];
  __shared__ float delta_sh[kLiWaves];
  __shared__ uint32_t fail_sh[2], count[3], over_sh;
  // a wavefront's own: products on their way to their pieces' lanes, then the pieces' sums to their columns'
  __shared__ float stage[kLiWaves][64 * kLiChunks + 8];
  const int S = a.S;
  float *xs = lds, *mus = xs + S;
  float *zs = mus + S, *ysums = zs + (ALPC ? S : 0), *wss = ysums + (ALPC ? S : 0), *uhs = wss + (ALPC ? S : 0);
  uint32_t *codes = reinterpret_cast<uint32_t *>(uhs + (ALPC ? S : 0));  // [words][S]
  uint32_t *marks = codes + a.words * S;                                   // [3][(S + 31) / 32]: set t % 3 the columns of t
  const int mark_words = (S + 31) / 32;
  uint16_t *touched = reinterpret_cast<uint16_t *>(marks + 3 * mark_words);  // [2][S]
  int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int p = blockIdx.x, P = 1 << a.pshift, die = p & (kDies - 1), per_die = P / kDies;

  // an earlier launch of this epoch gave up
  if (tid == 0) over_sh = __hip_atomic_load(a.ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.tag0 + 1u ? 1u : 0u;
  if (tid < 3) count[tid] = 0u;
  if (tid < 2) fail_sh[tid] = 0u;
  if (tid < kLiWaves) delta_sh[tid] = 0.0f;
  for (int l = tid; l < S; l += kLiThreads) {
    const int64_t at = (int64_t)p * S + l;
    mus[l] = a.mu[at];
    if (ALPC) {
      const float z = a.z[at], w = a.ws[at], y = a.y[at];
      zs[l] = z;
      wss[l] = w;
      uhs[l] = 0.0f;
      ysums[l] = a.it0 > 0 ? a.ysum[at] : 0.0f;
      xs[l] = (a.t1 * z + a.t2 * w) + a.t3 * y;
    } else {
      xs[l] = a.it0 > 0 ? a.x[at] : a.ws[at];
    }
  }
  for (int e = tid; e < a.words * S; e += kLiThreads) codes[e] = 0u;
  for (int e = tid; e < 3 * mark_words; e += kLiThreads) marks[e] = 0u;
  __syncthreads();
  if (over_sh) return;  // uniform

  // `loads` requests the words that a lane still lacks and says whether all are there; the wavefront waits as one.  (Words that
  // are there are not asked for again: what polls is in the way of what they wait for.)
  auto poll = [&](uint32_t limit, bool &ok, auto loads) {
    if (!ok) return;
    for (uint32_t k = 0; k < limit; ++k) {
      if (__ballot(!loads()) == 0ull) return;
      if ((k & 63u) == 63u &&
          __builtin_amdgcn_readfirstlane((int)__hip_atomic_load(a.ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) ==
              (int)(a.tag0 + 1u))
        break;
    }
    ok = false;
  };
  // ---- rows of this wavefront: batch positions of all vectors, consecutive ones in a workgroup (their slopes share a line)
  const int total_rows = a.nvec * a.B;
  int slot[kLiRows];
  bool has_row[kLiRows];
#pragma unroll
  for (int q = 0; q < kLiRows; ++q) {
    slot[q] = (q * P + p) * kLiWaves + wave;
    has_row[q] = slot[q] < total_rows;
  }
  typedef uint32_t words4 __attribute__((ext_vector_type(4)));
  typedef uint32_t words2 __attribute__((ext_vector_type(2)));
  words4 row[kLiRows];   // a RowPlan: first entry, end, label, snapshot slope
  int32_t len[kLiRows];
  uint32_t rx[kLiRows];  // of lane l: the column of the row's entry l, then where its x word lies, in bytes; kNoEntry: none
  uint32_t rv[kLiRows];  // ... and the entry's value
  auto x_at = [&](uint32_t c) { return 8u * ((c & (uint32_t)(P - 1)) * (uint32_t)S + (c >> a.pshift)); };
  auto x_word = [&](uint32_t at) { return ld_word(reinterpret_cast<const u64 *>(reinterpret_cast<const char *>(a.xw) + at)); };
  auto fetch_rows = [&](int t) {
#pragma unroll
    for (int q = 0; q < kLiRows; ++q)
      row[q] = __builtin_amdgcn_raw_buffer_load_b128(buffer(a.plan + (int64_t)(t - a.it0) * total_rows + slot[q], has_row[q] ? 16u : 0u), 0, 0, 0);
  };
  auto fetch_pairs = [&]() {
#pragma unroll
    for (int q = 0; q < kLiRows; ++q) {
      const int32_t lo = __builtin_amdgcn_readfirstlane((int)row[q].x);
      len[q] = __builtin_amdgcn_readfirstlane((int)row[q].y) - lo;
      rx[q] = __builtin_amdgcn_raw_buffer_load_b32(buffer(a.col_idx + lo, 4u * (uint32_t)len[q]), 4 * lane, 0, 0);
      rv[q] = __builtin_amdgcn_raw_buffer_load_b32(buffer(a.vals + lo, 4u * (uint32_t)len[q]), 4 * lane, 0, 0);
    }
  };
  // ---- this wavefront's list: vector `wave`'s entries in this workgroup's columns
  const bool quantizes = wave < a.N, listed = wave < a.nvec;
  // the shared batch's vector where the workers have all wavefronts
  const bool adds_shared = ALPC && a.N == kLiWaves && wave == 0;
  struct List {
    int64_t at;      // its first entry
    int32_t n;       // entries
    int32_t cols;    // columns
    int32_t pieces;  // runs of one column and one block of batch positions
    int32_t longest; // entries of the longest one
  };
  // lane l: word l of the list's record
  auto bounds_of = [&](int t, int v) {
    return a.rec[(((int64_t)(t - a.it0) * a.nvec + v) * P + p) * kRecord + (lane < kRecord ? lane : 0)];
  };
  auto list_of = [&](int t, int v, uint32_t b) {
    return List{((int64_t)(t - a.it0) * a.nvec + v) * a.cap + read_lane(b, 0), (int32_t)read_lane(b, 1), (int32_t)read_lane(b, 2),
                (int32_t)read_lane(b, 3), (int32_t)read_lane(b, 4)};
  };
  auto is_long = [&](const List &l) { return l.n > 64 * kLiChunks || l.pieces > 64 * kLiPairs; };
  words2 ent[kLiChunks], ent_n[kLiChunks];
  uint32_t col[kLiPairs], col_n[kLiPairs];  // lc + 1; a lane without a column: 0
  uint32_t piece[kLiPairs], piece_n[kLiPairs];  // a lane without a piece: 0
  List list{0, 0, 0, 0, 0}, list_n{0, 0, 0, 0, 0};
  uint32_t bounds = 0;
  auto fetch_list = [&](const List &l, words2 (&e)[kLiChunks], uint32_t (&c)[kLiPairs], uint32_t (&f)[kLiPairs]) {
#pragma unroll
    for (int r = 0; r < kLiChunks; ++r) {
      e[r] = words2{0u, 0u};
      if (r * 64 < l.n)  // uniform
        e[r] = __builtin_amdgcn_raw_buffer_load_b64(buffer(a.ent + l.at, 8u * (uint32_t)l.n), 8 * lane + 512 * r, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < kLiPairs; ++k) {
      c[k] = 0u;
      if (k * 64 < l.cols) c[k] = __builtin_amdgcn_raw_buffer_load_b32(buffer(a.cols + l.at, 4u * (uint32_t)l.cols), 4 * lane + 256 * k, 0, 0);
      f[k] = 0u;
      if (k * 64 < l.pieces)
        f[k] = __builtin_amdgcn_raw_buffer_load_b32(buffer(a.pieces + l.at, 4u * (uint32_t)l.pieces), 4 * lane + 256 * k, 0, 0);
    }
  };
  // the coming iteration's touched columns, each once
  auto mark = [&](int t, uint32_t lc1) {
    bool first = false;
    const uint32_t lc = lc1 - 1u;
    if (lc1 != 0u) {
      const uint32_t bit = 1u << (lc & 31u);
      first = !(atomicOr(&marks[(t % 3) * mark_words + (lc >> 5)], bit) & bit);
    }
    const uint64_t m = __ballot(first);
    if (m == 0ull) return;
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&count[t % 3], (uint32_t)__popcll(m));
    at = __builtin_amdgcn_readfirstlane((int)at);
    if (first) touched[(t & 1) * S + at + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)lc;
  };
  auto mark_from = [&](int t, const List &l, int i) {  // columns i .. from memory
    for (; i < l.cols; i += 64) mark(t, i + lane < l.cols ? a.cols[l.at + i + lane] : 0u);
  };
  auto mark_list = [&](int t, const List &l, const uint32_t (&c)[kLiPairs]) {
#pragma unroll
    for (int k = 0; k < kLiPairs; ++k)
      if (k * 64 < l.cols) mark(t, c[k]);
    mark_from(t, l, 64 * kLiPairs);
  };
  auto put_x = [&](int t, uint32_t lc, float x) {  // the iterate where iteration t's rows look
    st_word(a.xw + (uint32_t)(p * S) + lc, __builtin_bit_cast(uint32_t, x), a.tag0 + (uint32_t)t + 1u);
  };
  auto staged = [] {  // what the wavefront wrote to its stage is there, what it read has been read
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  // The wait for all that has been requested ahead, before the next words are stored: a wait for a load behind a store is one
  // for the store to arrive as well.
  auto settle = [&] {
#pragma unroll
    for (int q = 0; q < kLiRows; ++q) {
      rx[q] = lane < len[q] ? x_at(rx[q]) : kNoEntry;
      asm volatile("" : "+v"(rx[q]), "+v"(rv[q]), "+v"(row[q]));
    }
#pragma unroll
    for (int r = 0; r < kLiChunks; ++r) asm volatile("" : "+v"(ent_n[r]));
#pragma unroll
    for (int k = 0; k < kLiPairs; ++k) asm volatile("" : "+v"(col_n[k]), "+v"(piece_n[k]));
    asm volatile("" : "+v"(bounds));
  };
  if (listed) {
    list_n = list_of(a.it0, wave, bounds_of(a.it0, wave));
    bounds = bounds_of(a.it0 + 1 < a.it1 ? a.it0 + 1 : a.it0, wave);
  }
  fetch_list(list_n, ent_n, col_n, piece_n);
  if (listed) mark_list(a.it0, list_n, col_n);
  if (adds_shared) mark_from(a.it0, list_of(a.it0, a.N, bounds_of(a.it0, a.N)), 0);
  fetch_rows(a.it0);
  fetch_pairs();
  settle();
  __syncthreads();
  for (uint32_t i = tid; i < count[a.it0 % 3]; i += kLiThreads) {
    const uint32_t lc = touched[(a.it0 & 1) * S + i];
    put_x(a.it0, lc, xs[lc]);
  }

  const bool csigma = !PLAIN && a.qs.clip_mode != LPC_CLIP_LAMBDA;
  const float inv_n = 1.0f / (float)a.N;
  const float hi_q = (float)((1 << a.bits) / 2 - 1), lo_q = -(float)((1 << a.bits) / 2);
  const uint32_t mask = (1u << a.bits) - 1u;
  const int my_word = wave / a.fields, my_shift = (wave - my_word * a.fields) * a.bits;
  double weight = a.weight;
  bool gave_up = false;
  // What derives from these alone is computed again in every iteration: kept, it is 35 registers, which spilled.
  auto part = [&] {
    asm volatile("" : "+v"(tid));
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  };
  for (int t = a.it0; t < a.it1; ++t) {
    if constexpr (ALPC) part();
    const int par = t & 1;
    const uint32_t tag = a.tag0 + (uint32_t)t + 1u;
    const uint32_t limit = t == a.it0 ? (a.spin_limit > 0xffffffu ? ~0u : a.spin_limit * 256u) : a.spin_limit;
    const bool more = t + 1 < a.it1;
    bool ok = true;
    auto there = [&](u64 w) { return (uint32_t)(w >> 32) == tag; };
    list = list_n;
#pragma unroll
    for (int r = 0; r < kLiChunks; ++r) ent[r] = ent_n[r];
#pragma unroll
    for (int k = 0; k < kLiPairs; ++k) { col[k] = col_n[k]; piece[k] = piece_n[k]; }
    // ---- 1. the rows' margins and slope differences
    __builtin_amdgcn_s_setprio(3);
    {
      u64 xw[kLiRows];
#pragma unroll
      for (int q = 0; q < kLiRows; ++q) xw[q] = rx[q] != kNoEntry ? 0ull : (u64)tag << 32;
      poll(limit, ok, [&] {
        bool all = true;
#pragma unroll
        for (int q = 0; q < kLiRows; ++q)
          if (!there(xw[q])) xw[q] = x_word(rx[q]);
#pragma unroll
        for (int q = 0; q < kLiRows; ++q) all = all && there(xw[q]);
        return all;
      });
#pragma unroll
      for (int q = 0; q < kLiRows; ++q) {
        if (!has_row[q]) continue;  // uniform
        // Lane l < 16 adds the entries l, l + 16, ..., then the sixteen lanes, as the worker pass of lpc_csr.hip does: the margin of
        // x~ is then the snapshot pass's, and an epoch's numbers are those of the separate launches.  (Lanes past the row's
        // end: 0 * 0.)
        float s = 0.0f;
        auto add_rows = [&](uint32_t v, uint32_t x) {  // four entries per lane, of the four rows of sixteen lanes
          const auto v1 = __builtin_amdgcn_permlane16_swap(v, v, false, false), x1 = __builtin_amdgcn_permlane16_swap(x, x, false, false);
          const auto v2 = __builtin_amdgcn_permlane32_swap(v, v, false, false), x2 = __builtin_amdgcn_permlane32_swap(x, x, false, false);
          const uint32_t va = v1[1], xa = x1[1];
          const auto v3 = __builtin_amdgcn_permlane32_swap(va, va, false, false), x3 = __builtin_amdgcn_permlane32_swap(xa, xa, false, false);
          const uint32_t vb = v2[1], xb = x2[1], vc = v3[1], xc = x3[1];
          s = __builtin_fmaf(__builtin_bit_cast(float, v), __builtin_bit_cast(float, x), s);
          s = __builtin_fmaf(__builtin_bit_cast(float, va), __builtin_bit_cast(float, xa), s);
          s = __builtin_fmaf(__builtin_bit_cast(float, vb), __builtin_bit_cast(float, xb), s);
          s = __builtin_fmaf(__builtin_bit_cast(float, vc), __builtin_bit_cast(float, xc), s);
        };
        add_rows(rv[q], (uint32_t)xw[q]);
        for (int32_t k = 64; k < len[q]; k += 64) {  // rows longer than 64 entries
          const int64_t e = (int32_t)row[q].x + (k + lane < len[q] ? k + lane : len[q] - 1);
          const uint32_t at = x_at((uint32_t)a.col_idx[e]);
          const float v = a.vals[e];
          u64 far = 0;
          poll(limit, ok, [&] { if (!there(far)) far = x_word(at); return there(far); });
          const bool in = k + lane < len[q];
          add_rows(in ? __builtin_bit_cast(uint32_t, v) : 0u, in ? (uint32_t)far : 0u);
        }
        s = row16_sum(s);
        const float z = read_lane(s, 0);
        // (x_0 of Alg. 1 is the snapshot: zero, or NaN where the slope is; the builder left the snapshot's slope in row.z)
        const uint32_t label = row[q].z, snap = row[q].w;
        const float diff = loss_slope(a.loss, z, __builtin_bit_cast(float, label)) - __builtin_bit_cast(float, snap);
        const float coef = diff * a.scale;
        if (lane == 0) st_word(a.slope + par * total_rows + slot[q], __builtin_bit_cast(uint32_t, coef), tag);
      }
    }
    __builtin_amdgcn_s_setprio(1);
    // ---- while the slopes travel: the coming iteration's rows and entries requested, this one's random words
    {
      const int t1 = more ? t + 1 : t;  // (the last one's own again, to no purpose)
      fetch_rows(t1);
      list_n = list_of(t1, wave, bounds);
      if (!listed) list_n.n = list_n.cols = list_n.pieces = list_n.longest = 0;
      fetch_list(list_n, ent_n, col_n, piece_n);
      bounds = bounds_of(t + 2 < a.it1 ? t + 2 : t1, listed ? wave : 0);
    }
    auto random_word = [&](uint32_t lc) {
      StreamKey k = a.key;
      k.iter = (uint32_t)t;
      const Philox4 b = stream_block(k, kTagQuant, (uint32_t)wave, (lc << (a.pshift - 2)) | ((uint32_t)p >> 2));
      return (p & 2) ? ((p & 1) ? b.w : b.z) : ((p & 1) ? b.y : b.x);
    };
    uint32_t rnd[kLiPairs];
    float u[kLiPairs];
#pragma unroll
    for (int k = 0; k < kLiPairs; ++k) {
      rnd[k] = 0u;
      u[k] = 0.0f;
      if (quantizes && k * 64 < list.cols) rnd[k] = random_word(col[k] - 1u);
    }
    // ---- 2. u^i at this workgroup's columns
    // Sums over the pieces of a column, piece after piece, at its last one (chunk of 64 pieces; `open`: the sum of the pieces of
    // its first column in the chunk before, if it goes on).  After j turns a lane has its column's sum if it is the piece j.
    const int blocks = (a.B + a.block - 1) / a.block;
    auto sum_pieces = [&](float part, uint64_t ends, float &open, bool &closed) {
      const uint64_t heads = (ends << 1) | (closed ? 1ull : 0ull);
      const bool head = (heads >> lane) & 1ull;
      float s = part;
      for (int j = 1; j < blocks; ++j) {
        const float below = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, open), __builtin_bit_cast(int, s),
                                                                                  0x138, 0xF, 0xF, false));  // wave_shr:1
        s = head ? part : below + part;
      }
      open = read_lane(s, 63);
      closed = (ends >> 63) & 1ull;
      return s;
    };
    // A list in memory: products in the entries' place, then the k-th column's sum in that of the k-th piece (which has been
    // read by then).
    auto form_long = [&](const List &l, int v) {
      const u64 *sl = a.slope + par * total_rows + v * a.B;
      for (int i = 0; i < l.n; i += 64) {
        const uint2 e = a.ent[l.at + (i + lane < l.n ? i + lane : l.n - 1)];
        u64 f = 0;
        poll(limit, ok, [&] { if (!there(f)) f = ld_word(sl + e.x); return there(f); });
        if (i + lane < l.n)
          a.ent[l.at + i + lane].y = __float_as_uint(__uint_as_float((uint32_t)f) * __uint_as_float(e.y));
      }
      __threadfence_block();  // other lanes read the products
      auto begin_of = [&](uint32_t f) { return (int32_t)(f & (l.n > 64 * kLiChunks ? ~kLast : 0xfffu)); };
      float open = 0.0f;
      bool closed = true;
      int n = 0;
      for (int i = 0; i < l.pieces; i += 64) {
        const bool in = i + lane < l.pieces;
        const uint32_t f = in ? a.pieces[l.at + i + lane] : 0u;
        const int32_t end = i + lane + 1 < l.pieces ? begin_of(a.pieces[l.at + i + lane + 1]) : l.n;
        float part = 0.0f;
        if (in)
          for (int32_t k = begin_of(f); k < end; ++k) part += __uint_as_float(a.ent[l.at + k].y);
        const uint64_t ends = __ballot((f & kLast) != 0u);
        const float s = sum_pieces(part, ends, open, closed);
        if ((ends >> lane) & 1ull) a.pieces[l.at + n + __popcll(ends & ((1ull << lane) - 1ull))] = __builtin_bit_cast(uint32_t, s);
        n += __popcll(ends);
      }
      __threadfence_block();  // other lanes read the sums
    };
    auto sum_at = [&](const List &l, int k) { return __builtin_bit_cast(float, a.pieces[l.at + k]); };
    float mx = 0.0f;
    double sum = 0.0, sumsq = 0.0;
    bool bad = false;
    auto take = [&](float v) {
      const bool fin = isfinite(v);
      const float f = fin ? v : 0.0f;
      bad |= !fin;
      mx = fmaxf(mx, fabsf(f));
      if (csigma) { sum += (double)f; sumsq += (double)f * (double)f; }
    };
    const bool long_list = is_long(list);
    if (listed) {
      if (!long_list) {
        const u64 *sl = a.slope + par * total_rows + wave * a.B;
        u64 w[kLiChunks];
#pragma unroll
        for (int r = 0; r < kLiChunks; ++r) w[r] = r * 64 + lane < list.n ? 0ull : (u64)tag << 32;
        __builtin_amdgcn_s_setprio(0);
        poll(limit, ok, [&] {
          bool all = true;
#pragma unroll
          for (int r = 0; r < kLiChunks; ++r)
            if (r * 64 < list.n && !there(w[r])) w[r] = ld_word(sl + ent[r].x);
#pragma unroll
          for (int r = 0; r < kLiChunks; ++r) all = all && there(w[r]);
          return all;
        });
        __builtin_amdgcn_s_setprio(3);
        // Products to their pieces' lanes, each of which adds its own one after the other; the order is that of the worker pass
        // (rows of a block in batch order, then the blocks).
        float *mine = stage[wave];
#pragma unroll
        for (int r = 0; r < kLiChunks; ++r) {
          const uint32_t value = ent[r].y;
          if (r * 64 < list.n) mine[r * 64 + lane] = __builtin_bit_cast(float, (uint32_t)w[r]) * __builtin_bit_cast(float, value);
        }
        staged();
#pragma unroll
        for (int k = 0; k < kLiPairs; ++k) {
          if (k * 64 < list.pieces) {
            const int first = (int)(piece[k] & 0xfffu), size = (int)((piece[k] >> 12) & 0xfffu);
            float s = mine[first];
            if (list.longest > 1) {  // uniform
              // eight at a time, requested ahead, as long as a lane has them; then each lane's last ones (-0: nothing added).
              // Lanes that have no more read one address together: 64 addresses at random are five times the LDS's work.
              const int rest = size > 1 ? 1 + ((size - 1) & ~7) : 1;
              const float *end = mine + (rest < size ? first + rest : 0);
              float last[7];
#pragma unroll
              for (int i = 0; i < 7; ++i) last[i] = end[i];
              if (list.longest > 8) {
                auto from = [&](int i) { return mine + (i + 8 <= size ? first + i : 0); };
                float now[8];
                const float *p = from(1);
#pragma unroll
                for (int i = 0; i < 8; ++i) now[i] = p[i];
                for (int done = 1; done + 8 <= list.longest; done += 8) {
                  float next[8];
                  p = from(done + 8);
#pragma unroll
                  for (int i = 0; i < 8; ++i) next[i] = p[i];
                  float eight = s;
#pragma unroll
                  for (int i = 0; i < 8; ++i) eight += now[i];
                  s = done + 8 <= size ? eight : s;
#pragma unroll
                  for (int i = 0; i < 8; ++i) now[i] = next[i];
                }
              }
#pragma unroll
              for (int i = 0; i < 7; ++i) s += rest + i < size ? last[i] : -0.0f;
            }
            u[k] = s;
          }
        }
        if (list.pieces != list.cols) {  // uniform
          float open = 0.0f;
          bool closed = true;
          int n = 0;
          staged();
#pragma unroll
          for (int k = 0; k < kLiPairs; ++k) {
            if (k * 64 < list.pieces) {
              const uint64_t ends = __ballot((piece[k] & kLast) != 0u);
              const float s = sum_pieces(u[k], ends, open, closed);
              if ((ends >> lane) & 1ull) mine[n + __popcll(ends & ((1ull << lane) - 1ull))] = s;
              n += __popcll(ends);
            }
          }
          staged();
#pragma unroll
          for (int k = 0; k < kLiPairs; ++k)
            if (k * 64 < list.cols) u[k] = mine[k * 64 + lane];
        }
#pragma unroll
        for (int k = 0; k < kLiPairs; ++k) {
          if (k * 64 < list.cols) {
            if (col[k] == 0u) u[k] = 0.0f;
            take(u[k]);
            if (ALPC && !quantizes && col[k] != 0u) uhs[col[k] - 1u] = u[k];
          }
        }
      } else {
        form_long(list, wave);
        for (int k = lane; k < list.cols; k += 64) {
          take(sum_at(list, k));
          if (ALPC && !quantizes) uhs[a.cols[list.at + k] - 1u] = sum_at(list, k);
        }
      }
    }
    if (quantizes) {
      mx = wave_max(mx);
      if (csigma) { sum = wave_sum(sum); sumsq = wave_sum(sumsq); }
      if (__ballot(bad) != 0ull && lane == 0) atomicOr(&a.flags[0], 1u);
      u64 *st = a.stat + ((int64_t)par * a.N + wave) * 5 * P + die * per_die + p / kDies;
      uint32_t mine = __builtin_bit_cast(uint32_t, mx);
      if (csigma) {
        const u64 s = __builtin_bit_cast(u64, sum), s2 = __builtin_bit_cast(u64, sumsq);
        if (lane > 0) mine = (uint32_t)((lane < 3 ? s : s2) >> (lane & 1 ? 0 : 32));
      }
      if (lane < (csigma ? 5 : 1)) st_word(st + (int64_t)lane * P, mine, tag);
    }
    // One wavefront per vector and die takes the statistics of its die's owners together, every wavefront those of the dies:
    // all owners' words read by all of them are 8 MB for 16 vectors.
    float am = 0.0f;
    auto gather = [&](const u64 *from, int64_t stride, int words) {  // words <= 64, of lanes 0 .. words - 1
      u64 h[5] = {};
      poll(limit, ok, [&] {
        bool all = true;
#pragma unroll
        for (int i = 0; i < (PLAIN ? 1 : 5); ++i)
          if ((i == 0 || csigma) && !there(h[i])) h[i] = ld_word(from + i * stride);
#pragma unroll
        for (int i = 0; i < (PLAIN ? 1 : 5); ++i) all = all && (there(h[i]) || (i > 0 && !csigma));
        return all;
      });
      am = wave_max(__builtin_bit_cast(float, (uint32_t)h[0]));
      if (csigma) {
        const double d1 = __builtin_bit_cast(double, (h[1] & 0xffffffffull) | (h[2] << 32));
        const double d2 = __builtin_bit_cast(double, (h[3] & 0xffffffffull) | (h[4] << 32));
        sum = wave_sum(lane < words ? d1 : 0.0);
        sumsq = wave_sum(lane < words ? d2 : 0.0);
      }
    };
    if (quantizes && p / kDies == wave * per_die / kLiWaves) {
      gather(a.stat + ((int64_t)par * a.N + wave) * 5 * P + die * per_die + (lane < per_die ? lane : per_die - 1), P, per_die);
      uint32_t mine = __builtin_bit_cast(uint32_t, am);
      if (csigma) {
        const u64 s = __builtin_bit_cast(u64, sum), s2 = __builtin_bit_cast(u64, sumsq);
        if (lane > 0) mine = (uint32_t)((lane < 3 ? s : s2) >> (lane & 1 ? 0 : 32));
      }
      if (lane < (csigma ? 5 : 1)) st_word(a.stat2 + (((int64_t)par * a.N + wave) * kDies + die) * kLine + lane, mine, tag);
    }
    __builtin_amdgcn_s_setprio(0);
    // ---- while the statistics travel: the coming rows' pairs and columns, and the coordinates that no row of this iteration
    // touches
    fetch_pairs();
    for (int l = 4 * tid; l < S; l += 4 * kLiThreads) {  // S is a multiple of four
      const uint32_t taken = marks[(t % 3) * mark_words + (l >> 5)] >> (l & 31);
      const float4 m4 = *reinterpret_cast<const float4 *>(mus + l);
      float4 x4 = *reinterpret_cast<const float4 *>(xs + l);
      float *x = &x4.x;
      const float *m = &m4.x;
      if (ALPC) {
        float4 z4 = *reinterpret_cast<const float4 *>(zs + l), sum4 = *reinterpret_cast<const float4 *>(ysums + l);
        const float4 w4 = *reinterpret_cast<const float4 *>(wss + l);
        float *z = &z4.x, *acc = &sum4.x;
        const float *w = &w4.x;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float yn = prox_scalar(x[c], 0.0f + m[c], a.step_y, a.thr_y, a.shrink_y);
          const float zn = prox_scalar(z[c], 0.0f + m[c], a.alpha, a.thr_z, a.shrink_z);
          const bool stays = (taken >> c) & 1u;
          z[c] = stays ? z[c] : zn;
          acc[c] = stays ? acc[c] : (t == 0 ? (float)weight * yn : acc[c] + (float)weight * yn);
          x[c] = stays ? x[c] : (a.t1 * zn + a.t2 * w[c]) + a.t3 * yn;
          if (!more && !stays) a.y[(int64_t)p * S + l + c] = yn;
        }
        *reinterpret_cast<float4 *>(zs + l) = z4;
        *reinterpret_cast<float4 *>(ysums + l) = sum4;
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const float xn = prox_scalar(x[c], 0.0f + m[c], a.step, a.thr, a.shrink);
          x[c] = (taken >> c) & 1u ? x[c] : xn;
        }
      }
      *reinterpret_cast<float4 *>(xs + l) = x4;
    }
    if (adds_shared) {  // the shared batch's difference, in full precision
      const List l = list_of(t, a.N, bounds_of(t, a.N));
      form_long(l, a.N);
      for (int k = lane; k < l.cols; k += 64) uhs[a.cols[l.at + k] - 1u] = sum_at(l, k);
      if (more) mark_from(t + 1, list_of(t + 1, a.N, bounds_of(t + 1, a.N)), 0);
    }
    if (more && listed) mark_list(t + 1, list_n, col_n);
    // ---- 3. the scale factors (Sec. 3.2, eq. (3)), as in lpc_columns.hip
    QParams q{0.0f, 0.0f, 0.0f, 0.0f};
    if (quantizes) {
      gather(a.stat2 + (((int64_t)par * a.N + wave) * kDies + (lane & (kDies - 1))) * kLine, 1, kDies);
      if (csigma) {
        q = make_qparams(a.qs, (double)am, sum, sumsq, a.d);
      } else {
        const float delta = a.qs.clip * am / hi_q, rd = 1.0f / delta;
        const bool live = delta > 0.0f && isfinite(rd);
        q.delta = live ? delta : 0.0f;
        q.rdelta = live ? rd : 0.0f;
      }
      if (lane == 0) delta_sh[wave] = q.delta;
    }
    if (!PLAIN && a.scheme != LPC_SCHEME_A) {  // the largest of the N scale factors
      __syncthreads();
      const float dmax = wave_max(lane < a.N ? delta_sh[lane] : 0.0f);
      const float rd = 1.0f / dmax;
      const bool live = dmax > 0.0f && isfinite(rd);
      q.delta = live ? dmax : 0.0f;
      q.rdelta = live ? rd : 0.0f;
    }
    __builtin_amdgcn_s_setprio(3);
    // ---- codes (Sec. 3.2 rules (1), (2)) into their columns' fields
    if (quantizes) {
      auto code_of = [&](float v, uint32_t word, uint32_t lc) {
        const float s = fminf(fmaxf(v * q.rdelta, lo_q), hi_q);
        const float base = floorf(s), frac = s - base;
        const float unif = (float)(word >> 8) * 0x1.0p-24f;
        const int32_t code = q.delta > 0.0f ? (int32_t)base + ((unif < frac) ? 1 : 0) : 0;
        if (code != 0) atomicOr(&codes[my_word * S + lc], ((uint32_t)code & mask) << my_shift);
      };
      if (!long_list) {
#pragma unroll
        for (int k = 0; k < kLiPairs; ++k)
          if (k * 64 < list.cols && col[k] != 0u) code_of(u[k], rnd[k], col[k] - 1u);
      } else {
        for (int k = lane; k < list.cols; k += 64) {
          const uint32_t lc = a.cols[list.at + k] - 1u;
          code_of(sum_at(list, k), random_word(lc), lc);
        }
      }
    }
    if (!ok) fail_sh[par] = 1u;
    settle();
    __syncthreads();
    // ---- the receiver (eq. (4), or the integer sums of schemes (b), (c)) and the update of the touched columns; those that
    // the next iteration's rows hold are published at once, and so are the others that they hold
    {
      const uint32_t *next = marks + ((t + 1) % 3) * mark_words, *now = marks + (t % 3) * mark_words;
      auto marked = [&](const uint32_t *m, uint32_t lc) { return (m[lc >> 5] >> (lc & 31u)) & 1u; };
      const uint32_t n = count[t % 3];
      const float dl = lane < kLiWaves ? delta_sh[lane] : 0.0f;
      for (uint32_t i0 = wave * 64; i0 < n; i0 += kLiThreads) {  // whole wavefronts
        const bool in = i0 + lane < n;
        const uint32_t lc = in ? touched[par * S + i0 + lane] : 0u;
        const float m = mus[lc], x0 = xs[lc];
        const bool goes = in && more && marked(next, lc) != 0u;
        float avg = 0.0f;
        int32_t isum = 0;
        int v = 0;
        for (int wd = 0; wd < a.words; ++wd) {
          uint32_t f = in ? codes[wd * S + lc] : 0u;
          if (in) codes[wd * S + lc] = 0u;
          const int last = v + a.fields < a.N ? v + a.fields : a.N;
          if (__ballot(f != 0u) == 0ull) {
            v = last;
            continue;
          }
          for (int shift = 0; v < last; v += 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if (v + i < last) {
                const int32_t code = __builtin_amdgcn_sbfe((int)f, (uint32_t)shift, (uint32_t)a.bits);
                if (PLAIN || a.scheme == LPC_SCHEME_A) avg = __builtin_fmaf(read_lane(dl, v + i), (float)code, avg);
                else isum += code;
              }
              shift += a.bits;
            }
          }
          v = last;
        }
        if (PLAIN || a.scheme == LPC_SCHEME_A) {
          avg *= inv_n;
        } else {
          const float mean_code = (float)isum * inv_n;
          if (a.scheme == LPC_SCHEME_B) {
            avg = q.delta * mean_code;
          } else {  // eq. (5): the average rounded once more
            const float s = fminf(fmaxf(mean_code, lo_q), hi_q);
            const float base = floorf(s), frac = s - base;
            StreamKey k = a.key;
            k.iter = (uint32_t)t;
            const float unif = (float)(stream_word(k, kTagRequant, 0u, (lc << a.pshift) | (uint32_t)p) >> 8) * 0x1.0p-24f;
            avg = q.delta * (float)((int32_t)base + ((unif < frac) ? 1 : 0));
          }
        }
        if (in) {
          float x1;
          if (ALPC) {
            const float yn = prox_scalar(x0, avg + m, a.step_y, a.thr_y, a.shrink_y);
            const float zn = prox_scalar(zs[lc], uhs[lc] + m, a.alpha, a.thr_z, a.shrink_z);
            uhs[lc] = 0.0f;
            zs[lc] = zn;
            ysums[lc] = t == 0 ? (float)weight * yn : ysums[lc] + (float)weight * yn;
            x1 = (a.t1 * zn + a.t2 * wss[lc]) + a.t3 * yn;
            if (!more) a.y[(int64_t)p * S + lc] = yn;
          } else {
            x1 = prox_scalar(x0, avg + m, a.step, a.thr, a.shrink);
          }
          if (goes) put_x(t + 1, lc, x1);
          xs[lc] = x1;
        }
      }
      if (more) {
        const uint32_t n1 = count[(t + 1) % 3];
        for (uint32_t i = (kLiWaves - 1 - wave) * 64 + lane; i < n1; i += kLiThreads) {  // the other wavefronts first
          const uint32_t lc = touched[(1 - par) * S + i];
          if (!marked(now, lc)) put_x(t + 1, lc, xs[lc]);
        }
      }
      // of t - 1: nobody reads it any more, the first to write it is behind the barrier
      if (tid < mark_words) marks[((t + 2) % 3) * mark_words + tid] = 0u;
      for (int e = tid + kLiThreads; e < mark_words; e += kLiThreads) marks[((t + 2) % 3) * mark_words + e] = 0u;
      if (tid == 0) count[(t + 2) % 3] = 0u;
    }
    if (ALPC) weight *= a.theta;
    __syncthreads();
    if (fail_sh[par] != 0u) { gave_up = true; break; }  // uniform: written before the first barrier, next at t + 2
  }
  if (gave_up) {  // the others find the word at their next wait
    if (tid == 0) {
      __hip_atomic_store(a.ctl, a.tag0 + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      atomicOr(&a.flags[0], 2u);
    }
    return;
  }
  for (int l = tid; l < S; l += kLiThreads) {
    const int64_t at = (int64_t)p * S + l;
    if (ALPC) {
      a.z[at] = zs[l];
      a.ysum[at] = ysums[l];
    } else {
      a.x[at] = xs[l];
    }
  }
}

// Iterations of a launch.  n = d = 2^20, N = 16, B = 256: an epoch of 256 takes 3.80, 3.60 and 3.49 ms with 32, 64 and 128
constexpr int kListIters = 128;
// A launch and its lists are about 40 us.  Against the separate launches' 44.5, 22, 27, 21 us per iteration (n = 60000, 40 entries
// drawn per row, N = 16, B = 256; N = 4, B = 32; d = 2^20, N = 16, B = 64; d = 4500, N = 4, B = 64): 128 iterations a launch 14.5, 8.6,
// 11.1, 8.1, 16: 16.7, 10.8, 13.0, 10.6, 8: 21.1, 13.5, 16.2, 13.3, 5: 26.7, 16.7, 20.0, 16.6, 4: -, 19.4, 22.1, 18.5
constexpr int kLeastIters = 4;
// An epoch's own launches (plan, vectors to the owners and back) are about 50 us more.  Separate launches -> these, us per iteration,
// by m: d = 4500, N = 4, B = 64, 31 entries a row: 22.9 -> 65.6 (1), 21.8 -> 22.6 (4), 21.0 -> 19.2 (5); d = 60000, N = 4, B = 32, 25:
// 21.0 -> 22.5 (4), 22.4 -> 19.5 (5); d = 2^20, N = 16, 34: B = 64 60.6 -> 70.5 (1), 42.3 -> 39.9 (2); B = 256 104 -> 85 (1).
// Below five iterations therefore only where they sample enough entries (35000 an iteration and 139000 in the last two).
constexpr int64_t kFewIters = 4, kFewEntries = 50000;
// A batch of E entries takes the builder about 7.5 ms (E / 200000)^2, since it walks the batch once for every 6400 entries, and the
// lists of a launch's iterations are built 256 at a time; the separate launches' iteration is about 8 us per 1000 of E, 2.2 to
// 4 where u^i stays sparse.  Separate launches -> these, us per iteration (16 vectors, iterations a launch in brackets), u^i dense:
// d = 20000, B = 256, E = 102000 989 -> 197 [16], 205000 1848 -> 817 [10]; B = 512, E = 136000 1200 -> 743 [7], 200000 1630 ->
// 1832 [4]; d = 2000, B = 512, E = 113000 923 -> 623 [7], 159000 1194 -> 1403 [4]; sparse: d = 2^20, B = 256, E = 65000 137 -> 93
// [15], 79000 173 -> 138 [15], 118000 267 -> 291 [10].  By E over the iterations that are built at once that is a line each.  The
// rows' length by itself does not matter: 800 entries, B = 64 547 -> 57.  More than 301000 entries (2122 -> 1952, 2 vectors) was
// not measured.
constexpr int64_t kBuiltDense = 35000, kBuiltSparse = 11000, kMostEntries = 300000;
constexpr int kEntryBytes = 16;  // of a list's entry in `ent`, `cols` and `pieces`

struct Shape {
  int pshift, S, fields, words;
  size_t lds;
};

int bits_for(int64_t values) {  // of a number in [0, values)
  int b = 0;
  while (((int64_t)1 << b) < values) ++b;
  return b;
}

int64_t list_rows(const lpc_ctx *c) { return (int64_t)(c->cfg.N + (c->cfg.algo != LPC_ALGO_LPC ? 1 : 0)) * c->cfg.B; }
int64_t list_mean(const lpc_ctx *c) { return (c->prob.nnz + c->n - 1) / c->n; }
// Batch positions that are added up by themselves, as the separate launches do
int32_t list_block(const lpc_ctx *c) { return c->csr_sparse ? csr_sparse_block() : kMaxBatch; }
int64_t list_iters(const lpc_ctx *c) { return c->cfg.m < kListIters ? c->cfg.m : kListIters; }

// What the lists may add to the workspace, bytes: as much again as the entries themselves take (8 bytes each) and the
// column-major copy of them that the workspace holds anyway, but 128 MB for little data and 1 GB for much; the epoch's draws are
// a part of it where the separate launches do not keep them too.  A launch takes the iterations whose lists fit.
int64_t list_budget(const lpc_ctx *c) {
  const int64_t data = 16 * c->prob.nnz, least = (int64_t)128 << 20, most = (int64_t)1 << 30;
  const int64_t draws = c->csr_sparse ? 0 : (int64_t)sizeof(RowPlan) * c->cfg.m * (c->cfg.N + 1) * c->cfg.B;
  return (data < least ? least : data > most ? most : data) - draws;
}

// What does not depend on the rows' lengths; S = 0 where the kernel does not apply: a wavefront per vector, two rows per
// wavefront at most, the slices must fit LDS, the lists of kLeastIters iterations of mean rows what the workspace may grow by, and the
// separate launches must not be the better ones.
Shape shape_of(const lpc_ctx *c) {
  Shape s{};
  if (!c->csr || !c->quant || c->cfg.bits > 16 || c->cfg.N > kLiWaves || c->cfg.m < 1 || c->prob.nnz <= 0) return s;
  s.pshift = kOwnerBits;
  const int P = 1 << s.pshift;
  const bool alpc = c->cfg.algo != LPC_ALGO_LPC;
  const int64_t rows = list_rows(c), S = (c->d + 4 * P - 1) / (4 * P) * 4;
  if (c->cfg.B > kMaxBatch || rows > (int64_t)kLiRows * kLiWaves * P || S > 65535 || P > c->device_cus) return s;
  const int64_t least = c->cfg.m < kLeastIters ? c->cfg.m : kLeastIters;
  if (kEntryBytes * least * rows * list_mean(c) > list_budget(c)) return s;
  if (c->cfg.m <= kFewIters && c->cfg.m * rows * list_mean(c) < kFewEntries) return s;
  if (c->cfg.B * list_mean(c) > kMostEntries) return s;
  s.fields = 32 / c->cfg.bits;
  s.words = (c->cfg.N + s.fields - 1) / s.fields;
  s.lds = 4 * (size_t)S * ((alpc ? 6 : 2) + s.words + 1) + 12 * (size_t)((S + 31) / 32);
  if (s.lds > (size_t)kLiLds - 24 * 1024) return s;
  s.S = (int)S;
  return s;
}

}  // namespace

bool lists_supported(const lpc_ctx *c) { return shape_of(c).S > 0; }

// Room for the lists of kListIters iterations of rows three times as long as the mean, as far as the budget goes; how many
// iterations of the longest row that is, finish_lists says.
ListScratch lists_scratch(const lpc_ctx *c) {
  const Shape s = shape_of(c);
  const size_t P = (size_t)1 << s.pshift, N = (size_t)c->cfg.N, rows = (size_t)list_rows(c);
  ListScratch w;
  w.xw = P * s.S;
  w.slope = 2 * rows;
  w.stat = 2 * N * (5 * P + kDies * kLine);
  w.state = 6 * P * s.S;
  w.off = (size_t)list_iters(c) * (rows / c->cfg.B) * P * kRecord;
  const size_t all = (size_t)list_iters(c) * rows * (size_t)(3 * list_mean(c) + 16), most = (size_t)(list_budget(c) / kEntryBytes);
  w.entries = all < most ? all : most;
  return w;
}

// Once per context, when the rows' lengths are known: how many iterations a launch takes, or that the kernels do not apply.
// Waits for `st`.
hipError_t finish_lists(lpc_ctx *c, hipStream_t st) {
  const Shape s = shape_of(c);
  int32_t extents[2] = {0, 0}, *dev = reinterpret_cast<int32_t *>(c->s.li_state);
  hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t *>(dev), 0u, 2, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(row_extents_kernel, dim3((unsigned)(c->n < 4 * 2048 ? (c->n + 3) / 4 : 2048)), dim3(256), 0, st,
                     c->prob.row_ptr, c->prob.col_idx, c->n, dev);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  e = hipMemcpyAsync(extents, dev, sizeof(extents), hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return e;
  const int32_t longest = extents[0] < 1 ? 1 : extents[0];
  const int lc_bits = bits_for(s.S), pos_bits = c->cfg.B > 1 ? bits_for(c->cfg.B) : 1, k_bits = bits_for(longest);
  c->list_pos_bits = pos_bits;
  c->list_k_bits = k_bits;
  c->list_cap = (int64_t)c->cfg.B * longest;
  const int64_t lists = list_rows(c) / c->cfg.B;
  const int64_t fit = (int64_t)lists_scratch(c).entries / (lists * c->list_cap);
  c->list_iters = (int32_t)(fit < list_iters(c) ? fit : list_iters(c));
  const int64_t turns = (lists * c->list_iters + kOwners - 1) / kOwners;
  // (the builder sorts all of an owner's keys in LDS)
  c->lists_capable = lc_bits + pos_bits + k_bits <= 32 && lc_bits + pos_bits <= 30 &&
                     (int64_t)c->cfg.B * extents[1] <= kKeyCap &&
                     c->list_iters >= (c->cfg.m < kLeastIters ? c->cfg.m : kLeastIters) &&
                     c->cfg.B * list_mean(c) * turns <= (c->csr_sparse ? kBuiltSparse : kBuiltDense) * c->list_iters;
  return hipSuccess;
}

hipError_t launch_lists_begin(const lpc_ctx *c, const ResidentStep &rs, hipStream_t st) {
  const Shape s = shape_of(c);
  if ((1 << s.pshift) > c->usable_cus) return hipErrorCooperativeLaunchTooLarge;
  hipError_t e = launch_csr_plan(c, rs.z_snap, rs.key, rs.alpc, st);
  if (e != hipSuccess) return e;
  if (!rs.z_snap) {
    const int64_t rows = (int64_t)c->cfg.m * list_rows(c);
    hipLaunchKernelGGL(plan_margins_kernel, dim3((unsigned)((rows + 15) / 16)), dim3(256), 0, st, c->prob.col_idx, c->prob.vals,
                       rs.w_snap, rows, c->s.csr_plan);
  }
  const size_t slice = (size_t)s.S << s.pshift;
  DealArgs a{};
  a.d = (int32_t)c->d; a.S = s.S; a.pshift = s.pshift;
  a.from[0] = rs.mu; a.from[1] = rs.w_snap; a.from[2] = rs.y; a.from[3] = rs.z;
  for (int i = 0; i < 4; ++i) a.to[i] = c->s.li_state + i * slice;
  hipLaunchKernelGGL(deal_kernel, dim3((unsigned)((s.S + 31) / 32), (1u << s.pshift) / 64, rs.alpc ? 4 : 2), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_lists_epoch(const lpc_ctx *c, const ResidentStep &rs, int32_t t0, int32_t t1, double weight, hipStream_t st) {
  const Shape s = shape_of(c);
  const int P = 1 << s.pshift, nvec = c->cfg.N + (rs.alpc ? 1 : 0);
  ListBuildArgs b{};
  b.col_idx = c->prob.col_idx; b.vals = c->prob.vals; b.plan = c->s.csr_plan + (int64_t)t0 * nvec * c->cfg.B;
  b.rec = c->s.li_off; b.ent = reinterpret_cast<uint2 *>(c->s.li_ent); b.cols = c->s.li_cols;
  b.pieces = c->s.li_cols + lists_scratch(c).entries; b.block = list_block(c);
  b.cap = c->list_cap;
  b.B = c->cfg.B; b.pos_bits = c->list_pos_bits; b.k_bits = c->list_k_bits;
  b.map_words = (b.B + 31) / 32; b.loss = c->prob.loss;
  const void *build = reinterpret_cast<const void *>(&list_build_kernel);
  const int n_maps = kOwnBins * P * b.map_words;  // words
  b.map_space = n_maps > kKeyCap ? n_maps : kKeyCap;
  b.key_space = kKeyCap + kKeyCap / 4;
  const int n_ranks = kOwnBins * P / 2 * ((b.map_words + 1) / 2);
  if (b.key_space < n_ranks + 6 * b.B) b.key_space = n_ranks + 6 * b.B;  // ranks, and one owner's mapped entries (6 bytes)
  const int build_lds = 4 * (b.map_space + b.key_space + 2 * b.B);
  hipError_t e = hipFuncSetAttribute(build, hipFuncAttributeMaxDynamicSharedMemorySize, build_lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(list_build_kernel, dim3((unsigned)((t1 - t0) * nvec)), dim3(kLiThreads), build_lds, st, b);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  ListArgs a{};
  fill_method_args(a, c, rs, t0, t1, weight);
  a.col_idx = b.col_idx; a.vals = b.vals; a.plan = b.plan; a.rec = b.rec; a.ent = b.ent; a.cols = b.cols;
  a.pieces = b.pieces; a.block = b.block; a.cap = b.cap;
  const size_t slice = (size_t)s.S * P;
  float *state = c->s.li_state;
  a.mu = state; a.ws = state + slice; a.y = state + 2 * slice; a.z = state + 3 * slice; a.x = state + 4 * slice;
  a.ysum = state + 5 * slice;
  const ListScratch w = lists_scratch(c);
  a.xw = c->s.cl_msg; a.slope = a.xw + w.xw; a.stat = a.slope + w.slope;
  a.stat2 = a.stat + 2 * (size_t)c->cfg.N * 5 * P;
  a.S = s.S; a.pshift = s.pshift; a.fields = s.fields; a.words = s.words;
  const bool plain = c->cfg.clip_mode == LPC_CLIP_LAMBDA && c->cfg.scheme == LPC_SCHEME_A;
  const void *fn = rs.alpc ? (plain ? reinterpret_cast<const void *>(&list_epoch_kernel<true, true>)
                                    : reinterpret_cast<const void *>(&list_epoch_kernel<true, false>))
                           : (plain ? reinterpret_cast<const void *>(&list_epoch_kernel<false, true>)
                                    : reinterpret_cast<const void *>(&list_epoch_kernel<false, false>));
  e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)s.lds);
  if (e != hipSuccess) return e;
  void *args[] = {&a};
  return hipLaunchCooperativeKernel(fn, dim3((unsigned)P), dim3(kLiThreads), args, (unsigned)s.lds, st);
}

// The next snapshot and Alg. 2's vectors, unless a launch of the epoch gave up
hipError_t launch_lists_commit(const lpc_ctx *c, const ResidentStep &rs, double snap_scale, float *w_snap, hipStream_t st) {
  const Shape s = shape_of(c);
  const size_t slice = (size_t)s.S << s.pshift;
  float *state = c->s.li_state;
  DealArgs a{};
  a.d = (int32_t)c->d; a.S = s.S; a.pshift = s.pshift; a.back = 1; a.ctl = c->s.cl_ctl; a.launch_tag = rs.tag0 + 1u;
  a.from[0] = state + (rs.alpc ? 5 : 4) * slice; a.to[0] = w_snap; a.scale[0] = rs.alpc ? (float)snap_scale : 1.0f;
  a.from[1] = state + 2 * slice; a.to[1] = rs.y; a.scale[1] = 1.0f;
  a.from[2] = state + 3 * slice; a.to[2] = rs.z; a.scale[2] = 1.0f;
  hipLaunchKernelGGL(deal_kernel, dim3((unsigned)((s.S + 31) / 32), (1u << s.pshift) / 64, rs.alpc ? 3 : 1), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace lpc
