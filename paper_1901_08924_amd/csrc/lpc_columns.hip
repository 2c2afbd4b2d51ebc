// The inner loop of an epoch (Alg. 1 steps 5-11; Alg. 2 steps 5-15) in one launch for dense problems past d = 256: a worker is a
// group of G workgroups, each with a block of C = 64 K columns of the worker's rows, of its u^i and of the iterate.
//
// As separate launches an iteration is 15 to 29 us (rows, fold, exchange; five launches past d = 16384) for 8 to 41 MB of
// rows: launch gaps, the partial gradients' way through memory and back, and nothing in flight between.  By columns the
// partial gradients never leave a workgroup and the iterate never crosses at all; what crosses, as tagged words, is
//   1. the margins' partial sums, inside a worker's group (B words per workgroup),
//   2. the statistics of u^i, inside the group (schemes (b), (c): then the scale factors, across the groups),
//   3. the codes of a column block, across the groups: a word of four codes per four columns, and the scale factor;
// every workgroup then takes the receiver and the update for its own columns.
// Eight wavefronts hold the sampled rows in registers (eight rows each, a lane columns lane, lane + 64, ...) and request
// those of the next iteration as soon as the gradient is formed, so that memory works during the whole exchange.  Four
// others do everything else (four columns per lane): loads return in order, so a wavefront with rows on their way could
// not see a word before the last of them.
// A worker's group sits on one die (workgroup b runs on die b mod 8; only the speed depends on it): 1. and 2. stay inside
// that die's L2.
// Reuse of the two sets of slots: the slots of t are written again at t + 2 by somebody who has seen a word of t + 1 that
// each of their readers wrote after it had read t, or after a barrier that its reading wavefront had passed.
// The launch is cooperative: all workgroups are resident together; waits are bounded by LPC_TUNE_SPIN_LIMIT (the first
// iteration's by 256 times as much: other work on the GPU may hold compute units), a workgroup that gives up says so to the
// others, the epoch leaves the caller's vectors as they were (launch_commit_epoch), and the calls that answer to the host
// report LPC_EDEVICE.
// What bounds an iteration: at d = 4096, N = 8, B = 64 the chain of dependent trips (7.0 us: margins 0.8 + 1.2 for the
// words, gradient 0.4, statistics 0.7 + 1.0, codes 0.5, their words across the dies 1.5, update 0.4); at d = 20000 the rows
// (41 MB in 10 us, paced) and that memory rests while margins are formed.
// Measured on MI355X, snapshot pass (n = 16384) and 128 iterations, separate launches -> this kernel, us per iteration:
//   d = 300, N = 8, B = 64: 11.8 -> 5.6    d = 1500, N = 2, B = 16: 11.1 -> 4.7    d = 1500, N = 16, B = 64: 15.3 -> 7.3
//   d = 4096, N = 8, B = 64: 14.9 -> 7.5    d = 12000, N = 16, B = 40: 31.1 -> 15.1    d = 20000, N = 8, B = 64: 29.1 -> 15.8
//   d = 20000, N = 2, B = 8: 17.9 -> 9.1    d = 8192, N = 16, B = 64: Alg. 3 22.0 -> 12.7, scheme (b) 29.9 -> 13.7
// Steps that paid: all words of a wait requested together (waiting for them one after another: field words 3.4 us instead
// of 1.5), rows requested after the barrier and paced (21 % at d = 12000), blocks of 256 instead of 128 columns at d = 4096
// (25 %), the random words drawn while the rows' wavefronts work.  Steps that did not: rows
// touched ahead (a load per 128-byte line, of t + 2 after the requests, or of t + 1 while margins form): 10 to 25 % slower at
// K = 12, the memory system is busy with the rows alone; rows requested by halves 8 %, non-temporal loads 4 %, a pause
// between the polls of a wait 0 to 4 % slower.
#include <hip/hip_runtime.h>

#include "lpc_device.h"
#include "lpc_internal.h"

namespace lpc {

namespace {

constexpr int kColRowWaves = 8, kColRows = 8;  // rows of a batch: at most 64
constexpr int kColService = 256;               // threads that hold four columns each
constexpr int kCoThreads = 64 * kColRowWaves + kColService;
constexpr int kDies = 8;

struct ColumnArgs {
  const float *X;
  int64_t ldx, n;
  const float *y, *z_snap, *mu, *w_snap, *yv, *zv;
  float *x_mid, *ysum_mid, *y_mid, *z_mid;     // what a launch leaves for the next one, or for launch_commit_epoch
  uint32_t *packed;                            // messages, or null: nobody reads them
  float *delta_out;
  uint32_t *n_clipped;                         // per vector, or null: not counted
  uint32_t *flags, *ctl;                       // ctl[0]: first tag of a launch that gave up
  // [2][nvec][row waves][G][8]; [2][N][G * S][5]; [2][G][N]; [2][G][N][C (+ N words of scale factors)]; [2][G][C]
  u64 *marg, *stats, *scale_ex, *msg, *vec;
  int32_t d, W, N, nvec, G, per_die, B, it0, it1, bits, scheme, loss, rpw, S;
  uint32_t tag0, spin_limit;
  QuantSpec qs;
  StreamKey key;
  float scale, step, thr, shrink;
  float step_y, thr_y, shrink_y, alpha, thr_z, shrink_z, t1, t2, t3;
  double theta, weight;
};

// the operand of s_waitcnt that waits until at most n vector loads are on their way
constexpr int vmcnt_only(int n) { return n > 63 ? 0xcf7f : (n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14); }

enum : int { kPlain = 0, kOwnScale = 1, kSharedScale = 2 };  // as in lpc_cluster.hip

// K: 64-column chunks of a block; Q: the messages; ALPC: Alg. 2 and 3.
template <int K, int Q, bool ALPC>
__global__ __launch_bounds__(kCoThreads) void column_epoch_kernel(ColumnArgs a) {
  // ---- this workgroup's vector and column block (whole workgroups leave)
  const int die = blockIdx.x & (kDies - 1), slot = blockIdx.x / kDies;
  int v, g;
  if (slot < a.per_die * a.G) {
    const int turn = slot / a.G;
    v = die + kDies * turn;
    g = slot - turn * a.G;
    if (v >= a.nvec) return;
  } else {  // the shared batch's group where the workers fill their dies evenly
    v = a.N;
    g = (slot - a.per_die * a.G) * kDies + die;
    if (g >= a.G || v >= a.nvec) return;
  }
  touch_kernel_arguments<(int)(sizeof(ColumnArgs))>();
  constexpr int C = 64 * K, RG = kColRows / 4;
  // Rows that a wavefront has on their way.  The service wavefronts' words queue behind them in the compute unit: with all
  // eight requested at once a trip of the statistics takes 4 to 5 us.  us per iteration with 1, 2, 4, 8 on their way:
  // d = 4096, N = 8 (K = 4): 7.3, 7.4, 7.5, 7.8; d = 1500, N = 2, B = 16: 4.8, 4.6, 4.6, 5.1; d = 12000, N = 12 (K = 12):
  // 14.5, 15.3, 17.9, 18.2
  constexpr int kFlight = K <= 4 ? 2 : 1;
  __shared__ __attribute__((aligned(16))) float xs[C], part[kColRowWaves][C];
  __shared__ uint32_t rid[2][64], own[C / 2];
  __shared__ float ysh[2][64], ssh[2][64];
  __shared__ uint32_t fail_sh[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool service = wave >= kColRowWaves;
  const int c0 = g * C, cols = a.d - c0 < C ? a.d - c0 : C;  // > 0
  const bool shared = ALPC && v == a.N;

  // rows, labels and snapshot slopes of iteration t (set t & 1), by the last wavefront
  const int d_r = tid - (kCoThreads - 64);
  const bool draws = d_r >= 0 && d_r < a.B;
  auto draw = [&](int t) {
    StreamKey k = a.key;
    k.iter = (uint32_t)t;
    const uint32_t row = (uint32_t)sample_row(k, shared ? kTagShared : kTagBatch,
                                              shared ? kSharedWorkerField : (uint32_t)v, (uint32_t)d_r, a.n);
    rid[t & 1][d_r] = row;
    const float y = a.y[row];
    ysh[t & 1][d_r] = y;
    ssh[t & 1][d_r] = loss_slope(a.loss, a.z_snap[row], y);
  };
  // ---- row wavefronts: rows r0 .. r0 + rows - 1 of the batch
  const int r0 = wave * a.rpw;
  int rows = a.B - r0 < a.rpw ? a.B - r0 : a.rpw;
  if (service || rows < 0) rows = 0;
  const int at0 = rows > 0 ? r0 : 0;
  // ---- service threads: columns q_c .. q_c + 3 of the block, j of the problem
  const int q_w = wave - kColRowWaves, q_c = 4 * (tid - 64 * kColRowWaves), j = c0 + q_c;
  const bool holds = service && 256 * q_w < C && q_c < C;
  const bool quantizes = Q != kPlain && holds && !shared;
  float x4[4], mu4[4], y4[4], z4[4], ws4[4], ysum4[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    x4[c] = mu4[c] = y4[c] = z4[c] = ws4[c] = ysum4[c] = 0.0f;
    if (holds && q_c + c < cols) {
      mu4[c] = a.mu[j + c];
      ws4[c] = a.w_snap[j + c];
      x4[c] = !ALPC && a.it0 > 0 ? a.x_mid[j + c] : ws4[c];
      if (ALPC) {
        ysum4[c] = a.it0 > 0 ? a.ysum_mid[j + c] : 0.0f;
        y4[c] = a.yv[j + c];
        z4[c] = a.zv[j + c];
        x4[c] = (a.t1 * z4[c] + a.t2 * ws4[c]) + a.t3 * y4[c];
      }
    }
    if (holds) xs[q_c + c] = x4[c];
  }
  if (tid < 2) fail_sh[tid] = 0u;
  for (int e = tid; e < C / 2; e += kCoThreads) own[e] = 0u;
  if (draws) {
    draw(a.it0);
    if (a.it0 + 1 < a.it1) draw(a.it0 + 1);
  }
  __syncthreads();

  // `loads` requests all the words that a thread waits for and says whether they are there; one trip for all of them
  auto poll = [&](uint32_t limit, bool &ok, auto loads) {
    if (!ok) return;
    for (uint32_t k = 0; k < limit; ++k) {
      if (loads()) return;
      if ((k & 63u) == 63u && __hip_atomic_load(a.ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.tag0 + 1u) break;
    }
    ok = false;
  };
  bool gave_up = false;
  if (!service) {
    float x[kColRows][K];
    // a row's block through a buffer of its floats (of none where the wavefront has no such row): lanes past them read 0
    auto request = [&](int t) {
#pragma unroll
      for (int i = 0; i < kColRows; ++i) {
        const uint32_t row = __builtin_amdgcn_readfirstlane(rid[t & 1][at0 + (i < rows ? i : 0)]);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float *>(a.X + (int64_t)row * a.ldx + c0), 0, i < rows ? 4 * cols : 0, 0x00027000);
#pragma unroll
        for (int k = 0; k < K; ++k)
          x[i][k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, 4u * lane + 256u * k, 0, 0));
        if (i + 1 < kColRows && i + 1 >= kFlight) {  // at most kFlight rows on their way
          __builtin_amdgcn_sched_barrier(0);
          __builtin_amdgcn_s_waitcnt(vmcnt_only(K * (kFlight - 1)));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    request(a.it0);
    bool row_live[RG];
#pragma unroll
    for (int q = 0; q < RG; ++q) row_live[q] = 4 * q + (lane & 3) < rows;
    for (int t = a.it0; t < a.it1; ++t) {
      const int par = t & 1;
      const uint32_t tag = a.tag0 + (uint32_t)t + 1u;
      const uint32_t limit = t == a.it0 ? (a.spin_limit > 0xffffffu ? ~0u : a.spin_limit * 256u) : a.spin_limit;
      bool ok = true;
      float w[K], acc[K], yr[RG], sr[RG];
#pragma unroll
      for (int k = 0; k < K; ++k) { w[k] = xs[lane + 64 * k]; acc[k] = 0.0f; }
#pragma unroll
      for (int q = 0; q < RG; ++q) {
        const int at = at0 + (row_live[q] ? 4 * q + (lane & 3) : 0);
        yr[q] = ysh[par][at];
        sr[q] = ssh[par][at];
      }
      // ---- margins: this block's share out, everybody's in (lane l: row l & 3 of a group of four)
      u64 *ex = a.marg + ((int64_t)(par * a.nvec + v) * kColRowWaves + wave) * a.G * kColRows;
#pragma unroll
      for (int q = 0; q < RG; ++q) {
        float s[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s[r] = 0.0f;
#pragma unroll
          for (int k = 0; k < K; ++k) s[r] = __builtin_fmaf(x[4 * q + r][k], w[k], s[r]);
        }
        const float z = sum4(s, lane);
        if (lane < 4 && row_live[q])
          st_word(ex + (int64_t)(q * a.G + g) * 4 + lane, __builtin_bit_cast(uint32_t, z), tag);
      }
      float coef[RG];
      u64 f[RG][2];
      {
        const bool in0 = (lane >> 2) < a.G, in1 = (lane >> 2) + 16 < a.G;  // G <= 32
        poll(limit, ok, [&] {
          bool all = true;
#pragma unroll
          for (int q = 0; q < RG; ++q) {
            const u64 *from = ex + (int64_t)q * a.G * 4 + lane;
            f[q][0] = row_live[q] && in0 ? ld_word(from) : (u64)tag << 32;
            f[q][1] = row_live[q] && in1 ? ld_word(from + 64) : (u64)tag << 32;
          }
#pragma unroll
          for (int q = 0; q < RG; ++q) all = all && (uint32_t)(f[q][0] >> 32) == tag && (uint32_t)(f[q][1] >> 32) == tag;
          return all;
        });
      }
#pragma unroll
      for (int q = 0; q < RG; ++q) {
        float z = __builtin_bit_cast(float, (uint32_t)f[q][0]) + __builtin_bit_cast(float, (uint32_t)f[q][1]);
        z += dpp_move<0x124>(z);  // row_ror:4, row_ror:8: the lanes of a row of 16 that hold the same batch position
        z += dpp_move<0x128>(z);
        z = rows_sum(z);
        // (x_0 of Alg. 1 is the snapshot: its differences are exactly zero)
        const float diff = loss_slope(a.loss, z, yr[q]) - sr[q];
        coef[q] = row_live[q] && (ALPC || t > 0) ? diff : 0.0f;
      }
      if (!ok) fail_sh[par] = 1u;
#pragma unroll
      for (int q = 0; q < RG; ++q) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float c = read_lane(coef[q], r);
#pragma unroll
          for (int k = 0; k < K; ++k) acc[k] = __builtin_fmaf(c, x[4 * q + r][k], acc[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < K; ++k) part[wave][lane + 64 * k] = acc[k];
      __syncthreads();
      if (t + 1 < a.it1) request(t + 1);  // they arrive while this iteration goes on
      __syncthreads();
      if (fail_sh[par] != 0u) { gave_up = true; break; }  // uniform: written before the barrier, next at t + 2
    }
  } else {
    double weight = a.weight;
    const bool csigma = a.qs.clip_mode != LPC_CLIP_LAMBDA;
    const float inv_n = 1.0f / (float)a.N;
    const float hi_q = (float)((1 << (a.bits & 31)) / 2 - 1), lo_q = -(float)((1 << (a.bits & 31)) / 2);
    const uint32_t mask = (1u << (a.bits & 31)) - 1u;
    const int msg_block = a.N * C + a.N;  // words of a column block: the codes' words (or coordinates), the scale factors
    Philox4 rnd{0u, 0u, 0u, 0u};
    auto random_words = [&](int t) {
      StreamKey k = a.key;
      k.iter = (uint32_t)t;
      rnd = stream_block(k, kTagQuant, (uint32_t)v, (uint32_t)(j >> 2));
    };
    for (int t = a.it0; t < a.it1; ++t) {
      const int par = t & 1;
      const uint32_t tag = a.tag0 + (uint32_t)t + 1u;
      const uint32_t limit = t == a.it0 ? (a.spin_limit > 0xffffffu ? ~0u : a.spin_limit * 256u) : a.spin_limit;
      bool ok = true;
      auto there = [&](u64 w) { return (uint32_t)(w >> 32) == tag; };
      u64 *out = a.msg + ((int64_t)par * a.G + g) * msg_block;
      if (quantizes) random_words(t);  // while the rows' wavefronts are at work
      __syncthreads();
      // ---- u^i (columns past the problem's hold zeros) and its statistics
      float u4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (holds) {
        float4 p[kColRowWaves];
#pragma unroll
        for (int s = 0; s < kColRowWaves; ++s) p[s] = *reinterpret_cast<const float4 *>(&part[s][q_c]);
#pragma unroll
        for (int s = 0; s < kColRowWaves; ++s) { u4[0] += p[s].x; u4[1] += p[s].y; u4[2] += p[s].z; u4[3] += p[s].w; }
#pragma unroll
        for (int c = 0; c < 4; ++c) u4[c] *= a.scale;
      }
      if (holds && (Q == kPlain || shared)) {  // handed on in full precision
        u64 *to = shared ? a.vec + ((int64_t)par * a.G + g) * C + q_c : out + (int64_t)v * C + q_c;
#pragma unroll
        for (int c = 0; c < 4; ++c) st_word(to + c, __builtin_bit_cast(uint32_t, u4[c]), tag);
      }
      if constexpr (Q != kPlain) {
        if (!shared && 256 * q_w < C) {  // wavefronts with columns
          float mx = 0.0f;
          double sum = 0.0, sumsq = 0.0;
          bool bad = false;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const bool fin = isfinite(u4[c]);
            const float f = fin ? u4[c] : 0.0f;
            bad |= !fin;
            mx = fmaxf(mx, fabsf(f));
            if (csigma) { sum += (double)f; sumsq += (double)f * (double)f; }
          }
          mx = wave_max(mx);
          if (csigma) { sum = wave_sum(sum); sumsq = wave_sum(sumsq); }
          if (__ballot(bad) != 0ull && lane == 0) atomicOr(&a.flags[0], 1u);
          const int n_part = a.G * a.S;  // a.S: wavefronts with columns
          u64 *st = a.stats + (int64_t)(par * a.N + v) * n_part * 5;
          {
            const u64 s = __builtin_bit_cast(u64, sum), s2 = __builtin_bit_cast(u64, sumsq);
            const uint32_t mine = lane == 0 ? __builtin_bit_cast(uint32_t, mx)
                                            : (uint32_t)((lane < 3 ? s : s2) >> (lane & 1 ? 0 : 32));
            if (lane < (csigma ? 5 : 1)) st_word(st + lane * n_part + g * a.S + q_w, mine, tag);
          }
          float am = 0.0f;
          sum = sumsq = 0.0;
          for (int e = lane; e < n_part; e += 64) {
            u64 h[5] = {};
            poll(limit, ok, [&] {
              bool all = true;
#pragma unroll
              for (int i = 0; i < 5; ++i)
                if (i == 0 || csigma) h[i] = ld_word(st + i * n_part + e);
#pragma unroll
              for (int i = 0; i < 5; ++i) all = all && (there(h[i]) || (i > 0 && !csigma));
              return all;
            });
            am = fmaxf(am, __builtin_bit_cast(float, (uint32_t)h[0]));
            if (csigma) {
              sum += __builtin_bit_cast(double, (h[1] & 0xffffffffull) | (h[2] << 32));
              sumsq += __builtin_bit_cast(double, (h[3] & 0xffffffffull) | (h[4] << 32));
            }
          }
          am = wave_max(am);
          if (csigma) { sum = wave_sum(sum); sumsq = wave_sum(sumsq); }
          // Sec. 3.2, eq. (3); the reciprocal is the correctly rounded one, as 1/double(delta) rounded to float is
          QParams q{0.0f, 0.0f, 0.0f, 0.0f};
          if (csigma) {
            q = make_qparams(a.qs, (double)am, sum, sumsq, a.d);
          } else {
            q.thresh = a.qs.clip * am;
            const float delta = q.thresh / hi_q, rd = 1.0f / delta;
            const bool live = delta > 0.0f && isfinite(rd);
            q.delta = live ? delta : 0.0f;
            q.rdelta = live ? rd : 0.0f;
          }
          if constexpr (Q == kSharedScale) {  // the largest of the N scale factors
            u64 *sc = a.scale_ex + ((int64_t)par * a.G + g) * a.N;
            if (q_c == 0) st_word(sc + v, __builtin_bit_cast(uint32_t, q.delta), tag);
            float dmax = 0.0f;
            if (lane < a.N) {  // N <= 64
              u64 w = 0;
              poll(limit, ok, [&] { w = ld_word(sc + lane); return there(w); });
              dmax = __builtin_bit_cast(float, (uint32_t)w);
            }
            dmax = wave_max(dmax);
            const float rd = 1.0f / dmax;
            const bool live = dmax > 0.0f && isfinite(rd);
            q.delta = live ? dmax : 0.0f;
            q.rdelta = live ? rd : 0.0f;
            q.thresh = dmax * hi_q;
          }
          // ---- codes (Sec. 3.2 rules (1), (2)): four to a word
          if (holds) {
            const uint32_t words[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
            uint32_t field = 0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const float s = fminf(fmaxf(u4[c] * q.rdelta, lo_q), hi_q);
              const float base = floorf(s), frac = s - base;
              const float unif = (float)(words[c] >> 8) * 0x1.0p-24f;
              const int32_t code = q.delta > 0.0f ? (int32_t)base + ((unif < frac) ? 1 : 0) : 0;
              field |= ((uint32_t)code & mask) << (c * a.bits);
            }
            st_word(out + (int64_t)v * C + (q_c >> 2), field, tag);
            if (q_c == 0) st_word(out + (int64_t)a.N * C + v, __builtin_bit_cast(uint32_t, q.delta), tag);
            if (a.packed) {  // a traced epoch: the message as it would be sent, a wavefront its own words
              const int bit = q_c * a.bits;
              const u64 f = (u64)field << (bit & 31);
              if ((uint32_t)f) atomicOr(&own[bit >> 5], (uint32_t)f);
              if ((uint32_t)(f >> 32)) atomicOr(&own[(bit >> 5) + 1], (uint32_t)(f >> 32));
              if (q_c == 0 && g == 0) a.delta_out[v] = q.delta;
            }
            if (a.n_clipped) {
              uint32_t clipped = 0;
#pragma unroll
              for (int c = 0; c < 4; ++c) clipped += (u4[c] > q.thresh || u4[c] < lo_q * q.delta) ? 1u : 0u;
              if (clipped) atomicAdd(&a.n_clipped[v], clipped);
            }
          }
          if (a.packed) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const int first = 8 * a.bits * q_w, most = C * a.bits / 32, whole = first + 8 * a.bits;
            for (int wd = first + lane; wd < (whole < most ? whole : most); wd += 64) {
              const int to = g * most + wd;
              if (to < a.W) a.packed[(int64_t)v * a.W + to] = own[wd];
              own[wd] = 0u;
            }
          }
        }
      }
      // ---- while the words travel: the rows of t + 2
      if (draws && t + 2 < a.it1) draw(t + 2);
      // ---- the receiver (eq. (4), or the integer sums of schemes (b), (c))
      if (256 * q_w < C) {  // whole wavefronts: a lane without columns reads the first ones' words
        const int q_r = holds ? q_c : 0;
        float avg[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (Q == kPlain) {
          for (int i0 = 0; i0 < a.N; i0 += 2) {
            const u64 *p = out + (int64_t)i0 * C + q_r;
            const int64_t next = i0 + 1 < a.N ? C : 0;
            u64 f[8] = {};
            poll(limit, ok, [&] {
              bool all = true;
#pragma unroll
              for (int c = 0; c < 8; ++c) f[c] = ld_word(p + (c & 3) + (c < 4 ? 0 : next));
#pragma unroll
              for (int c = 0; c < 8; ++c) all = all && there(f[c]);
              return all;
            });
#pragma unroll
            for (int c = 0; c < 4; ++c) avg[c] += __builtin_bit_cast(float, (uint32_t)f[c]);
            if (next) {
#pragma unroll
              for (int c = 0; c < 4; ++c) avg[c] += __builtin_bit_cast(float, (uint32_t)f[4 + c]);
            }
          }
#pragma unroll
          for (int c = 0; c < 4; ++c) avg[c] *= inv_n;
        } else {
          int32_t isum[4] = {0, 0, 0, 0};
          const u64 *p = out + (q_r >> 2), *pd = out + (int64_t)a.N * C;
          u64 fd = 0;  // a lane holds a worker's scale factor (N <= 64)
          for (int i0 = 0; i0 < a.N; i0 += 8) {
            u64 f[8] = {};
            poll(limit, ok, [&] {
              bool all = true;
              if (i0 == 0) fd = ld_word(pd + (lane < a.N ? lane : 0));
#pragma unroll
              for (int r = 0; r < 8; ++r) f[r] = ld_word(p + (int64_t)(i0 + r < a.N ? i0 + r : a.N - 1) * C);
#pragma unroll
              for (int r = 0; r < 8; ++r) all = all && there(f[r]);
              return all && there(fd);
            });
#pragma unroll
            for (int r = 0; r < 8; ++r) {
              if (i0 + r < a.N) {
                const uint32_t field = (uint32_t)f[r];
                const float delta = read_lane(__builtin_bit_cast(float, (uint32_t)fd), i0 + r);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                  const int32_t code = (int32_t)((field >> (c * a.bits)) << (32 - a.bits)) >> (32 - a.bits);
                  if constexpr (Q == kOwnScale) avg[c] = __builtin_fmaf(delta, (float)code, avg[c]);
                  else isum[c] += code;
                }
              }
            }
          }
          const float delta = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane((int)(uint32_t)fd));
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            if constexpr (Q == kOwnScale) {
              avg[c] *= inv_n;
            } else {
              const float mean_code = (float)isum[c] * inv_n;
              if (a.scheme == LPC_SCHEME_B) {
                avg[c] = delta * mean_code;
              } else {  // eq. (5): the average rounded once more
                const float s = fminf(fmaxf(mean_code, lo_q), hi_q);
                const float base = floorf(s), frac = s - base;
                StreamKey k = a.key;
                k.iter = (uint32_t)t;
                const float unif = (float)(stream_word(k, kTagRequant, 0u, (uint32_t)(j + c)) >> 8) * 0x1.0p-24f;
                avg[c] = delta * (float)((int32_t)base + ((unif < frac) ? 1 : 0));
              }
            }
          }
        }
        float uh[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (ALPC) {
          const u64 *p = a.vec + ((int64_t)par * a.G + g) * C + q_r;
          u64 f[4] = {};
          poll(limit, ok, [&] {
            bool all = true;
#pragma unroll
            for (int c = 0; c < 4; ++c) f[c] = ld_word(p + c);
#pragma unroll
            for (int c = 0; c < 4; ++c) all = all && there(f[c]);
            return all;
          });
#pragma unroll
          for (int c = 0; c < 4; ++c) uh[c] = __builtin_bit_cast(float, (uint32_t)f[c]);
        }
        // ---- the update
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if constexpr (ALPC) {
            const float yn = prox_scalar(x4[c], avg[c] + mu4[c], a.step_y, a.thr_y, a.shrink_y);
            const float zn = prox_scalar(z4[c], uh[c] + mu4[c], a.alpha, a.thr_z, a.shrink_z);
            y4[c] = yn;
            z4[c] = zn;
            ysum4[c] = t == 0 ? (float)weight * yn : ysum4[c] + (float)weight * yn;
            x4[c] = (a.t1 * zn + a.t2 * ws4[c]) + a.t3 * yn;
          } else {
            x4[c] = prox_scalar(x4[c], avg[c] + mu4[c], a.step, a.thr, a.shrink);
          }
        }
        if (holds) *reinterpret_cast<float4 *>(&xs[q_c]) = make_float4(x4[0], x4[1], x4[2], x4[3]);
      }
      if constexpr (ALPC) weight *= a.theta;
      if (!ok) fail_sh[par] = 1u;
      __syncthreads();
      if (fail_sh[par] != 0u) { gave_up = true; break; }
    }
  }
  if (gave_up) {  // the iterate is not to be trusted; the others find the word at their next wait
    if (tid == 0) {
      __hip_atomic_store(a.ctl, a.tag0 + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      atomicOr(&a.flags[0], 2u);
    }
    return;
  }
  if (v == 0 && holds) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (q_c + c < cols) {
        if (ALPC) {
          a.y_mid[j + c] = y4[c];
          a.z_mid[j + c] = z4[c];
          a.ysum_mid[j + c] = ysum4[c];
        } else {
          a.x_mid[j + c] = x4[c];
        }
      }
    }
  }
}

struct Shape {
  int k, G, per_die, slots;
};

// The launch for a context, or k = 0 where the kernel does not apply: the batch must fit the registers of the row
// wavefronts, four codes a word (b <= 8), and the groups the dies.  Eight rows per wavefront, 64 in all, are what its
// registers hold of the widest block.  Narrower blocks leave room for more, but there is no instantiation with more: one
// row past the line takes the separate launches (d = 4096, N = 8: B = 64 7.5 us per iteration here, 14.9 there; B = 65 15.4,
// B = 128 16.8 there).
// Few workgroups wait for fewer words, many have fewer rows to fetch.  Up to 16 workgroups per group and 24 per die the
// narrowest block is the fastest (us per iteration by K = 4, 6, 8, 10, 12: d = 4096, N = 8, B = 64: 7.6, 8.3, 8.3, -, -;
// d = 5000, N = 16, B = 30: -, 8.4, 7.9, 8.1, 8.2), beyond that the widest is (d = 8192, N = 8: 11.8, 10.5, 9.8, 9.8, 9.9; Alg. 3,
// N = 16: -, -, -, 13.6, 12.8; d = 20000, N = 8: -, -, -, 16.5, 15.5; K = 2 lost everywhere: d = 4096: 10.2).
Shape shape_of(const lpc_ctx *c) {
  Shape s{};
  if (c->csr || c->mlp || !c->grad_ok || c->n_full != c->n || c->n >= ((int64_t)1 << 31)) return s;
  if (c->cfg.B > kColRowWaves * kColRows || c->cfg.N > 64 || c->cfg.m < 1 || (c->quant && c->cfg.bits > 8)) return s;
  const int N = c->cfg.N, alpc = c->cfg.algo != LPC_ALGO_LPC ? 1 : 0;
  for (int k : {4, 6, 8, 10, 12}) {
    const int G = (int)((c->d + 64 * k - 1) / (64 * k));
    const bool extra = alpc && N % kDies == 0;  // the shared batch's group spread over what the workers leave
    const int per_die = (N + (extra ? 0 : alpc) + kDies - 1) / kDies;
    const int slots = per_die * G + (extra ? (G + kDies - 1) / kDies : 0);
    if (slots * kDies > c->device_cus || (k < 12 ? G > 16 || slots > 24 : G > 32)) continue;
    s.k = k; s.G = G; s.per_die = per_die; s.slots = slots;
    return s;
  }
  return s;
}

}  // namespace

bool columns_supported(const lpc_ctx *c) { return shape_of(c).k > 0; }

ColumnScratch columns_scratch(const lpc_ctx *c) {
  const Shape s = shape_of(c);
  const size_t N = (size_t)c->cfg.N, G = (size_t)s.G, C = 64 * (size_t)s.k, S = (C + 255) / 256;
  ColumnScratch w;
  w.marg = 2 * (N + 1) * kColRowWaves * G * kColRows;
  w.stats = 2 * N * G * S * 5;
  w.scale = 2 * G * N;
  w.msg = 2 * G * (N * C + N);
  w.vec = 2 * G * C;
  return w;
}

hipError_t launch_columns_epoch(const lpc_ctx *c, const ResidentStep &rs, int32_t t0, int32_t t1, double weight,
                                bool traced, uint32_t *n_clipped, hipStream_t st) {
  const Shape s = shape_of(c);
  if (s.slots * kDies > c->usable_cus) return hipErrorCooperativeLaunchTooLarge;
  ColumnArgs a{};
  fill_loop_args(a, c, rs, t0, t1, weight, n_clipped);
  if (t0 > 0) { a.yv = c->s.cl_y; a.zv = c->s.cl_z; }
  a.x_mid = c->s.w; a.ysum_mid = c->s.ysum; a.y_mid = c->s.cl_y; a.z_mid = c->s.cl_z;
  a.packed = traced ? c->s.packed : nullptr; a.delta_out = c->s.delta;
  const ColumnScratch w = columns_scratch(c);
  a.marg = c->s.cl_msg; a.stats = a.marg + w.marg; a.scale_ex = a.stats + w.stats; a.msg = a.scale_ex + w.scale;
  a.vec = a.msg + w.msg;
  a.G = s.G; a.per_die = s.per_die; a.rpw = (c->cfg.B + kColRowWaves - 1) / kColRowWaves; a.S = (64 * s.k + 255) / 256;
  const void *fn = nullptr;
  const int q = !c->quant ? kPlain : (c->cfg.scheme == LPC_SCHEME_A ? kOwnScale : kSharedScale);
#define LPC_COLUMNS_Q(K_, Q_)                                                                    \
  if (s.k == K_ && q == Q_)                                                                      \
    fn = rs.alpc ? reinterpret_cast<const void *>(&column_epoch_kernel<K_, Q_, true>)            \
                 : reinterpret_cast<const void *>(&column_epoch_kernel<K_, Q_, false>);
#define LPC_COLUMNS(K_) LPC_COLUMNS_Q(K_, kPlain) LPC_COLUMNS_Q(K_, kOwnScale) LPC_COLUMNS_Q(K_, kSharedScale)
  LPC_COLUMNS(4) LPC_COLUMNS(6) LPC_COLUMNS(8) LPC_COLUMNS(10) LPC_COLUMNS(12)
#undef LPC_COLUMNS
#undef LPC_COLUMNS_Q
  if (!fn) return hipErrorInvalidValue;
  void *args[] = {&a};
  return hipLaunchCooperativeKernel(fn, dim3((unsigned)(s.slots * kDies)), dim3(kCoThreads), args, 0, st);
}

}  // namespace lpc
