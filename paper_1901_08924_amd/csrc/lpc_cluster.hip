// The inner loop of an epoch (Alg. 1 steps 5-11; Alg. 2 steps 5-15) in one launch for narrow dense problems (d <= 256, or
// d <= 1024 with more than 8 bits; a worker's batch small enough for the registers of one workgroup): a workgroup per
// worker, as in the paper, or one workgroup for all of them where even that is more than the work needs.
//
// Such an iteration moves tens or hundreds of KB and takes a few thousand instructions; as three launches (rows, fold,
// exchange; five or six for the schemes (b) and (c)) it is 11 to 33 us of launch gaps and first trips to memory.  Here a
// workgroup of sixteen wavefronts
//   - holds its workers' sampled rows in registers (a wavefront some rows, a lane columns lane, lane + 64, ...), requested
//     one iteration ahead: which rows an iteration samples does not depend on the iterate;
//   - forms margins, slopes and u^i, the statistics of u^i, its scale factor, its codes and its message in LDS;
//   - hands its message to the other workgroups and waits for theirs: this is the only wait between workgroups, once per
//     iteration (schemes (b), (c): one more, for the shared scale factor);
//   - takes eq. (4) and the update for ALL coordinates itself, so every workgroup holds the new iterate and nothing else
//     has to cross.
// Messages cross as 64-bit words (value, tag) in device memory, written and read with agent-scope atomics; the tag grows
// with every iteration of every launch of the context, a reader takes the word once its tag is the expected one, so
// neither flag nor fence stands between writer and reader.  Two sets of slots alternate: who writes iteration t + 2 has
// read everybody's t + 1, which were written after their owners had read t.
// The launch with several workgroups is cooperative, so that all are resident together; every wait is bounded by
// LPC_TUNE_SPIN_LIMIT, a workgroup that gives up says so to the others, the epoch leaves the caller's vectors as they were
// (launch_commit_epoch), and the calls that answer to the host report LPC_EDEVICE.  One workgroup waits for nobody and
// writes the caller's vectors itself.
// What bounds an iteration is the chain of dependent steps: rows 1.1 us, statistics 0.5 us, codes 0.5 us, messages there
// and back 0.9 us, receiver and update 0.9 us (d = 90, N = 8, B = 64; the words stay inside one die's L2).
// Measured on MI355X, snapshot pass (n = 16384) and 128 iterations, separate launches -> this kernel, us per iteration:
//   d = 64, N = 4, B = 16: 10.4 -> 3.0       d = 90, N = 8, B = 64: 11.6 -> 4.3     d = 256, N = 16, B = 32: 11.7 -> 5.2
//   d = 512, N = 8, B = 64, b = 9: 11.6 -> 6.7     d = 1000, N = 14, B = 32, b = 9: 12.9 -> 10.2
//   scheme (b), d = 256, N = 4, B = 16: 21.8 -> 4.8;  quantization off, d = 64, N = 4, B = 16: 15.6 -> 2.1
// Steps that paid: the kernel made for its messages and algorithm (23 %: one branch less in every phase), no division
// inside the loop and messages assembled by LDS atomics instead of a loop over a word's codes (25 %), labels and snapshot
// slopes fetched with the rows (8 %).
#include <hip/hip_runtime.h>

#include "lpc_device.h"
#include "lpc_internal.h"

namespace lpc {

namespace {

constexpr int kClThreads = 1024, kClWaves = 16;
constexpr int kClLds = 156 * 1024;  // dynamic LDS of a launch, at most

struct ClusterArgs {
  const float *X;
  int64_t ldx, n;
  const float *y, *z_snap, *mu, *w_snap, *yv, *zv;
  const float *in;              // where it0 > 0: x (Alg. 2, 3: the weighted sum of y), as the launch before left it
  float *out, *y_out, *z_out;
  uint32_t *packed;
  float *delta_out;
  uint32_t *n_clipped;        // per vector, or null: not counted
  uint32_t *flags, *ctl;      // ctl[0]: first tag of a launch that gave up
  u64 *msg, *vec, *scale_ex;  // [2][N][W + 1] (words, then the scale factor), [2][vectors in full precision][d], [2][N]
  int32_t d, dp, W, N, nvec, nv, G, spread, B, it0, it1, bits, scheme, loss, rpw, wpv;
  uint32_t tag0, spin_limit, inv_w1;  // inv_w1: ceil(2^32 / (W + 1))
  QuantSpec qs;
  StreamKey key;
  float scale, step, thr, shrink;
  float step_y, thr_y, shrink_y, alpha, thr_z, shrink_z, t1, t2, t3, out_scale;
  double theta, weight;
};

// What the messages of a launch are: kPlain: quantization off (vectors in full precision); kOwnScale: scheme (a);
// kSharedScale: schemes (b) and (c).
enum : int { kPlain = 0, kOwnScale = 1, kSharedScale = 2 };

// K: 64-column chunks of a row (d <= 64 K); RW: rows a wavefront holds; Q: the messages; ALPC: Alg. 2 and 3.
template <int K, int RW, int Q, bool ALPC>  // Q == kPlain: K <= 4 only
__global__ __launch_bounds__(kClThreads) void cluster_epoch_kernel(ClusterArgs a) {
  if (blockIdx.x % a.spread != 0) return;  // whole workgroups: see launch_cluster_epoch
  touch_kernel_arguments<(int)(sizeof(ClusterArgs))>();
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  __shared__ float red_max[32];
  __shared__ double red_sum[2][32];
  __shared__ uint32_t red_bad[32];
  __shared__ float delta_sh[kClWaves];
  __shared__ uint32_t fail_sh;
  constexpr int D = 64 * K, RG = (RW + 3) / 4;
  constexpr bool kWaveOwns = K <= 4;  // a wavefront holds a whole vector, four coordinates per lane
  int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // What derives from these alone is else kept in registers for the whole loop, and takes others with it: this compiler's choice,
  // to be looked at again with another one (K = 2 and 4: 98 -> 85, 108 -> 93 vector registers, 78 -> 62 scalar ones in memory).
  // Where taking them afresh in every iteration pays: d = 90, N = 8, B = 64, 905 iterations 3784 -> 3616 us, fifteen drawn problems of these kernels 0.95 to
  // 1.006 times; the others of Alg. 1 the same, Alg. 2 and 3 up to 1.12 times.
  constexpr bool kAfresh = !ALPC && Q == kOwnScale && K >= 2 && K <= 4 && RW == 4;
  const int g = blockIdx.x / a.spread, v0 = g * a.nv;
  const int nv = a.nvec - v0 < a.nv ? a.nvec - v0 : a.nv;  // this workgroup's vectors: v0 .. v0 + nv - 1
  const int nB = a.nv * a.B, dp = a.dp, W1 = a.W + 1;
  const bool alone = a.G == 1;
  // LDS: iterate, partial vectors, vectors, shared difference, messages (all, and this workgroup's), draws (two sets)
  float *xs = reinterpret_cast<float *>(lds_raw);
  float *part = xs + D;
  float *us = part + kClWaves * D;
  float *uh = us + a.nv * dp;
  uint32_t *msg = reinterpret_cast<uint32_t *>(uh + D);        // [N][W + 1]
  uint32_t *own = alone ? msg : msg + a.N * W1;                // [nv][W + 1]; one workgroup's are all there are
  uint32_t *rid = msg + (a.N + a.nv) * W1;
  float *ysh = reinterpret_cast<float *>(rid + 2 * nB), *ssh = ysh + 2 * nB;

  // ---- the state of this thread's coordinate (every workgroup carries all of them)
  const int j = tid;
  const bool mine = j < a.d;
  float x_j = 0.0f, mu_j = 0.0f, y_j = 0.0f, z_j = 0.0f, ws_j = 0.0f, ysum_j = 0.0f;
  if (mine) {
    mu_j = a.mu[j];
    ws_j = a.w_snap[j];
    x_j = !ALPC && a.it0 > 0 ? a.in[j] : ws_j;
    if (ALPC) {
      ysum_j = a.it0 > 0 ? a.in[j] : 0.0f;
      y_j = a.yv[j];
      z_j = a.zv[j];
      x_j = (a.t1 * z_j + a.t2 * ws_j) + a.t3 * y_j;
    }
  }
  if (tid < D) xs[tid] = x_j;
  if (tid == 0) fail_sh = 0u;

  // rows, labels and snapshot slopes of iteration t (set t & 1): threads 0 .. nv * B - 1, batch position d_r of vector d_lv
  const int d_lv = tid / a.B, d_r = tid - d_lv * a.B;
  const bool draws = tid < nv * a.B, d_shared = ALPC && v0 + d_lv == a.N;
  auto draw = [&](int t) {
    StreamKey k = a.key;
    k.iter = (uint32_t)t;
    const uint32_t row = (uint32_t)sample_row(k, d_shared ? kTagShared : kTagBatch,
                                              d_shared ? kSharedWorkerField : (uint32_t)(v0 + d_lv), (uint32_t)d_r, a.n);
    const int at = (t & 1) * nB + tid;
    rid[at] = row;
    const float y = a.y[row];
    ysh[at] = y;
    ssh[at] = loss_slope(a.loss, a.z_snap[row], y);  // the snapshot's slope does not wait for the iterate
  };
  const int lv_w = wave / a.wpv, sub = wave - lv_w * a.wpv;  // this wavefront's vector and its share of the batch
  const int r0 = sub * a.rpw;                                // its rows: r0 .. r0 + rows - 1 of the batch
  int rows = a.B - r0 < a.rpw ? a.B - r0 : a.rpw;
  if (lv_w >= nv || rows < 0) rows = 0;
  const int at0 = lv_w < nv ? lv_w * a.B + (rows > 0 ? r0 : 0) : 0;
  float x[RW][K];
  // a row through a buffer of its d floats (of none where the wavefront has no such row): a lane past them reads zero
  auto request = [&](int t) {
    const uint32_t *ids = rid + (t & 1) * nB + at0;
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      const uint32_t row = __builtin_amdgcn_readfirstlane(ids[i < rows ? i : 0]);
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<float *>(a.X + (int64_t)row * a.ldx), 0, i < rows ? 4 * a.d : 0, 0x00027000);
#pragma unroll
      for (int k = 0; k < K; ++k)
        x[i][k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, 4u * lane + 256u * k, 0, 0));
    }
  };
  if (draws) draw(a.it0);
  __syncthreads();
  request(a.it0);
  if (draws && a.it0 + 1 < a.it1) draw(a.it0 + 1);
  for (int e = tid; e < nv * W1; e += kClThreads) own[e] = 0u;
  __syncthreads();

  double weight = a.weight;
  // what this thread does in the loop's phases (no divisions inside)
  const int u_lv = tid / dp, u_c = tid - u_lv * dp;  // !kWaveOwns: coordinate u_c of vector u_lv (nv * dp <= 1024)
  // four coordinates to quantize: of vector `wave`, or (!kWaveOwns) counted from the last thread
  const int qg = kClThreads - 1 - tid;
  const int q_lv = kWaveOwns ? wave : 4 * qg / dp, q_c = kWaveOwns ? 4 * lane : 4 * qg - q_lv * dp;
  const bool q_in = q_lv < nv && q_c < dp;
  const bool quantizes = Q != kPlain && q_in && v0 + q_lv < a.N;
  const int bit_j = j * a.bits, wi_j = bit_j >> 5, sh_j = bit_j & 31;
  const bool two_j = sh_j + a.bits > 32;
  const int own_quant = a.N - v0 < nv ? (a.N - v0 > 0 ? a.N - v0 : 0) : nv;  // of this workgroup's vectors, the quantized
  const float inv_n = 1.0f / (float)a.N;
  const float hi_q = (float)((1 << (a.bits & 31)) / 2 - 1), lo_q = -(float)((1 << (a.bits & 31)) / 2);
  const uint32_t mask = (1u << (a.bits & 31)) - 1u;
  bool row_live[RG];
#pragma unroll
  for (int q = 0; q < RG; ++q) row_live[q] = 4 * q + (lane & 3) < rows;
  Philox4 rnd{0u, 0u, 0u, 0u};
  auto random_words = [&](int t) {  // of this thread's codes
    StreamKey k = a.key;
    k.iter = (uint32_t)t;
    rnd = stream_block(k, kTagQuant, (uint32_t)(v0 + q_lv), (uint32_t)(q_c >> 2));
  };
  if (quantizes) random_words(a.it0);
  bool gave_up = false;
  for (int t = a.it0; t < a.it1; ++t) {
    if constexpr (kAfresh) {
      asm volatile("" : "+v"(tid));
      lane = tid & 63;
      wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    }
    const int par = t & 1;
    const uint32_t tag = a.tag0 + (uint32_t)t + 1u;
    bool ok = true;
    // (other work on the GPU may hold compute units from workgroups that have yet to start)
    const uint32_t limit = t == a.it0 ? (a.spin_limit > 0xffffffu ? ~0u : a.spin_limit * 256u) : a.spin_limit;
    auto wait = [&](const u64 *p) { return wait_word(p, tag, limit, a.ctl, a.tag0 + 1u, ok); };
    // ---- rows: margins, slopes, this wavefront's share of u
    {
      float w[K], acc[K], yr[RG], sr[RG];
#pragma unroll
      for (int k = 0; k < K; ++k) { w[k] = xs[lane + 64 * k]; acc[k] = 0.0f; }
#pragma unroll
      for (int q = 0; q < RG; ++q) {
        const int at = par * nB + at0 + (row_live[q] ? 4 * q + (lane & 3) : 0);
        yr[q] = ysh[at];
        sr[q] = ssh[at];
      }
#pragma unroll
      for (int q = 0; q < RG; ++q) {
        float s[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          s[r] = 0.0f;
          if (4 * q + r < RW) {
#pragma unroll
            for (int k = 0; k < K; ++k) s[r] = __builtin_fmaf(x[4 * q + r][k], w[k], s[r]);
          }
        }
        const float z = sum4(s, lane);
        // (x_0 of Alg. 1 is the snapshot: its differences are exactly zero)
        const float diff = loss_slope(a.loss, z, yr[q]) - sr[q];
        const float coef = row_live[q] && (ALPC || t > 0) ? diff : 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (4 * q + r < RW) {
            const float c = read_lane(coef, r);
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] = __builtin_fmaf(c, x[4 * q + r][k], acc[k]);
          }
        }
      }
#pragma unroll
      for (int k = 0; k < K; ++k) part[wave * D + lane + 64 * k] = acc[k];
    }
    __syncthreads();
    if (t + 1 < a.it1) request(t + 1);  // they arrive while this iteration goes on
    // ---- u^i, its statistics and scale factor
    float u4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    QParams q{0.0f, 0.0f, 0.0f, 0.0f};
    const bool csigma = a.qs.clip_mode != LPC_CLIP_LAMBDA;
    // a vector (or coordinate) that is handed on in full precision
    auto hand_on = [&](int lv, int c, float u) {
      const int v = v0 + lv;
      if (Q != kPlain && !(ALPC && v == a.N)) return;
      if (!alone)
        st_word(a.vec + ((int64_t)par * (Q == kPlain ? a.nvec : 1) + (Q == kPlain ? v : 0)) * a.d + c,
                __builtin_bit_cast(uint32_t, u), tag);
      else if (ALPC && v == a.N) uh[c] = u;
      else us[lv * dp + c] = u;
    };
    // Sec. 3.2, eq. (3); the reciprocal is the correctly rounded one, as 1/double(delta) rounded to float is
    auto scale_of = [&](float am, double s, double s2) {
      if (csigma) q = make_qparams(a.qs, (double)am, s, s2, a.d);
      else q.thresh = a.qs.clip * am;
      const float delta = q.thresh / hi_q;
      const float rd = 1.0f / delta;
      const bool live = delta > 0.0f && isfinite(rd);
      q.delta = live ? delta : 0.0f;
      q.rdelta = live ? rd : 0.0f;
    };
    if constexpr (kWaveOwns) {
      if (wave < nv) {
        const float4 *p = reinterpret_cast<const float4 *>(part + q_lv * a.wpv * D) + lane;
        if (q_c < D) {
          for (int s = 0; s < a.wpv; s += 4) {
            float4 r[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = p[(s + i < a.wpv ? s + i : s) * (D / 4)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if (s + i < a.wpv) { u4[0] += r[i].x; u4[1] += r[i].y; u4[2] += r[i].z; u4[3] += r[i].w; }
            }
          }
        }
        float mx = 0.0f;
        double sum = 0.0, sumsq = 0.0;
        bool bad = false;
#pragma unroll
        for (int c = 0; c < 4; ++c) {  // columns past d hold zeros
          u4[c] *= a.scale;
          const bool fin = isfinite(u4[c]);
          const float f = fin ? u4[c] : 0.0f;
          bad |= !fin;
          mx = fmaxf(mx, fabsf(f));
          if (csigma) { sum += (double)f; sumsq += (double)f * (double)f; }
        }
        if (Q == kPlain || (ALPC && v0 + q_lv == a.N)) {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if (q_c + c < a.d) hand_on(q_lv, q_c + c, u4[c]);
        }
        if (Q != kPlain) {
          mx = wave_max(mx);
          if (csigma) { sum = wave_sum(sum); sumsq = wave_sum(sumsq); }
          if (__ballot(bad) != 0ull && lane == 0 && v0 + q_lv < a.N) atomicOr(&a.flags[0], 1u);
          scale_of(mx, sum, sumsq);
        }
      }
    } else {
      float u = 0.0f;
      if (u_lv < nv && u_c < a.d) {
        const float *p = part + u_lv * a.wpv * D + u_c;
        for (int s = 0; s < a.wpv; s += 4) {
          float r[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) r[i] = s + i < a.wpv ? p[(s + i) * D] : 0.0f;
          u += (r[0] + r[1]) + (r[2] + r[3]);
        }
        u *= a.scale;
        hand_on(u_lv, u_c, u);
      }
      if (u_lv < nv) us[tid] = u;
      if (Q != kPlain) {
        // 32 lanes hold coordinates of one vector (dp is a multiple of 32)
        const bool fin = isfinite(u);
        float mx = row16_max(fin ? fabsf(u) : 0.0f);
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        const uint64_t bad = __ballot(!fin);
        const int half = tid >> 5;
        if ((tid & 31) == 0) {
          red_max[half] = mx;
          red_bad[half] = (uint32_t)(bad >> (32 * (half & 1)));
        }
        if (csigma) {
          double s = row16_sum(fin ? (double)u : 0.0), s2 = row16_sum(fin ? (double)u * (double)u : 0.0);
          s += __shfl_xor(s, 16, 64);
          s2 += __shfl_xor(s2, 16, 64);
          if ((tid & 31) == 0) { red_sum[0][half] = s; red_sum[1][half] = s2; }
        }
        __syncthreads();
        if (quantizes) {  // the threads of a vector each derive the same scale factor
          const int n32 = dp / 32, first = q_lv * n32;
          float am = 0.0f;
          uint32_t any = 0u;
          double s = 0.0, s2 = 0.0;
          for (int h0 = 0; h0 < n32; h0 += 4) {
#pragma unroll
            for (int h = 0; h < 4; ++h) {
              const int at = h0 + h < n32 ? first + h0 + h : first;
              am = fmaxf(am, red_max[at]);
              any |= red_bad[at];
            }
          }
          if (csigma)
            for (int h = 0; h < n32; ++h) { s += red_sum[0][first + h]; s2 += red_sum[1][first + h]; }
          scale_of(am, s, s2);
          if (q_c == 0 && any) atomicOr(&a.flags[0], 1u);
          const float4 v4 = *reinterpret_cast<const float4 *>(us + q_lv * dp + q_c);
          u4[0] = v4.x; u4[1] = v4.y; u4[2] = v4.z; u4[3] = v4.w;
        }
      }
    }
    if constexpr (Q == kSharedScale) {  // the largest of the N scale factors, for everybody
      if (quantizes && q_c == 0) {
        if (!alone) st_word(a.scale_ex + (int64_t)par * a.N + v0 + q_lv, __builtin_bit_cast(uint32_t, q.delta), tag);
        else delta_sh[q_lv] = q.delta;
      }
      if (alone) __syncthreads();
      float dmax = 0.0f;
      if (wave < nv || !kWaveOwns) {
        for (int i = lane; i < a.N; i += 64)
          dmax = fmaxf(dmax, alone ? delta_sh[i]
                                   : __builtin_bit_cast(float, wait(a.scale_ex + (int64_t)par * a.N + i)));
        dmax = wave_max(dmax);
      }
      const float rd = 1.0f / dmax;
      const bool live = dmax > 0.0f && isfinite(rd);
      q.delta = live ? dmax : 0.0f;
      q.rdelta = live ? rd : 0.0f;
      q.thresh = dmax * hi_q;
    }
    // ---- codes (Sec. 3.2 rules (1), (2)) and words of the messages
    if (quantizes) {
      const uint32_t words[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
      u64 field = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float s = fminf(fmaxf(u4[c] * q.rdelta, lo_q), hi_q);
        const float base = floorf(s), frac = s - base;
        const float unif = (float)(words[c] >> 8) * 0x1.0p-24f;
        const int32_t code = q.delta > 0.0f ? (int32_t)base + ((unif < frac) ? 1 : 0) : 0;
        field |= (u64)((uint32_t)code & mask) << (c * a.bits);
      }
      // the 4 * bits bits of the group, OR-ed into the up to three words that they touch
      const int bit = q_c * a.bits, sh = bit & 31;
      uint32_t *to = own + q_lv * W1 + (bit >> 5);
      const u64 low = field << sh;
      const uint32_t high = sh ? (uint32_t)(field >> (64 - sh)) : 0u;
      if ((uint32_t)low) atomicOr(to, (uint32_t)low);
      if ((uint32_t)(low >> 32)) atomicOr(to + 1, (uint32_t)(low >> 32));
      if (high) atomicOr(to + 2, high);
      if (q_c == 0) own[q_lv * W1 + a.W] = __builtin_bit_cast(uint32_t, q.delta);
      if (a.n_clipped) {
        uint32_t clipped = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) clipped += (u4[c] > q.thresh || u4[c] < lo_q * q.delta) ? 1u : 0u;
        if (clipped) atomicAdd(&a.n_clipped[v0 + q_lv], clipped);
      }
    }
    // ---- this workgroup's messages out
    if constexpr (Q != kPlain) {
      auto send = [&](int lv, int wd) {
        const int v = v0 + lv;
        const uint32_t word = own[lv * W1 + wd];
        if (!alone) {
          st_word(a.msg + ((int64_t)par * a.N + v) * W1 + wd, word, tag);
          own[lv * W1 + wd] = 0u;  // for the next iteration
        }
        if (wd < a.W) a.packed[(int64_t)v * a.W + wd] = word;
        else a.delta_out[v] = __builtin_bit_cast(float, word);
      };
      if constexpr (kWaveOwns) {  // the wavefront's own words: no barrier between
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (wave < own_quant)
          for (int wd = lane; wd < W1; wd += 64) send(wave, wd);
      } else {
        __syncthreads();
        for (int e = tid; e < own_quant * W1; e += kClThreads) {
          const int lv = (int)__umulhi((uint32_t)e, a.inv_w1);
          send(lv, e - lv * W1);
        }
      }
    }
    // ---- while the words travel: the random words of the next codes, the rows of t + 2
    if (quantizes && t + 1 < a.it1) random_words(t + 1);
    if (draws && t + 2 < a.it1) draw(t + 2);
    // ---- everybody's messages; vectors in full precision: this thread's coordinate of each
    float avg = 0.0f, u_hat = 0.0f;
    if (!alone) {
      if constexpr (Q != kPlain)
        for (int e = tid; e < a.N * W1; e += kClThreads) msg[e] = wait(a.msg + (int64_t)par * a.N * W1 + e);
      if ((Q == kPlain || ALPC) && mine) {
        const u64 *src = a.vec + (int64_t)par * (Q == kPlain ? a.nvec : 1) * a.d + j;
        if constexpr (Q == kPlain) {
          for (int i0 = 0; i0 < a.N; i0 += 4) {  // four in flight
            u64 first[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) first[r] = ld_word(src + (int64_t)(i0 + r < a.N ? i0 + r : i0) * a.d);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              if (i0 + r < a.N)
                avg += __builtin_bit_cast(float, (uint32_t)(first[r] >> 32) == tag
                                                     ? (uint32_t)first[r]
                                                     : wait(src + (int64_t)(i0 + r) * a.d));
            }
          }
        }
        if constexpr (ALPC) u_hat = __builtin_bit_cast(float, wait(src + (Q == kPlain ? (int64_t)a.N * a.d : 0)));
      }
      if (!ok) fail_sh = 1u;
    }
    __syncthreads();
    if (!alone && fail_sh != 0u) { gave_up = true; break; }  // uniform: written before the barrier
    // ---- the receiver (eq. (4), or the integer sums of schemes (b), (c)) and the update
    if (mine) {
      if (alone) {
        if constexpr (Q == kPlain)
          for (int i = 0; i < a.N; ++i) avg += us[i * dp + j];
        if constexpr (ALPC) u_hat = uh[j];
      }
      if constexpr (Q == kPlain) avg *= inv_n;
      if constexpr (Q != kPlain) {
        float acc = 0.0f;
        int32_t isum = 0;
        const uint32_t *m = msg + wi_j, *md = msg + a.W;
        for (int i0 = 0; i0 < a.N; i0 += 4) {
          uint32_t lo[4], hi[4];
          float de[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int at = (i0 + r < a.N ? i0 + r : a.N - 1) * W1;
            lo[r] = m[at];
            hi[r] = m[at + 1];  // past the last word: the scale factor, not used then
            de[r] = __builtin_bit_cast(float, md[at]);
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (i0 + r < a.N) {
              const uint32_t field = two_j ? (lo[r] >> sh_j) | (hi[r] << (32 - sh_j)) : lo[r] >> sh_j;
              const int32_t code = (int32_t)(field << (32 - a.bits)) >> (32 - a.bits);
              if constexpr (Q == kOwnScale) acc = __builtin_fmaf(de[r], (float)code, acc);
              else isum += code;
            }
          }
        }
        if constexpr (Q == kOwnScale) {
          avg = acc * inv_n;
        } else {
          const float mean_code = (float)isum * inv_n, delta = __builtin_bit_cast(float, msg[a.W]);
          if (a.scheme == LPC_SCHEME_B) {
            avg = delta * mean_code;
          } else {  // eq. (5): the average rounded once more
            const float s = fminf(fmaxf(mean_code, lo_q), hi_q);
            const float base = floorf(s), frac = s - base;
            StreamKey k = a.key;
            k.iter = (uint32_t)t;
            const float unif = (float)(stream_word(k, kTagRequant, 0u, (uint32_t)j) >> 8) * 0x1.0p-24f;
            avg = delta * (float)((int32_t)base + ((unif < frac) ? 1 : 0));
          }
        }
      }
      if constexpr (ALPC) {
        const float yn = prox_scalar(x_j, avg + mu_j, a.step_y, a.thr_y, a.shrink_y);
        const float zn = prox_scalar(z_j, u_hat + mu_j, a.alpha, a.thr_z, a.shrink_z);
        y_j = yn;
        z_j = zn;
        ysum_j = t == 0 ? (float)weight * yn : ysum_j + (float)weight * yn;
        x_j = (a.t1 * zn + a.t2 * ws_j) + a.t3 * yn;
      } else {
        x_j = prox_scalar(x_j, avg + mu_j, a.step, a.thr, a.shrink);
      }
      xs[j] = x_j;
    }
    if constexpr (ALPC) weight *= a.theta;
    __syncthreads();
    if (Q != kPlain && alone)  // the messages have been read: cleared for the next codes, a barrier from here
      for (int e = tid; e < nv * W1; e += kClThreads) own[e] = 0u;
  }
  if (gave_up) {  // the iterate is not to be trusted; the others find the word at their next wait
    if (tid == 0) {
      __hip_atomic_store(a.ctl, a.tag0 + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      atomicOr(&a.flags[0], 2u);
    }
    return;
  }
  if (g == 0 && mine) {
    if (ALPC) {
      a.y_out[j] = y_j;
      a.z_out[j] = z_j;
      a.out[j] = ysum_j * a.out_scale;
    } else {
      a.out[j] = x_j;
    }
  }
}

struct Shape {
  int k, rw, nv, wpv, rpw, G;
  size_t lds;
};

// The launch for a context, or G = 0 where the kernel does not apply: a wavefront must hold its share of a batch in
// registers (64 K columns x RW rows: K RW values per lane, at most 32).
// One workgroup takes all vectors where every wavefront then has at most four rows of 64 columns: the exchange between
// workgroups (about 1.5 us) costs more than the other compute units give.  With twice as many rows it no longer does
// (d = 64, N = 16, B = 8: 7.1 us per iteration by one workgroup, 4.6 by sixteen).
Shape shape_of(const lpc_ctx *c) {
  Shape s{};
  const int32_t nvec = c->cfg.N + (c->cfg.algo != LPC_ALGO_LPC ? 1 : 0), B = c->cfg.B;
  if (c->csr || c->mlp || !c->grad_ok || c->n_full != c->n || c->n >= ((int64_t)1 << 31)) return s;
  if (c->d > 1024 || nvec > 64 || c->cfg.m < 1) return s;
  if (c->d > 256 && !c->quant) return s;  // vectors in full precision cross in column blocks (lpc_columns.hip)
  if ((int64_t)c->cfg.N * (c->quant ? c->W + 1 : 1) > 8192) return s;
  const int chunks = (int)((c->d + 63) / 64);
  s.k = chunks <= 1 ? 1 : (chunks <= 2 ? 2 : (chunks <= 4 ? 4 : (chunks <= 8 ? 8 : 16)));
  const int most = s.k == 16 ? 2 : (s.k == 8 ? 4 : (s.k == 4 ? 8 : 16));
  auto fits = [&](int nv) {
    if (nv > kClWaves || (int64_t)nv * c->d_pad > kClThreads || (int64_t)nv * B > kClThreads) return false;
    s.nv = nv;
    s.wpv = kClWaves / nv;
    s.rpw = (B + s.wpv - 1) / s.wpv;
    s.G = (nvec + nv - 1) / nv;
    return s.rpw <= most;
  };
  const bool ok = (fits(nvec) && s.rpw * s.k <= 4) || fits(1);
  if (!ok) {
    s.G = 0;
    return s;
  }
  s.rw = s.rpw <= 4 ? (s.k == 16 ? 2 : 4) : most;
  const size_t D = 64 * (size_t)s.k;
  s.lds = 4 * (D + kClWaves * D + (size_t)s.nv * c->d_pad + D +
               (size_t)(c->cfg.N + s.nv) * ((c->quant ? c->W : 0) + 1) + 6 * (size_t)s.nv * B);
  if (s.lds > (size_t)kClLds) s.G = 0;
  return s;
}

// The next snapshot and Alg. 2's vectors, out of what the loop's last launch left, unless one of its launches gave up: then
// the epoch has not taken place.  Only a launch of its own sees whether ALL workgroups came through; where the loop's
// workgroups wrote the caller's vectors themselves, some could have written their columns and others not.
__global__ __launch_bounds__(256) void commit_epoch_kernel(const uint32_t *__restrict__ ctl, uint32_t launch_tag, int32_t d,
                                                           const float *__restrict__ from, float scale,
                                                           float *__restrict__ w_snap, const float *__restrict__ y_from,
                                                           float *__restrict__ y, const float *__restrict__ z_from,
                                                           float *__restrict__ z) {
  if (ctl[0] == launch_tag) return;
  const int j = (int)(blockIdx.x * 256 + threadIdx.x);
  if (j >= d) return;
  w_snap[j] = y ? from[j] * scale : from[j];
  if (y) {
    y[j] = y_from[j];
    z[j] = z_from[j];
  }
}

}  // namespace

bool cluster_supported(const lpc_ctx *c) { return shape_of(c).G > 0; }

ClusterScratch cluster_scratch(const lpc_ctx *c) {
  const size_t N = (size_t)c->cfg.N, d = (size_t)c->d;
  ClusterScratch s;
  s.msg = 2 * N * ((c->quant ? (size_t)c->W : 0) + 1);
  s.vec = 2 * (c->quant ? 1 : N + 1) * d;
  s.scale = 2 * N;
  return s;
}

bool cluster_waits(const lpc_ctx *c) { return shape_of(c).G > 1; }

hipError_t launch_commit_epoch(const lpc_ctx *c, const ResidentStep &rs, double snap_scale, float *w_snap,
                               hipStream_t st) {
  hipLaunchKernelGGL(commit_epoch_kernel, dim3((unsigned)((c->d + 255) / 256)), dim3(256), 0, st, c->s.cl_ctl,
                     rs.tag0 + 1u, (int32_t)c->d, rs.alpc ? c->s.ysum : c->s.w, (float)snap_scale, w_snap, c->s.cl_y,
                     rs.alpc ? rs.y : nullptr, c->s.cl_z, rs.alpc ? rs.z : nullptr);
  return hipGetLastError();
}

hipError_t launch_cluster_epoch(const lpc_ctx *c, const ResidentStep &rs, float *w_snap, double snap_scale, int32_t t0,
                                int32_t t1, double weight, uint32_t *n_clipped, hipStream_t st) {
  const Shape s = shape_of(c);
  if (s.G > c->usable_cus) return hipErrorCooperativeLaunchTooLarge;
  ClusterArgs a{};
  fill_loop_args(a, c, rs, t0, t1, weight, n_clipped);
  // one workgroup in a launch: nobody can give up, the caller's vectors are written in place
  const bool alone = s.G == 1, last = alone && t1 == c->cfg.m;
  if (!alone && t0 > 0) { a.yv = c->s.cl_y; a.zv = c->s.cl_z; }
  float *kept = rs.alpc ? c->s.ysum : c->s.w;
  a.in = kept; a.out = last ? w_snap : kept; a.out_scale = last ? (float)snap_scale : 1.0f;
  a.y_out = alone ? rs.y : c->s.cl_y; a.z_out = alone ? rs.z : c->s.cl_z;
  a.packed = c->s.packed; a.delta_out = c->s.delta;
  a.msg = c->s.cl_msg; a.vec = c->s.cl_vec; a.scale_ex = c->s.cl_scale;
  a.dp = (int32_t)c->d_pad; a.nv = s.nv; a.G = s.G; a.wpv = s.wpv; a.rpw = s.rpw;
  a.inv_w1 = (uint32_t)((0x100000000ull + (uint64_t)a.W) / ((uint64_t)a.W + 1));
  const void *fn = nullptr;
  const int q = !c->quant ? kPlain : (c->cfg.scheme == LPC_SCHEME_A ? kOwnScale : kSharedScale);
#define LPC_CLUSTER_Q(K_, RW_, Q_)                                                                               \
  if (q == Q_)                                                                                                   \
    fn = rs.alpc ? reinterpret_cast<const void *>(&cluster_epoch_kernel<K_, RW_, Q_, true>)                      \
                 : reinterpret_cast<const void *>(&cluster_epoch_kernel<K_, RW_, Q_, false>);
#define LPC_CLUSTER_MESSAGES(K_, RW_)                                                                            \
  if (s.k == K_ && s.rw == RW_) { LPC_CLUSTER_Q(K_, RW_, kOwnScale) LPC_CLUSTER_Q(K_, RW_, kSharedScale) }
#define LPC_CLUSTER(K_, RW_)                                                                                     \
  LPC_CLUSTER_MESSAGES(K_, RW_)                                                                                  \
  if (s.k == K_ && s.rw == RW_) { LPC_CLUSTER_Q(K_, RW_, kPlain) }
  LPC_CLUSTER(1, 4) LPC_CLUSTER(1, 16) LPC_CLUSTER(2, 4) LPC_CLUSTER(2, 16) LPC_CLUSTER(4, 4) LPC_CLUSTER(4, 8)
  LPC_CLUSTER_MESSAGES(8, 4) LPC_CLUSTER_MESSAGES(16, 2)
#undef LPC_CLUSTER
#undef LPC_CLUSTER_MESSAGES
#undef LPC_CLUSTER_Q
  if (!fn) return hipErrorInvalidValue;
  if (s.lds > 60000) {  // wide rows only; asked for at every launch, because it holds for the current device alone
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kClLds);
    if (e != hipSuccess) return e;
  }
  void *args[] = {&a};
  if (s.G == 1) {
    a.spread = 1;
    return hipLaunchKernel(fn, dim3(1), dim3(kClThreads), args, s.lds, st);
  }
  // workgroup k of a launch runs on die k mod 8: every eighth one works, the others leave at once, so that the words
  // cross inside one die's L2 (only the speed depends on it)
  a.spread = 8 * s.G <= c->usable_cus ? 8 : 1;
  return hipLaunchCooperativeKernel(fn, dim3((unsigned)(s.G * a.spread)), dim3(kClThreads), args, (unsigned)s.lds, st);
}

}  // namespace lpc
