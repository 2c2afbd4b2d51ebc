// Evaluators beside the hot path (gfx950): the gradient-mapping metric of
// Sec. 3.3, the histogram of a packed message's codes and the optimal
// prefix-code size it implies (entropy coding of the messages, Sec. 6.1), and
// the left-hand side of Theorem 2's step-size conditions (eq. (6), (7)), and the emission of the entropy-coded
// bit stream (canonical prefix code, codewords most significant bit first).
// None of these runs inside an epoch.  Sums are fp64, in a fixed order; the launches are wide and leave what the host asks
// for in a slot that it polls, because a monitored run calls them after every epoch.
#include <hip/hip_runtime.h>

#include <functional>
#include <queue>
#include <vector>

#include "lpc_device.h"
#include "lpc_internal.h"

namespace lpc {

namespace {

// partial[g] = workgroup g's share of |G_eta(w)|^2, G_eta(w) = (w - prox_{eta h}(w - eta*grad))/eta: coordinates
// g*1024 + tid, then in steps of 1024*gridDim.x, four in flight per thread; fp64, fixed order.  (One workgroup for
// all of d took 58 us on 150,001 coordinates, its threads walking 147 coordinates and fp64 divisions one by one.)
__global__ __launch_bounds__(1024) void gradient_mapping_kernel(const float *__restrict__ w,
                                                                const float *__restrict__ grad, int64_t d, double eta,
                                                                double l1, double l2, double *__restrict__ partial) {
  __shared__ double red[16];
  const int tid = threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * 1024;
  const double thr = eta * l1, shrink = 1.0 / (1.0 + eta * l2), inv = 1.0 / eta;
  double a = 0.0;
  for (int64_t j = (int64_t)blockIdx.x * 1024 + tid; j < d; j += 4 * stride) {
    float wv[4], gv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool in = j + q * stride < d;
      wv[q] = in ? w[j + q * stride] : 0.0f;
      gv[q] = in ? grad[j + q * stride] : 0.0f;  // zeros map to zero
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double x = (double)wv[q];
      const double p = x - eta * (double)gv[q];
      const double mag = fabs(p) - thr;
      const double px = mag > 0.0 ? copysign(mag, p) * shrink : 0.0;
      const double g = (x - px) * inv;
      a += g * g;
    }
  }
  a = wave_sum(a);
  if ((tid & 63) == 0) red[tid >> 6] = a;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int k = 0; k < 16; ++k) t += red[k];
    partial[blockIdx.x] = t;
  }
}

// total += sum_i n_clipped[i] (one thread; N is the number of workers)
__global__ void accumulate_clipped_kernel(const uint32_t *__restrict__ n_clipped, int32_t N,
                                          unsigned long long *__restrict__ total) {
  unsigned long long t = *total;
  for (int32_t i = 0; i < N; ++i) t += n_clipped[i];
  *total = t;
}

__global__ void zero_u64_kernel(unsigned long long *__restrict__ dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = 0ull;
}

// The B words of one 32-coordinate segment and its symbols (bin index = code + 2^(B-1)).  B is a template parameter so
// that a field's word and shift are constants and the words stay in registers.
template <int B>
struct Segment {
  uint32_t w[B];
  __device__ __forceinline__ void load(const uint32_t *__restrict__ seg) {
    if constexpr (B % 4 == 0) {
#pragma unroll
      for (int i = 0; i < B; i += 4) {
        const uint4 t = *reinterpret_cast<const uint4 *>(seg + i);
        w[i] = t.x; w[i + 1] = t.y; w[i + 2] = t.z; w[i + 3] = t.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < B; ++i) w[i] = seg[i];
    }
  }
  template <int J>
  __device__ __forceinline__ uint32_t symbol() const {
    constexpr int off = J * B, wi = off >> 5, sh = off & 31;
    constexpr uint32_t mask = (1u << B) - 1u, bias = 1u << (B - 1);
    uint32_t f = w[wi] >> sh;
    if constexpr (sh + B > 32) f |= w[wi + 1] << (32 - sh);
    // two's complement field -> bin index: adding 2^(B-1) modulo 2^B maps -2^(B-1).. to 0..
    return ((f & mask) + bias) & mask;
  }
};
// f(symbol) for the first cnt (of 32) coordinates of a segment, in order; whole segments without a check per coordinate
template <int B, bool WHOLE, int J, class F>
__device__ __forceinline__ void for_symbols_from(const Segment<B> &s, int cnt, F &f) {
  if constexpr (J < 32) {
    if (WHOLE || J < cnt) f(s.template symbol<J>());
    for_symbols_from<B, WHOLE, J + 1>(s, cnt, f);
  }
}
template <int B, class F>
__device__ __forceinline__ void for_symbols(const Segment<B> &s, int cnt, F f) {
  if (cnt == 32) for_symbols_from<B, true, 0>(s, cnt, f);
  else for_symbols_from<B, false, 0>(s, cnt, f);
}

// counts[symbol] += 1 for the first d coordinates of one packed message, one 32-coordinate segment per thread and step.
// Up to 8192 bins are counted in LDS.  The codes of a message are close to normal: with 16 bins most of a wavefront
// asks for the same few counters, and additions to one LDS address are taken one after the other.  Up to 256 bins
// (B <= 8) therefore have 32 copies, one per LDS bank: lane l uses copy l % 32 of its bin, so a wavefront's additions
// hit distinct banks.  4.2 M coordinates, B = 4: 13.7 us with one copy, 6.2 us with 32.
constexpr int kHistCopies = 32;
constexpr int kLdsBins = 8192;

template <int B>
__global__ __launch_bounds__(256) void code_histogram_kernel(const uint32_t *__restrict__ words, int64_t d,
                                                             unsigned long long *__restrict__ counts) {
  constexpr int kBins = 1 << B;
  constexpr bool kCopied = kBins * kHistCopies <= kLdsBins, kLds = kBins <= kLdsBins;
  constexpr int kSize = kCopied ? kBins * kHistCopies : (kLds ? kBins : 1);
  __shared__ uint32_t bins[kSize];
  const int tid = threadIdx.x;
  if constexpr (kLds) {
    for (int k = tid; k < kSize; k += 256) bins[k] = 0u;
    __syncthreads();
  }
  const int64_t segs = (d + 31) / 32;
  for (int64_t s = (int64_t)blockIdx.x * 256 + tid; s < segs; s += (int64_t)gridDim.x * 256) {
    Segment<B> seg;
    seg.load(words + s * B);
    const int64_t left = d - s * 32;
    for_symbols<B>(seg, left < 32 ? (int)left : 32, [&](uint32_t bin) {
      if constexpr (kCopied) atomicAdd(&bins[bin * kHistCopies + (tid & (kHistCopies - 1))], 1u);
      else if constexpr (kLds) atomicAdd(&bins[bin], 1u);
      else atomicAdd(&counts[bin], 1ull);
    });
  }
  if constexpr (kLds) {
    __syncthreads();
    for (int k = tid; k < kBins; k += 256) {
      uint32_t t = 0u;
      if constexpr (kCopied) {
        for (int r = 0; r < kHistCopies; ++r) t += bins[k * kHistCopies + ((r + k) & (kHistCopies - 1))];
      } else {
        t = bins[k];
      }
      if (t) atomicAdd(&counts[k], (unsigned long long)t);
    }
  }
}

}  // namespace

hipError_t launch_gradient_mapping(const lpc_ctx *c, const float *w, const float *grad, double eta, hipStream_t st) {
  hipLaunchKernelGGL(gradient_mapping_kernel, dim3((unsigned)result_groups(c)), dim3(1024), 0, st, w, grad, c->d, eta,
                     (double)c->prob.lambda1, (double)c->prob.lambda2, c->s.stat_part);
  return hipGetLastError();
}

namespace {

// ---- entropy-coded stream of one message ---------------------------------------------------------------------------
// Two launches.  A workgroup owns kEmitSegs = 255 consecutive segments, one per thread.
//   measure: the encoded size of every workgroup's share (bit 31: a coordinate's symbol has no codeword);
//   emit:    every workgroup adds up the sizes of the shares before its own (a few hundred words out of the L2), scans
//            its segments' sizes, and assembles its part of the stream in LDS.  A stream word belongs to the workgroup
//            in whose share its first bit lies; the last word of a share is completed from the following segment, which
//            thread 255 encodes (it has at least 32 coordinates of at least one bit, or it is the message's last).  So
//            every word is written once, with a plain store, and the output needs no clearing.
// 4.2 M coordinates, b = 4 (one MI355X): 282 us for sizes per segment, a scan by one workgroup whose threads walked
// their shares word by word, a fill, and codewords OR-ed into global memory; 14.5 us for these two launches.
constexpr int kEmitSegs = 255;
constexpr uint32_t kBadBit = 0x80000000u;

// codewords of up to 256 symbols travel in the kernel's arguments (no copy to the device ahead of the launch);
// `far` holds the table where there are more
struct HuffTable {
  HuffEntry e[256];
  const HuffEntry *far;
};

template <int B>
__device__ __forceinline__ const HuffEntry *huffman_stage(const HuffTable &t, HuffEntry *lds, int tid) {
  if constexpr (B > 8) {
    return t.far;
  } else {
    if (tid < (1 << B)) lds[tid] = t.e[tid];
    __syncthreads();
    return lds;
  }
}

// encoded bits of this thread's segment (kBadBit: a symbol without codeword)
template <int B>
__device__ __forceinline__ uint32_t huffman_segment_bits(const Segment<B> &seg, int cnt, const HuffEntry *table) {
  uint32_t total = 0, bad = 0;
  for_symbols<B>(seg, cnt, [&](uint32_t s) {
    const uint32_t len = table[s].len;
    bad |= len == 0 ? kBadBit : 0u;
    total += len;
  });
  return total | bad;
}

template <int B>
__global__ __launch_bounds__(256) void huffman_measure_kernel(const uint32_t *__restrict__ words, int64_t d,
                                                              HuffTable table, uint32_t *__restrict__ wg_bits) {
  __shared__ HuffEntry lds[B > 8 ? 1 : (1 << B)];
  __shared__ uint32_t red[4];
  const int tid = threadIdx.x;
  const HuffEntry *tab = huffman_stage<B>(table, lds, tid);
  const int64_t s = (int64_t)blockIdx.x * kEmitSegs + tid, left = d - s * 32;
  uint32_t bits = 0;
  if (tid < kEmitSegs && left > 0) {
    Segment<B> seg;
    seg.load(words + s * B);
    bits = huffman_segment_bits<B>(seg, left < 32 ? (int)left : 32, tab);
  }
  const uint32_t sum = wave_sum(bits & ~kBadBit);
  const uint32_t bad = __ballot((bits & kBadBit) != 0u) ? kBadBit : 0u;
  if ((tid & 63) == 0) red[tid >> 6] = sum | bad;
  __syncthreads();
  if (tid == 0)
    wg_bits[blockIdx.x] = (((red[0] & ~kBadBit) + (red[1] & ~kBadBit)) + ((red[2] & ~kBadBit) + (red[3] & ~kBadBit))) |
                          ((red[0] | red[1] | red[2] | red[3]) & kBadBit);
}

// meta (a host slot): total bits, and whether a coordinate has no codeword; out is written only if all is well and
// the stream fits capacity_words.  Dynamic LDS: 256 * (longest codeword) + 2 words.
template <int B>
__global__ __launch_bounds__(256) void huffman_emit_kernel(const uint32_t *__restrict__ words, int64_t d,
                                                           HuffTable table, const uint32_t *__restrict__ wg_bits,
                                                           uint32_t buffer_words, int64_t capacity_words,
                                                           uint32_t *__restrict__ out,
                                                           unsigned long long *__restrict__ meta) {
  extern __shared__ uint32_t buf[];
  __shared__ HuffEntry lds[B > 8 ? 1 : (1 << B)];
  __shared__ unsigned long long before_sh[4], all_sh[4];
  __shared__ uint32_t bad_sh[4], scan_sh[4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t s = (int64_t)blockIdx.x * kEmitSegs + tid, left = d - s * 32;
  const int cnt = left < 32 ? (left > 0 ? (int)left : 0) : 32;
  Segment<B> seg;
  if (cnt > 0) seg.load(words + s * B);
  // the shares before this one, and all of them
  unsigned long long before = 0, all = 0;
  uint32_t bad = 0;
  for (uint32_t k = tid; k < gridDim.x; k += 256) {
    const uint32_t t = wg_bits[k];
    const uint32_t v = t & ~kBadBit;
    bad |= t & kBadBit;
    all += v;
    if (k < blockIdx.x) before += v;
  }
  const uint32_t share = wg_bits[blockIdx.x] & ~kBadBit, used_words = share / 32 + 3;  // with the skew and a part word
  for (uint32_t k = tid; k < (used_words < buffer_words ? used_words : buffer_words); k += 256) buf[k] = 0u;
  const HuffEntry *tab = huffman_stage<B>(table, lds, tid);  // a barrier for B <= 8
  const uint32_t mine = huffman_segment_bits<B>(seg, cnt, tab) & ~kBadBit;
  uint32_t incl = mine;  // inclusive scan over the wavefront
#pragma unroll
  for (int step = 1; step < 64; step <<= 1) {
    const uint32_t up = __shfl_up(incl, step, 64);
    if (lane >= step) incl += up;
  }
#pragma unroll
  for (int step = 32; step >= 1; step >>= 1) {
    before += __shfl_xor(before, step, 64);
    all += __shfl_xor(all, step, 64);
  }
  bad = __ballot(bad != 0u) ? 1u : 0u;
  if (lane == 63) scan_sh[wv] = incl;
  if (lane == 0) { before_sh[wv] = before; all_sh[wv] = all; bad_sh[wv] = bad; }
  __syncthreads();
  before = before_sh[0] + before_sh[1] + before_sh[2] + before_sh[3];
  all = all_sh[0] + all_sh[1] + all_sh[2] + all_sh[3];
  bad = bad_sh[0] | bad_sh[1] | bad_sh[2] | bad_sh[3];
  if (blockIdx.x == 0 && tid == 0) { meta[0] = all; meta[1] = bad; hand_over(meta); }
  const int64_t need = (int64_t)((all + 31) / 32);
  if (bad || need > capacity_words) return;  // uniform over the launch
  for (int k = 0; k < wv; ++k) incl += scan_sh[k];
  const uint32_t skew = (uint32_t)(before & 31ull);          // bits of the first word that belong to earlier shares
  const uint32_t at = skew + incl - mine;                    // this segment's first bit in buf
  uint32_t wi = at >> 5, filled = at & 31u;
  const uint32_t stop = tid < kEmitSegs ? buffer_words : wi + 1;  // the following segment completes one word only
  unsigned long long acc = 0;
  for_symbols<B>(seg, cnt, [&](uint32_t sym) {
    const HuffEntry e = tab[sym];
    acc |= (unsigned long long)e.rev << filled;  // filled <= 31, e.len <= 32
    filled += e.len;
    if (filled >= 32) {
      if (wi < stop) atomicOr(&buf[wi], (uint32_t)acc);
      acc >>= 32;
      filled -= 32;
      ++wi;
    }
  });
  if ((uint32_t)acc && wi < stop) atomicOr(&buf[wi], (uint32_t)acc);
  __syncthreads();
  // words whose first bit lies in [before, before + share)
  const unsigned long long end = before + (unsigned long long)share;
  const int64_t w0 = (int64_t)(before >> 5), first = (int64_t)((before + 31) >> 5), last = (int64_t)((end + 31) >> 5);
  for (int64_t w = first + tid; w < last; w += 256) out[w] = buf[w - w0];
}

}  // namespace

int64_t huffman_wgs(int64_t d) { return ((d + 31) / 32 + kEmitSegs - 1) / kEmitSegs; }

// Both launches: sizes, then the stream into out (nothing when it does not fit or a symbol has no codeword) with
// {total bits, bad symbol} in meta.  table: 2^bits codewords on the host, far: the same on the device where bits > 8.
hipError_t launch_huffman(const lpc_ctx *c, const uint32_t *words, const HuffEntry *table, const HuffEntry *far,
                          uint32_t *out, int64_t capacity_words, unsigned long long *meta, hipStream_t st) {
  HuffTable t{};
  t.far = far;
  const int nsym = 1 << c->cfg.bits;
  uint32_t longest = 0;
  for (int k = 0; k < nsym; ++k) {
    if (nsym <= 256) t.e[k] = table[k];
    longest = table[k].len > longest ? table[k].len : longest;
  }
  const dim3 grid((unsigned)huffman_wgs(c->d));
  const uint32_t buffer_words = 256u * longest + 2u;
#define CALL(BITS)                                                                                                     \
  do {                                                                                                                 \
    hipLaunchKernelGGL(huffman_measure_kernel<BITS>, grid, dim3(256), 0, st, words, c->d, t, c->s.huff_wg_bits);       \
    hipLaunchKernelGGL(huffman_emit_kernel<BITS>, grid, dim3(256), buffer_words * sizeof(uint32_t), st, words, c->d,   \
                       t, (const uint32_t *)c->s.huff_wg_bits, buffer_words, capacity_words, out, meta);               \
  } while (0)
  LPC_DISPATCH_BITS(c->cfg.bits, CALL)
#undef CALL
  return hipGetLastError();
}

// out[0] = sum of the n clip counts, out[1] = bits of the largest of the n scale factors (one workgroup, fixed order)
__global__ __launch_bounds__(256) void epoch_report_kernel(const float *__restrict__ delta,
                                                           const uint32_t *__restrict__ nclip, int64_t n,
                                                           unsigned long long *__restrict__ out) {
  __shared__ double sum_sh[4];
  __shared__ float max_sh[4];
  const int tid = threadIdx.x;
  double sum = 0.0;
  float mx = 0.0f;
  for (int64_t k = tid; k < n; k += 256) {
    sum += (double)nclip[k];
    mx = fmaxf(mx, delta[k]);
  }
  sum = wave_sum(sum);
  mx = wave_max(mx);
  if ((tid & 63) == 0) { sum_sh[tid >> 6] = sum; max_sh[tid >> 6] = mx; }
  __syncthreads();
  if (tid == 0) {
    out[0] = (unsigned long long)(((sum_sh[0] + sum_sh[1]) + sum_sh[2]) + sum_sh[3]);
    out[1] = (unsigned long long)__float_as_uint(fmaxf(fmaxf(max_sh[0], max_sh[1]), fmaxf(max_sh[2], max_sh[3])));
  }
}

hipError_t launch_epoch_report(const float *delta, const uint32_t *nclip, int64_t n, unsigned long long *out,
                               hipStream_t st) {
  hipLaunchKernelGGL(epoch_report_kernel, dim3(1), dim3(256), 0, st, delta, nclip, n, out);
  return hipGetLastError();
}

hipError_t launch_accumulate_clipped(const uint32_t *n_clipped, int32_t N, unsigned long long *total, hipStream_t st) {
  hipLaunchKernelGGL(accumulate_clipped_kernel, dim3(1), dim3(1), 0, st, n_clipped, N, total);
  return hipGetLastError();
}

hipError_t launch_code_histogram(const uint32_t *words, int64_t d, int32_t bits, uint64_t *counts, hipStream_t st) {
  const int64_t nbins = (int64_t)1 << bits;
  auto *cnt = reinterpret_cast<unsigned long long *>(counts);
  hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)((nbins + 255) / 256)), dim3(256), 0, st, cnt, nbins);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || d <= 0) return e;
  const int64_t segs = (d + 31) / 32;
  int64_t wgs = (segs + 255) / 256;
  if (wgs > 256) wgs = 256;  // one per CU: every further one repeats the 2^b additions to the global counters
#define CALL(BITS) hipLaunchKernelGGL(code_histogram_kernel<BITS>, dim3((unsigned)wgs), dim3(256), 0, st, words, d, cnt)
  LPC_DISPATCH_BITS(bits, CALL)
#undef CALL
  return hipGetLastError();
}

}  // namespace lpc
