// HIP kernels of the Monte-Carlo diagnostics for gfx950 (MI355X).
//
// From what the loss call returns or reads per token t (the log-partition
// L_t, the student logits at the M cached draws, the cached teacher and
// behaviour log-probs), the one-sample terms of the estimator
//   log p = z - L,  A = tau - log p,  rho = exp(log p - beta),  X = -rho A
// give the statistics of Sec. 5.2 (the tail of rho_theta, Fig. 5) and App. E
// (variance of the m-sample estimator at a fixed prefix and averaged over a
// sequence, Table 6).  The data is a few megabytes, so launches and serial
// chains are what costs; the calls run in five launches:
//   zero     the quantile's histograms
//   rows     4 to 64 lanes per token (as M needs): mean, unbiased variance and
//            largest rho of its M terms; count of rho outside [1 - eps, 1 +
//            eps]; means of replicate groups of m draws and their variance; the
//            workgroup's parts of the batch sums; the histogram of the top 11
//            bits of rho
//   mid      the histogram of the next 11 bits within the bucket that holds the
//            wanted rank; and, in workgroups of their own, sums of the X
//            columns over pieces of the sequences
//   low      the histogram of the last 10 bits; and, in up to kDiagSeqGroups
//            workgroups of their own, the column averages of each sequence (from
//            the pieces, or from X where a sequence is short), the set variances
//            and their sums
//   final    the quantile; fixed-order sums of the parts in double; the batch
//            outputs
// rho >= 0, so its bits order like values.  Integer histograms make the
// selection exact and order-independent; every floating-point sum has a fixed
// order.  Measured (32,768 tokens, M = 16, three group sizes, 2,048-token
// sequences): 36 us a call (rows 18.9, mid 4.8, low 9.5, final 5.5 in a trace),
// against 116 in thirteen launches with a launch each for the parts and each
// bucket's choice and four passes of 8 bits, and 38 with the set variances in the
// final launch, where 2,048 sequences of one token and 256 draws took 13.6 ms (36
// us so).
#include <math.h>

#include "opd_device.h"

namespace opd {
namespace {

constexpr int kDiagThreads = 256;
constexpr int kDiagWaves = kDiagThreads / 64;
constexpr int kDiagQ = 3 + kDiagMaxGroups;
// key of a masked token's entries: above every ratio's
constexpr uint32_t kNoKey = 0xFFFFFFFFu;

// Sort key of one ratio: its bits, with every NaN mapped above +inf.
__device__ __forceinline__ uint32_t rho_key(float r) {
  return r != r ? 0x7FC00000u : __float_as_uint(r);
}

// The three digits of a key (top 11 of 32 bits, of which the first is 0; 11;
// 10) and where their histograms start.
constexpr int kBins0 = 1024, kBins1 = 2048, kBins2 = 1024;
constexpr int kHist1 = kBins0, kHist2 = kBins0 + kBins1, kSel = kHist2 + kBins2;
static_assert(kSel + 4 == kDiagHistWords, "the workspace holds the histograms and the state");
constexpr int digit_bins(int pass) { return pass == 1 ? kBins1 : kBins0; }
constexpr int digit_at(int pass) { return pass == 0 ? 0 : (pass == 1 ? kHist1 : kHist2); }
__device__ __forceinline__ uint32_t digit(uint32_t key, int pass) {
  return pass == 0 ? key >> 21 : (pass == 1 ? (key >> 10) & 2047u : key & 1023u);
}

__global__ void __launch_bounds__(1024) k_diag_zero(DiagArgs a) {
  for (int i = threadIdx.x; i < kDiagHistWords; i += 1024) a.ws_hist[i] = 0u;
}

// sums and maxima over the WIDTH lanes (a power of two) that share a token
template <int WIDTH>
__device__ __forceinline__ float sub_sum(float v) {
#pragma unroll
  for (int o = WIDTH >> 1; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
template <int WIDTH>
__device__ __forceinline__ float sub_max(float v) {
#pragma unroll
  for (int o = WIDTH >> 1; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// the sum over a wavefront, in lane 63 (DPP row shifts, then the row
// broadcasts; lanes without a source add 0)
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add_f64(double v) {
  u32x2 h = __builtin_bit_cast(u32x2, v);
  h[0] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h[0], CTRL, ROWS, 0xF, false);
  h[1] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h[1], CTRL, ROWS, 0xF, false);
  return v + __builtin_bit_cast(double, h);
}
__device__ __forceinline__ double wave_sum_f64(double v) {
  v = dpp_add_f64<0x111, 0xF>(v);
  v = dpp_add_f64<0x112, 0xF>(v);
  v = dpp_add_f64<0x114, 0xF>(v);
  v = dpp_add_f64<0x118, 0xF>(v);
  v = dpp_add_f64<0x142, 0xA>(v);
  return dpp_add_f64<0x143, 0xC>(v);
}

// Many waves, so that a wave does one or two rounds of its chain of loads and
// reductions, and few workgroups, so that few histograms are merged.
constexpr int kRowsThreads = 1024;
constexpr int kRowsWaves = kRowsThreads / 64;

// Workgroup b takes tokens [b per, (b + 1) per).  Quantities of the batch sums:
// [0] sum of row_var, [1] clipped entries, [2] valid tokens, [3 + k] sum of the
// group-k variances.
template <int WIDTH>
__global__ void __launch_bounds__(kRowsThreads, 8) k_diag_rows(DiagArgs a, int64_t per) {
  constexpr int NG = WIDTH < 64 ? 1 : kKMax / 64;  // groups per lane at most
  __shared__ float s_x[kRowsWaves][kKMax];
  __shared__ uint32_t s_h[kBins0];
  __shared__ double s_q[kRowsWaves][kDiagQ];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int M = a.M;
  constexpr int tpw = 64 / WIDTH;               // tokens per wave at a time
  const int sub = lane / WIDTH, l = lane & (WIDTH - 1);
  const int64_t t_end = min((int64_t)(blockIdx.x + 1) * per, a.N);
  for (int i = threadIdx.x; i < kBins0; i += kRowsThreads) s_h[i] = 0u;
  __syncthreads();
  double q[kDiagQ];
#pragma unroll
  for (int i = 0; i < kDiagQ; ++i) q[i] = 0.0;
  float* sx = &s_x[w][sub * M];  // (tpw > 1 only where M <= WIDTH)
  for (int64_t tb = (int64_t)blockIdx.x * per + w * tpw; tb < t_end; tb += kRowsWaves * tpw) {
    const int64_t t = tb + sub;
    const bool in = t < t_end;
    const bool valid = in && (!a.mask || a.mask[t] != 0);
    const float L = valid ? a.lse[t] : 0.f;
    float sum = 0.f, rmax = kNegInf, clip = 0.f;
    for (int i = l; i < M; i += WIDTH) {
      uint32_t key = kNoKey;
      float X = 0.f;
      if (valid) {
        const int64_t e = t * M + i;
        const float lp = a.gathered[e] - L;
        const float r = fast_exp2((lp - a.beta[e]) * kLog2e);
        X = -r * (a.tau[e] - lp);
        key = rho_key(r);
        if (a.rho_quantile) atomicAdd(&s_h[digit(key, 0)], 1u);
        rmax = fmaxf(rmax, r);
        clip += fabsf(r - 1.f) > a.clip_eps ? 1.f : 0.f;
        sum += X;
      }
      if (in) {
        if (a.rho_quantile) a.ws_rho[t * M + i] = key;
        if (a.ws_x) a.ws_x[t * M + i] = X;
      }
      sx[i] = X;
    }
    // (each wave reads back only what it wrote)
    __builtin_amdgcn_wave_barrier();
    const float mean = sub_sum<WIDTH>(sum) / (float)M;
    rmax = sub_max<WIDTH>(rmax);
    clip = sub_sum<WIDTH>(clip);
    float ss = 0.f;
    for (int i = l; i < M; i += WIDTH) {
      const float d = sx[i] - mean;
      ss += d * d;
    }
    ss = sub_sum<WIDTH>(ss);
    const float var = M >= 2 ? ss / (float)(M - 1) : __builtin_nanf("");
    if (l == 0 && in) {
      if (a.row_mean) a.row_mean[t] = valid ? mean : 0.f;
      if (a.row_var) a.row_var[t] = valid ? var : 0.f;
      if (a.row_rho_max)
        a.row_rho_max[t] = !valid ? 0.f : (rmax == kNegInf ? __builtin_nanf("") : rmax);
      if (valid) {
        q[0] += M >= 2 ? (double)var : 0.0;
        q[1] += (double)clip;
        q[2] += 1.0;
      }
    }
    // replicate groups of m consecutive draws
#pragma unroll 1
    for (int k = 0; k < a.n_groups; ++k) {
      const int m = a.group[k], G = M / m;
      float ys = 0.f;
      float y[NG];
#pragma unroll
      for (int h = 0; h < NG; ++h) {
        const int g = l + WIDTH * h;
        y[h] = 0.f;
        if (g < G) {
          float acc = 0.f;
          for (int i = g * m; i < g * m + m; ++i) acc += sx[i];
          y[h] = acc / (float)m;
          ys += y[h];
        }
      }
      const float ym = sub_sum<WIDTH>(ys) / (float)G;
      float yss = 0.f;
#pragma unroll
      for (int h = 0; h < NG; ++h)
        if (l + WIDTH * h < G) yss += (y[h] - ym) * (y[h] - ym);
      yss = sub_sum<WIDTH>(yss);
      const double v = l == 0 && valid ? (double)(yss / (float)(G - 1)) : 0.0;
#pragma unroll
      for (int i = 0; i < kDiagMaxGroups; ++i)
        if (i == k) q[3 + i] += v;
    }
    __builtin_amdgcn_wave_barrier();
  }
  // the workgroup's parts, in a fixed order
#pragma unroll
  for (int i = 0; i < kDiagQ; ++i)
    if (i < 3 + a.n_groups) {
      const double v = wave_sum_f64(q[i]);
      if (lane == 63) s_q[w][i] = v;
    }
  __syncthreads();
  if (threadIdx.x < 3 + a.n_groups) {
    double v = 0.0;
    for (int k = 0; k < kRowsWaves; ++k) v += s_q[k][threadIdx.x];
    a.ws_parts[(int64_t)blockIdx.x * kDiagQ + threadIdx.x] = v;
  }
  if (a.rho_quantile)
    for (int i = threadIdx.x; i < kBins0; i += kRowsThreads)
      if (s_h[i]) atomicAdd(&a.ws_hist[i], s_h[i]);
}

// The bucket of a pass's histogram that holds the wanted rank, found by every
// workgroup for itself (T lanes; an inclusive scan of the counts): the key
// prefix so far, and the rank within it.  Pass 0 turns the quantile into a
// rank.  `n` receives the count of entries (pass 0 only).  The state goes to
// the workspace for the launches after (the same values from each workgroup).
struct Picked {
  uint32_t prefix, rank, n;
};
template <int T, int PASS>
struct Pick {
  static constexpr int kBins = digit_bins(PASS), kPer = (kBins + T - 1) / T;
  uint32_t h[kPer];
  // requests this lane's buckets
  __device__ __forceinline__ void load(const DiagArgs& a) {
    const uint32_t* hist = a.ws_hist + digit_at(PASS);
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int b = (int)threadIdx.x * kPer + k;
      h[k] = b < kBins ? hist[b] : 0u;
    }
  }
  __device__ __forceinline__ Picked find(const DiagArgs& a, uint32_t prefix, uint32_t rank,
                                         uint32_t* s_w, uint32_t* s_out) const;
};
template <int T, int PASS>
__device__ __forceinline__ Picked Pick<T, PASS>::find(const DiagArgs& a, uint32_t prefix,
                                                      uint32_t rank, uint32_t* s_w,
                                                      uint32_t* s_out) const {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  uint32_t own = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) own += h[k];
  uint32_t incl = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t t = (uint32_t)__shfl_up((int)incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) s_w[w] = incl;
  __syncthreads();
  uint32_t n = 0;
  for (int j = 0; j < T / 64; ++j) {
    if (j < w) incl += s_w[j];
    n += s_w[j];
  }
  if (PASS == 0) {
    // nearest rank: the ceil(q n)-th smallest, at least the first
    const double want = ceil((double)a.q * (double)n);
    rank = n == 0 ? 1u : (uint32_t)(want < 1.0 ? 1.0 : (want > n ? (double)n : want));
  }
  // the one bucket with excl < rank <= incl (no entry: the last bucket)
  uint32_t excl = incl - own;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int b = tid * kPer + k;
    if (b < kBins &&
        ((excl < rank && rank <= excl + h[k]) || (b == kBins - 1 && excl + h[k] < rank))) {
      s_out[0] = prefix * (uint32_t)kBins + (uint32_t)b;
      s_out[1] = rank - excl;
    }
    excl += h[k];
  }
  __syncthreads();
  const Picked r{s_out[0], s_out[1], n};
  __syncthreads();
  return r;
}

// Sequence level: set 0 = the M single-draw columns, set k >= 1 = the means of
// group[k - 1] consecutive ones (a column's average over tokens commutes with the
// mean over draws); sequences without a valid token are skipped.  Workgroup b
// takes a range of sequences, as many at a time as fill its lanes, and leaves each
// set's sum of variances over them, in order.
__device__ __forceinline__ void seq_variances(const DiagArgs& a, int b, double* s_avg,
                                              double* s_var) {
  constexpr int T = kDiagThreads;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int M = a.M, sets = a.n_groups + 1;
  static_assert(T == kDiagSeqLanes, "a lane for each column and each set of a batch");
  const int64_t batch = a.seq_batch;
  // whole batches to a workgroup
  const int64_t per = ((a.nseq + batch - 1) / batch + a.seq_groups - 1) / a.seq_groups * batch;
  const int64_t s_end = min((int64_t)(b + 1) * per, a.nseq);
  double seq = 0.0;  // lane k < sets: set k
  for (int64_t s0 = (int64_t)b * per; s0 < s_end; s0 += batch) {
    const int ns = (int)min(batch, s_end - s0);
    if (tid < ns * M) {  // a column's average over the valid tokens of one sequence
      const int64_t s = s0 + tid / M;
      const int c = tid % M;
      double v = 0.0, n = 0.0;
      if (a.ws_psum) {
        const double* p = a.ws_psum + s * a.pieces * (M + 1);
#pragma unroll 8
        for (int64_t k = 0; k < a.pieces; ++k) {
          v += p[k * (M + 1) + c];
          n += p[k * (M + 1) + M];
        }
      } else {
        const int64_t t0 = s * a.seq_len, t1 = min(t0 + a.seq_len, a.N);
#pragma unroll 8
        for (int64_t t = t0; t < t1; ++t) {  // (a masked token's terms are 0)
          v += (double)a.ws_x[t * M + c];
          n += !a.mask || a.mask[t] != 0 ? 1.0 : 0.0;
        }
      }
      s_avg[tid] = n > 0.0 ? v / n : __builtin_nan("");
    }
    __syncthreads();
    if (M <= 64) {
      // a lane for each set of each sequence
      if (tid < ns * sets) {
        const int k = tid % sets, m = k ? a.group[k - 1] : 1, n = M / m;
        const double* avg = s_avg + (tid / sets) * M;
        double mean = 0.0;
        for (int c = 0; c < n * m; ++c) mean += avg[c];
        mean /= (double)(n * m);
        double ss = 0.0;
        for (int g = 0; g < n; ++g) {
          double y = 0.0;
          for (int c = g * m; c < g * m + m; ++c) y += avg[c];
          y = y / m - mean;
          ss += y * y;
        }
        s_var[tid] = avg[0] == avg[0] ? ss / (n - 1) : 0.0;
      }
    } else {
      // a wave for each, its lanes over the columns and then the groups
      for (int i = w; i < ns * sets; i += T / 64) {
        const int k = i % sets, m = k ? a.group[k - 1] : 1, n = M / m;
        const double* avg = s_avg + (i / sets) * M;
        double v = 0.0;
        for (int c = lane; c < n * m; c += 64) v += avg[c];
        const double mean = __shfl(wave_sum_f64(v), 63, 64) / (double)(n * m);
        double ss = 0.0;
        for (int g = lane; g < n; g += 64) {
          double y = 0.0;
          for (int c = g * m; c < g * m + m; ++c) y += avg[c];
          y = y / m - mean;
          ss += y * y;
        }
        ss = wave_sum_f64(ss);
        if (lane == 63) s_var[i] = avg[0] == avg[0] ? ss / (n - 1) : 0.0;
      }
    }
    __syncthreads();
    if (tid < sets)
      for (int s = 0; s < ns; ++s) seq += s_var[s * sets + tid];
    __syncthreads();
  }
  if (tid < sets) a.ws_seq[(int64_t)b * (kDiagMaxGroups + 1) + tid] = seq;
}

// The histogram of one of the later digits, over the keys whose earlier ones
// are the picked bucket's; workgroups from hist_groups on sum one piece of a
// sequence each in pass 1, and make the set variances in pass 2.
template <int PASS>
__global__ void __launch_bounds__(kDiagThreads) k_diag_hist(DiagArgs a, unsigned hist_groups) {
  __shared__ uint32_t h[digit_bins(PASS)];
  __shared__ uint32_t s_w[kDiagWaves], s_out[2];
  const int tid = threadIdx.x;
  if (PASS == 1 && blockIdx.x >= hist_groups) {
    // lanes as (token, column): c = tid % M of token tid / M
    __shared__ double s_sum[kDiagThreads];
    __shared__ uint32_t s_n[kDiagThreads];
    const int64_t piece = blockIdx.x - hist_groups;
    const int64_t s = piece / a.pieces, k = piece % a.pieces;
    const int64_t t0 = s * a.seq_len + k * kDiagPiece;
    const int64_t t1 = min(min(t0 + kDiagPiece, (s + 1) * a.seq_len), a.N);
    const int M = a.M, R = kDiagThreads / M, tr = tid / M, c = tid - tr * M;
    double acc = 0.0;
    uint32_t nv = 0;
    if (tr < R)
#pragma unroll 4
      for (int64_t t = t0 + tr; t < t1; t += R) {  // (a masked token's terms are 0)
        acc += (double)a.ws_x[t * M + c];
        nv += !a.mask || a.mask[t] != 0 ? 1u : 0u;
      }
    s_sum[tid] = acc;
    s_n[tid] = nv;
    __syncthreads();
    if (tid < M) {
      double v = 0.0;
      uint32_t n = 0;
      for (int j = 0; j < R; ++j) {
        v += s_sum[j * M + tid];
        n += s_n[j * M + tid];
      }
      a.ws_psum[piece * (M + 1) + tid] = v;
      if (tid == 0) a.ws_psum[piece * (M + 1) + M] = (double)n;
    }
    return;
  }
  if (PASS == 2 && blockIdx.x >= hist_groups) {
    __shared__ double s_avg[kDiagThreads];
    __shared__ double s_var[kDiagThreads];
    seq_variances(a, (int)(blockIdx.x - hist_groups), s_avg, s_var);
    return;
  }
  Pick<kDiagThreads, PASS - 1> before;
  before.load(a);
  const Picked p = before.find(a, PASS == 1 ? 0u : a.ws_hist[kSel],
                               PASS == 1 ? 0u : a.ws_hist[kSel + 1], s_w, s_out);
  for (int i = tid; i < digit_bins(PASS); i += kDiagThreads) h[i] = 0u;
  __syncthreads();
  const uint32_t prefix = p.prefix;
  auto count = [&](uint32_t key) {
    if ((PASS == 1 ? key >> 21 : key >> 10) == prefix) atomicAdd(&h[digit(key, PASS)], 1u);
  };
  // (a masked token's key shares no prefix with a ratio's)
  const int64_t total = a.N * a.M, quads = total / 4;
  for (int64_t e = (int64_t)blockIdx.x * kDiagThreads + tid; e < quads;
       e += (int64_t)hist_groups * kDiagThreads) {
    const u32x4 v = ((const u32x4*)a.ws_rho)[e];
#pragma unroll
    for (int k = 0; k < 4; ++k) count(v[k]);
  }
  if (blockIdx.x == 0 && tid < (int)(total - 4 * quads)) count(a.ws_rho[4 * quads + tid]);
  __syncthreads();
  for (int i = tid; i < digit_bins(PASS); i += kDiagThreads)
    if (h[i]) atomicAdd(&a.ws_hist[digit_at(PASS) + i], h[i]);
  // Pass 2 still reads its state here, so it leaves its own in other words.
  if (blockIdx.x == 0 && tid == 0) {
    a.ws_hist[kSel + (PASS == 1 ? 0 : 2)] = p.prefix;
    a.ws_hist[kSel + (PASS == 1 ? 1 : 3)] = p.rank;
  }
}

// One workgroup: the quantile, the batch sums, the sequence-level ratios.
constexpr int kFinalThreads = 1024;

__global__ void __launch_bounds__(kFinalThreads) k_diag_final(DiagArgs a, int parts) {
  constexpr int T = kFinalThreads, W = T / 64;
  __shared__ uint32_t s_w[W], s_out[2];
  static_assert(kDiagQ <= W, "a wave for each quantity");
  __shared__ double tot[kDiagQ];
  __shared__ double seq[kDiagMaxGroups + 1];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int M = a.M, sets = a.n_groups + 1;
  // what every part below needs from memory is requested first: one round trip
  Pick<T, 2> last;
  uint32_t prefix = 0, rank = 0;
  if (a.rho_quantile) {
    last.load(a);
    prefix = a.ws_hist[kSel + 2];
    rank = a.ws_hist[kSel + 3];
  }
  const bool with_seq = a.ratio_seq && a.ws_seq;
  // batch sums: wave i adds the parts of quantity i, and those of set i
  double v = 0.0, sv = 0.0;
  if (w < 3 + a.n_groups) {
#pragma unroll 8
    for (int p = lane; p < parts; p += 64) v += a.ws_parts[(int64_t)p * kDiagQ + w];
  }
  if (with_seq && w < sets) {
#pragma unroll 4
    for (int p = lane; p < a.seq_groups; p += 64)
      sv += a.ws_seq[(int64_t)p * (kDiagMaxGroups + 1) + w];
  }
  v = wave_sum_f64(v);
  sv = wave_sum_f64(sv);
  if (lane == 63) {
    if (w < 3 + a.n_groups) tot[w] = v;
    if (w < sets) seq[w] = sv;
  }
  __syncthreads();
  if (a.rho_quantile) {
    const Picked p = last.find(a, prefix, rank, s_w, s_out);
    // (tot[2] valid tokens; none: no ratio)
    if (tid == 0) a.rho_quantile[0] = tot[2] > 0.0 ? __uint_as_float(p.prefix) : __builtin_nanf("");
  }
  if (tid == 0) {
    const double n = tot[2] * (double)M;
    if (a.clip_frac) a.clip_frac[0] = n > 0 ? (float)(tot[1] / n) : __builtin_nanf("");
    for (int k = 0; k < a.n_groups; ++k) {
      if (a.ratio_local) a.ratio_local[k] = (float)(tot[3 + k] / tot[0]);
      if (with_seq) a.ratio_seq[k] = (float)(seq[1 + k] / seq[0]);
    }
  }
}

}  // namespace

hipError_t launch_diag(const DiagArgs& a, hipStream_t stream) {
  if (a.N == 0) return hipSuccess;
  const dim3 blk(kDiagThreads);
  const int parts = diag_parts(a.N);
  const int64_t per = (a.N + parts - 1) / parts;
  if (a.rho_quantile) hipLaunchKernelGGL(k_diag_zero, dim3(1), dim3(1024), 0, stream, a);
  // lanes per token: the power of two that holds its M entries, 64 at most
  const dim3 rgrid((unsigned)parts), rblk(kRowsThreads);
  if (a.M <= 4)
    hipLaunchKernelGGL(k_diag_rows<4>, rgrid, rblk, 0, stream, a, per);
  else if (a.M <= 8)
    hipLaunchKernelGGL(k_diag_rows<8>, rgrid, rblk, 0, stream, a, per);
  else if (a.M <= 16)
    hipLaunchKernelGGL(k_diag_rows<16>, rgrid, rblk, 0, stream, a, per);
  else if (a.M <= 32)
    hipLaunchKernelGGL(k_diag_rows<32>, rgrid, rblk, 0, stream, a, per);
  else
    hipLaunchKernelGGL(k_diag_rows<64>, rgrid, rblk, 0, stream, a, per);
  const int64_t quads = (a.N * a.M / 4 + kDiagThreads - 1) / kDiagThreads;
  const unsigned groups = a.rho_quantile ? (unsigned)(quads < 1 ? 1 : (quads < 512 ? quads : 512)) : 0u;
  const unsigned pieces = a.ws_psum ? (unsigned)(a.nseq * a.pieces) : 0u;
  const unsigned seqs = a.ws_seq ? (unsigned)a.seq_groups : 0u;
  if (groups + pieces > 0)
    hipLaunchKernelGGL(k_diag_hist<1>, dim3(groups + pieces), blk, 0, stream, a, groups);
  if (groups + seqs > 0)
    hipLaunchKernelGGL(k_diag_hist<2>, dim3(groups + seqs), blk, 0, stream, a, groups);
  hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(kFinalThreads), 0, stream, a, parts);
  return hipGetLastError();
}

}  // namespace opd
