// HIP kernels that build the teacher-score cache for gfx950 (MI355X).
//
// Sec. 4.1 splits the pipeline into Stage 1, where rollout draws actions
// from the stale student p_old and records their rollout-time
// log-probabilities (or keeps its top-k support), and Stage 2, where the
// teacher scores the cached actions.  Three row operations cover it:
//   sample  M draws from softmax(z) by inversion of its index-order CDF at
//           caller-supplied uniforms (rollout at temperature 1 with no top-p
//           or top-k truncation, App. B), plus log softmax(z) at the draws;
//   top-k   the k largest logits (descending, equal values by lower index),
//           plus log softmax(z) there;
//   score   log softmax(z) at given ids.
// One 1024-lane workgroup per token row.  A row that fits the registers
// (bf16 up to 155,648 entries, fp32 up to 77,824) is loaded once and kept
// there; wider rows are streamed.
#include <math.h>

#include <type_traits>

#include "opd_device.h"

namespace opd {
namespace {

constexpr int NT = kRowThreads;
constexpr int NW = NT / 64;
// ids_out[row * k] of a row the streamed top-k kernel leaves to the resident one
constexpr int32_t kTopkRedo = -2;

// ---------------------------------------------------------------- rows

// max of three fp32 values by the hardware instruction, without the quieting
// of signalling NaNs that fmaxf adds for inputs of unknown origin (where it
// is used, a NaN input is caught another way)
__device__ __forceinline__ float max3_raw(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}


// Elements [valid, 4) of a vector replaced by -inf, without branches (the
// masks depend only on the wave-uniform count).
template <class TI>
__device__ __forceinline__ typename TI::Vec tail_masked(typename TI::Vec x, int valid) {
  if constexpr (TI::BYTES == 2) {
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const uint32_t keep = (2 * d < valid ? 0x0000FFFFu : 0u) | (2 * d + 1 < valid ? 0xFFFF0000u : 0u);
      x[d] = (x[d] & keep) | (0xFF80FF80u & ~keep);
    }
  } else {
#pragma unroll
    for (int d = 0; d < 4; ++d) x[d] = d < valid ? x[d] : 0xFF800000u;
  }
  return x;
}

// Resident row in the slot layout of the loss kernels.  Lanes outside the
// row, and elements of the last vector past V, read as -inf.
template <class TI, int NSLOT>
__device__ __forceinline__ void load_row(const void* zrow, uint32_t nvec, int tail, int tid,
                                         typename TI::Vec (&x)[NSLOT]) {
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const uint32_t b = slot_base<NT>(s, nvec);
    x[s] = ld_nt<TI>((const typename TI::Vec*)zrow + b, slot_off<NT>(s, b, tid, nvec));
  }
#pragma unroll
  for (int s = 0; s < NSLOT; ++s)
    if ((uint32_t)(s * NT + NT) > nvec && !slot_owns<NT>(s, slot_base<NT>(s, nvec), tid, nvec))
      x[s] = neg_inf_vec<TI>();
  if (tail != TI::EPV) {
    // the one slot that owns the last vector (a wave-uniform test), and in
    // it the one lane that holds it
    const uint32_t vt = nvec - 1;
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
      const uint32_t b = slot_base<NT>(s, nvec);
      if (vt >= b && vt < b + NT && vt >= (uint32_t)(s * NT) && (uint32_t)tid == vt - b)
        x[s] = tail_masked<TI>(x[s], tail);
    }
  }
}

// One vector of a streamed row, with the tail past V read as -inf.
template <class TI>
__device__ __forceinline__ typename TI::Vec load_vec(const void* zrow, uint32_t v, uint32_t nvec,
                                                     int tail) {
  const typename TI::Vec x = ld_cached<TI>(zrow, v);
  return v == nvec - 1 ? tail_masked<TI>(x, tail) : x;
}

// exp(z - m) with nm = -m log2(e): the one expression every pass uses, so a
// value recomputed later is bit-identical to the one summed earlier.
__device__ __forceinline__ float ez(float f, float nm) { return fast_exp2(fmaf(f, kLog2e, nm)); }

template <class TI, int NSLOT>
__device__ __forceinline__ float lane_max(const typename TI::Vec (&x)[NSLOT]) {
  float mx = kNegInf;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    float f[4];
    unpack<TI>(x[s], f);
#pragma unroll
    for (int e = 0; e < 4; ++e) mx = fmaxf(mx, f[e]);
  }
  return mx;
}

template <class TI, int NSLOT>
__device__ __forceinline__ float lane_sumexp(const typename TI::Vec (&x)[NSLOT], float nm) {
  float sm = 0.f;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    float f[4];
    unpack<TI>(x[s], f);
#pragma unroll
    for (int e = 0; e < 4; ++e) sm += ez(f[e], nm);
  }
  return sm;
}

// Sum of exp(z - m) over one vector, added left to right onto acc.
template <class TI>
__device__ __forceinline__ float vec_sumexp(const typename TI::Vec& x, float nm, float acc) {
  float f[4];
  unpack<TI>(x, f);
#pragma unroll
  for (int e = 0; e < 4; ++e) acc += ez(f[e], nm);
  return acc;
}

// Inclusive prefix sum over the 64 lanes of a wavefront (DPP row shifts,
// then the row broadcasts of lanes 15 and 31).
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ uint32_t block_add_u32(uint32_t v, uint32_t* red) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t r = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) r += red[w];
  __syncthreads();
  return r;
}

// ---------------------------------------------------------------- sampling
// Draws by inversion of the index-order CDF of softmax(z) (Sec. 4.1, Stage 1:
// the rollout samples at temperature 1 with no top-p or top-k truncation,
// App. B): draw i is the first index whose cumulative probability exceeds
// u_i.  The CDF is evaluated in double precision, so a draw is the one exact
// arithmetic gives unless u_i lies within about 1e-14 of a cumulative value.
//
// One 256-lane workgroup per row, several per CU; the row is read once.  It
// is cut into at most 2048 chunks of CV = G * 128 consecutive vectors (G * 512
// elements; G = 1 up to V = 1,048,576).  The 16 lanes of one DPP row take one
// chunk in steps of 128 vectors, eight coalesced loads per lane per step
// (each instruction covers 16 consecutive vectors).  A chunk's record is its
// maximum m_q (fp32, exact) and s_q = sum exp(z - m_q) in double.  After the
// row, each record is scaled to the row maximum M (s'_q = s_q f_q, f_q =
// exp(m_q - M)), each thread sums a run of C consecutive chunks, and a block
// scan gives the run prefixes.  One wavefront per draw then finds the run
// (a ballot over the prefixes), the chunk (a wave scan of the run's records)
// and the element (wave scans over the chunk in index order, two vectors per
// lane, with the very terms the record summed).  Where rounding leaves no
// crossing at a level, the nearest entry of nonzero mass is taken, so a drawn
// id always has positive probability.
constexpr int kSmpThreads = 256;
constexpr int kSmpLoads = 8;                   // loads per lane per step
constexpr int kSmpStepVecs = 16 * kSmpLoads;   // vectors per DPP-row step (128)
constexpr int kSmpMaxChunks = 2048;            // records per row

// exp(z - m) in double for a logit z <= m, table-driven (Tang, ACM TOMS
// 15(2), 1989): d = z - m (exact in double) = (n / 512) ln 2 + r with |r|
// at most about ln 2 / 1024, exp(d) = 2^(n >> 9) 2^((n & 511) / 512) exp(r),
// and exp(r) by a cubic: the interpolant of exp at the four Chebyshev nodes
// of [-1.002 ln 2 / 1024, 1.002 ln 2 / 1024], computed in 50-digit decimal
// arithmetic and rounded to double (within 1.2e-15 relative of exp there).
// d is first raised to at least -2000, which keeps the reduction in range
// (-inf and far negative terms come out as 0).  n = round(d 512 / ln 2)
// comes from one fused multiply-add onto 1.5 * 2^52, whose low word is then
// n and whose value less 1.5 * 2^52 is n as a double; ln 2 / 512 is split in
// the Cody-Waite way (the high part's 32 significant bits make n times it
// exact for |n| < 2^21).  2^(n >> 9) is applied by ldexp, which rounds
// through double's gradual underflow (a term below about 4.9e-324 of the
// chunk max is 0).  The clamp also turns a NaN d into 0: NaN logits and
// infinite maxima are caught by the chunk max instead (chunk_record), whose
// record is then NaN, and so the row undefined.
constexpr int kExpTab = 512;
constexpr int kExpTabBits = 9;
constexpr double kDeadArg = -2000.0;
constexpr double kInvStep = 738.6598609351493;             // 512 / ln 2
constexpr double kShift52 = 6755399441055744.0;            // 1.5 * 2^52
constexpr double kStepHi = 6.93147180369123816490e-01 / kExpTab;
constexpr double kStepLo = 1.90821492927058770002e-10 / kExpTab;
constexpr double kQ3 = 0.16666667050025266, kQ2 = 0.50000001916793,
                 kQ1 = 0.9999999999999998, kQ0 = 0.9999999999999989;

template <int T, int MAXC>
struct SmpLds {
  double s[MAXC];       // chunk sum at its max; then at the row max
  float m[MAXC];        // chunk max
  double p[T];          // inclusive prefix of the runs
  double tab[kExpTab];  // 2^(j / 512)
  double wt[T / 64];
  float red[T / 64];
};

// (c2 is kQ2, passed in a vector register: one instruction cannot read two
// scalar constants, and a register the caller holds is not re-materialised
// per call)
__device__ __forceinline__ double exp_reduced(double d, const double* tab, double c2) {
  d = fmax(d, kDeadArg);
  const double xs = fma(d, kInvStep, kShift52);
  const double nd = xs - kShift52;
  const int n = (int)(uint32_t)__builtin_bit_cast(uint64_t, xs);
  double r = fma(-nd, kStepHi, d);
  r = fma(-nd, kStepLo, r);
  double p = fma(r, kQ3, c2);
  p = fma(p, r, kQ1);
  p = fma(p, r, kQ0);
  return ldexp(tab[n & (kExpTab - 1)] * p, n >> kExpTabBits);
}

// kQ2 in a vector register (see exp_reduced)
__device__ __forceinline__ double c2_reg() {
  double c = kQ2;
  asm volatile("" : "+v"(c));
  return c;
}

// The term for one fp32 logit z against the chunk max (md, in double).  The
// single expression both the chunk records and the draws use, so the draws
// recompute bit for bit the terms the records summed.
__device__ __forceinline__ double term(float z, double md, const double* tab, double c2) {
  return exp_reduced((double)z - md, tab, c2);
}

// exp(x) for one double x <= 0 (the row-max scale of a chunk record)
__device__ __forceinline__ double exp_neg(double x, const double* tab) {
  return exp_reduced(x, tab, c2_reg());
}

// max that propagates NaN (IEEE 754-2019 maximum; v_maximum3_f32 on gfx950)
__device__ __forceinline__ float max_nan(float a, float b) {
  return __builtin_elementwise_maximum(a, b);
}
__device__ __forceinline__ float max3_nan(float a, float b, float c) {
  return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c);
}

// max over the 16 lanes of a DPP row, in every lane of the row (NaN if any
// lane holds NaN)
__device__ __forceinline__ float row16_max(float x) {
  x = max_nan(x, dpp_move<0x140>(x));  // row_mirror
  x = max_nan(x, dpp_move<0x141>(x));  // row_half_mirror
  x = max_nan(x, dpp_move<0xB1>(x));   // quad_perm [1,0,3,2]
  x = max_nan(x, dpp_move<0x4E>(x));   // quad_perm [2,3,0,1]
  return x;
}
// a double moved across lanes by one DPP pattern (both halves)
template <int CTRL>
__device__ __forceinline__ double dpp_move_f64(double v) {
  u32x2 h = __builtin_bit_cast(u32x2, v);
  h[0] = (uint32_t)__builtin_amdgcn_mov_dpp((int)h[0], CTRL, 0xF, 0xF, false);
  h[1] = (uint32_t)__builtin_amdgcn_mov_dpp((int)h[1], CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, h);
}
// sum over the 16 lanes of a DPP row, in every lane of the row: the same
// four patterns as row16_max; each step adds two values that every lane of a
// pair holds in swapped order, so all 16 lanes end with the same sum
__device__ __forceinline__ double row16_sum(double x) {
  x += dpp_move_f64<0x140>(x);  // row_mirror
  x += dpp_move_f64<0x141>(x);  // row_half_mirror
  x += dpp_move_f64<0xB1>(x);   // quad_perm [1,0,3,2]
  x += dpp_move_f64<0x4E>(x);   // quad_perm [2,3,0,1]
  return x;
}
// inclusive prefix sum over the 64 lanes of a wavefront, in double: row shifts
// by 1, 2, 4 and 8 within each 16 lanes, then lanes 15 and 31 onto the rows
// after them (lanes without a source add 0)
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_from_f64(double v) {
  u32x2 h = __builtin_bit_cast(u32x2, v);
  h[0] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h[0], CTRL, ROWS, 0xF, false);
  h[1] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h[1], CTRL, ROWS, 0xF, false);
  return __builtin_bit_cast(double, h);
}
__device__ __forceinline__ double wave_incl_scan_f64(double x) {
  x += dpp_from_f64<0x111, 0xF>(x);  // row_shr:1
  x += dpp_from_f64<0x112, 0xF>(x);  // row_shr:2
  x += dpp_from_f64<0x114, 0xF>(x);  // row_shr:4
  x += dpp_from_f64<0x118, 0xF>(x);  // row_shr:8
  x += dpp_from_f64<0x142, 0xA>(x);  // row_bcast:15 to rows 1 and 3
  x += dpp_from_f64<0x143, 0xC>(x);  // row_bcast:31 to rows 2 and 3
  return x;
}
// a double of one lane, the same in every lane (lane: wave-uniform)
__device__ __forceinline__ double from_lane(double v, int lane) {
  u32x2 h = __builtin_bit_cast(u32x2, v);
  h[0] = (uint32_t)__builtin_amdgcn_readlane((int)h[0], lane);
  h[1] = (uint32_t)__builtin_amdgcn_readlane((int)h[1], lane);
  return __builtin_bit_cast(double, h);
}

__device__ __forceinline__ int first_lane(uint64_t b) { return b ? __ffsll((long long)b) - 1 : -1; }
__device__ __forceinline__ int last_lane(uint64_t b) { return b ? 63 - __clzll((long long)b) : -1; }

enum Pick : int { kCross = 0, kFirst = 1, kLast = 2 };

// First (or last) chunk in [lo, hi) with positive mass, by wave ballots; -1 if none.
__device__ __forceinline__ int64_t chunk_positive(const double* s, int64_t lo, int64_t hi,
                                                  bool last) {
  const int lane = threadIdx.x & 63;
  if (!last) {
    for (int64_t b = lo; b < hi; b += 64) {
      const int64_t q = b + lane;
      const int f = first_lane(__ballot(q < hi && s[q] > 0.0));
      if (f >= 0) return b + f;
    }
  } else {
    for (int64_t b = hi; b > lo; b -= 64) {
      const int64_t q = b - 64 + lane;
      const int l = last_lane(__ballot(q >= lo && q < b && s[q] > 0.0));
      if (l >= 0) return b - 64 + l;
    }
  }
  return -1;
}

// The terms of a row whose records are kept at their chunk's maximum: exp(z -
// m_q), to be scaled by f_q = exp(m_q - M).
struct ExpTerms {
  const float* m;     // chunk maxima
  const double* tab;  // 2^(j / 512)
  double Md;          // row maximum
  struct Chunk {
    double md, scale, c2;
  };
  __device__ __forceinline__ Chunk chunk(int64_t q) const {
    const double mq = (double)m[q];
    return Chunk{mq, exp_neg(mq - Md, tab), c2_reg()};
  }
  __device__ __forceinline__ double operator()(float z, const Chunk& k) const {
    return term(z, k.md, tab, k.c2);
  }
  // the record s of chunk q at the row maximum (a NaN record stays NaN: the
  // row has no distribution)
  __device__ __forceinline__ double record(int64_t q, double s) const {
    return m[q] == kNegInf ? 0.0 : s * exp_neg((double)m[q] - Md, tab);
  }
};

// This lane's two vectors of the 128-vector step that starts at vector v0, and
// their eight terms (vectors at or past the chunk end c1 give 0).
template <class TI>
__device__ __forceinline__ void step_load(const void* zrow, uint32_t v0, uint32_t c1,
                                          uint32_t nvec, int tail, typename TI::Vec (&x)[2]) {
  const uint32_t v = v0 + 2u * (uint32_t)(threadIdx.x & 63);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    x[h] = neg_inf_vec<TI>();
    if (v + h < c1) x[h] = load_vec<TI>(zrow, v + h, nvec, tail);
  }
}
template <class TI, class Terms>
__device__ __forceinline__ void step_terms(const typename TI::Vec (&x)[2], uint32_t v0,
                                           uint32_t c1, const Terms& terms,
                                           const typename Terms::Chunk& ck, double (&w)[8]) {
  const uint32_t v = v0 + 2u * (uint32_t)(threadIdx.x & 63);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float f[4];
    unpack<TI>(x[h], f);
#pragma unroll
    for (int e = 0; e < 4; ++e) w[4 * h + e] = v + h < c1 ? terms(f[e], ck) : 0.0;
  }
}

// Where a draw falls: chunk q and what is left of t there, in the row's scale.
// pick says how the element is found: the crossing, or, where rounding left no
// crossing, the first or last element of mass.  (All wave-uniform.)
struct DrawAt {
  int64_t q;
  double r;
  int pick;
};
template <int T, class Lds>
__device__ __forceinline__ DrawAt smp_locate(const Lds& c, uint32_t nchunk, uint32_t C, double t,
                                             double S) {
  constexpr int PL = T / 64;  // run prefixes per lane
  const int lane = threadIdx.x & 63;
  DrawAt d{-1, 0.0, kLast};
  if (t < S) {
    // run: the first i with p[i] > t (each lane looks at PL entries)
    int li = -1;
#pragma unroll
    for (int k = PL - 1; k >= 0; --k)
      if (c.p[PL * lane + k] > t) li = PL * lane + k;
    const int fl = first_lane(__ballot(li >= 0));
    const int i = __builtin_amdgcn_readlane(li, fl < 0 ? 0 : fl);  // fl >= 0: p[T - 1] = S > t
    d.r = fmax(t - (i ? c.p[i - 1] : 0.0), 0.0);
    if (C == 1 && c.s[i] > 0.0) {  // a run is one chunk
      d.q = i;
      d.pick = kCross;
      return d;
    }
    // chunk within the run (C <= 8 chunks, one per lane)
    const uint32_t r0 = min((uint32_t)i * C, nchunk), r1 = min(r0 + C, nchunk);
    const uint32_t qq = r0 + (uint32_t)lane;
    const double sq = qq < r1 ? c.s[qq] : 0.0;
    const double incl = wave_incl_scan_f64(sq);
    const int cl = first_lane(__ballot(qq < r1 && incl > d.r));
    if (cl >= 0) {
      const double before = cl > 0 ? from_lane(incl, cl - 1) : 0.0;
      d.q = r0 + cl;
      d.r = fmax(d.r - before, 0.0);
      d.pick = kCross;
    } else {
      const int ll = last_lane(__ballot(qq < r1 && sq > 0.0));
      if (ll >= 0) {
        d.q = r0 + ll;
      } else {
        d.q = chunk_positive(c.s, r1, nchunk, false);
        d.pick = kFirst;
        if (d.q < 0) {
          d.q = chunk_positive(c.s, 0, r0, true);
          d.pick = kLast;
        }
      }
    }
  } else {
    d.q = chunk_positive(c.s, 0, nchunk, true);
  }
  return d;
}

// The element of a 128-vector step at which the mass acc (of the chunk's
// earlier steps, unscaled) plus the step's, times fq, first exceeds r: its
// offset in the step, -2 if rounding hides it in its lane, -1 if the step ends
// below r (acc is then the mass so far).
__device__ __forceinline__ int step_crossing(const double (&w)[8], double r, double fq,
                                             double& acc) {
  double lsum = 0.0;
#pragma unroll
  for (int e = 0; e < 8; ++e) lsum += w[e];
  const double incl = acc + wave_incl_scan_f64(lsum);
  const int vl = first_lane(__ballot(incl * fq > r));
  if (vl < 0) {
    acc = from_lane(incl, 63);
    return -1;
  }
  double cum = vl > 0 ? from_lane(incl, vl - 1) : acc;
  int ec = -1;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    cum += w[e];
    if (ec < 0 && cum * fq > r) ec = e;
  }
  const int el = __builtin_amdgcn_readlane(ec, vl);
  return el >= 0 ? 8 * vl + el : -2;
}

// The element of a draw (wave-uniform): the first whose cumulative mass
// exceeds t = u * S.
template <class TI, class Terms>
__device__ __forceinline__ int64_t smp_element(DrawAt d, const Terms& terms, const void* zrow, uint32_t nvec,
                               int tail, uint32_t CV) {
  if (d.q < 0) return -1;  // no chunk of positive mass (excluded by S > 0)
  // element within chunk q, in steps of 128 vectors: lane l holds vectors
  // 2l and 2l + 1 of the step (elements 8l .. 8l + 7, in index order)
  const typename Terms::Chunk ck = terms.chunk(d.q);
  const uint32_t c0 = (uint32_t)d.q * CV, c1 = min(c0 + CV, nvec);
  if (d.pick == kCross) {
    double acc = 0.0;  // unscaled mass of the earlier steps
    for (uint32_t v0 = c0; v0 < c1; v0 += kSmpStepVecs) {
      typename TI::Vec x[2];
      double w[8];
      step_load<TI>(zrow, v0, c1, nvec, tail, x);
      step_terms<TI>(x, v0, c1, terms, ck, w);
      const int at = step_crossing(w, d.r, ck.scale, acc);
      if (at >= 0) return (int64_t)v0 * 4 + at;
      if (at == -2) break;
    }
    d.pick = kLast;  // rounding left no crossing: the last entry of mass
  }
  // first (or last) element of positive mass in the chunk
  const bool last = d.pick == kLast;
  const uint32_t nsteps = (c1 - c0 + kSmpStepVecs - 1) / kSmpStepVecs;
  for (uint32_t k = 0; k < nsteps; ++k) {
    const uint32_t v0 = c0 + (last ? nsteps - 1 - k : k) * kSmpStepVecs;
    typename TI::Vec x[2];
    double w[8];
    step_load<TI>(zrow, v0, c1, nvec, tail, x);
    step_terms<TI>(x, v0, c1, terms, ck, w);
    int ef = -1, eb = -1;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (w[e] > 0.0) {
        if (ef < 0) ef = e;
        eb = e;
      }
    const int vl = last ? last_lane(__ballot(eb >= 0)) : first_lane(__ballot(ef >= 0));
    if (vl >= 0) return ((int64_t)v0 + 2 * vl) * 4 + __builtin_amdgcn_readlane(last ? eb : ef, vl);
  }
  return -1;
}

// The chunk pass of one DPP row over chunk q (vectors [q CV, q CV + CV)): the
// chunk max and the double sum of exp(z - max), in every lane of the row.
// WIDE (more than one step per chunk) takes a max pass and a term pass over
// the chunk; otherwise the step's eight vectors stay in registers, loaded
// through one buffer resource that starts at the wave's first chunk qw
// (wave-uniform): the lane offset is fixed and each load's step an
// immediate.  A q past the last chunk gives the record (-inf, 0).
template <class TI, bool WIDE>
__device__ __forceinline__ void chunk_record(const void* zrow, uint32_t q, uint32_t qw,
                                             uint32_t CV, uint32_t nvec, int tail,
                                             const double* tab, float& mq_out, double& sq_out) {
  typedef typename TI::Vec Vec;
  constexpr int R = kSmpLoads;
  const uint32_t rl = threadIdx.x & 15;
  const bool ragged = tail != TI::EPV;
  const uint32_t c0 = q * CV, c1 = min(c0 + CV, nvec);
  Vec x[R];
  // (unused when WIDE)
  const uint32_t wv = (uint32_t)__builtin_amdgcn_readfirstlane((int)(qw * CV));
  const Rsrc wr = slot_rsrc(zrow, nvec * (uint32_t)sizeof(Vec), wv * (uint32_t)sizeof(Vec));
  uint32_t loff = (c0 - wv + rl) * (uint32_t)sizeof(Vec);
  asm("" : "+v"(loff));  // (kept whole, so each load's step is its immediate offset)
  // all R loads are issued before any is used; lanes past the chunk, and
  // elements past V, then become -inf through per-dword selects
  auto load_step = [&](uint32_t s0) {
#pragma unroll
    for (int b = 0; b < R; ++b) {
      if constexpr (WIDE) {
        x[b] = ld_cached<TI>(zrow, min(s0 + rl + 16u * b, nvec - 1));
      } else {
        // (s0 is c0 here; lanes past the row read zeros, replaced below)
        x[b] = buf_ld<TI, kAuxNt>(wr, loff + 16u * (uint32_t)sizeof(Vec) * b);
      }
    }
    // (a step wholly inside the chunk and clear of a ragged last vector
    // needs no selects)
    if (!(s0 + kSmpStepVecs <= c1 && !(ragged && s0 + kSmpStepVecs >= nvec))) {
#pragma unroll
      for (int b = 0; b < R; ++b) {
        const uint32_t v = s0 + rl + 16u * b;
        const Vec t = tail_masked<TI>(x[b], tail);
        const Vec n = neg_inf_vec<TI>();
        const bool out = v >= c1, last = ragged && v == nvec - 1;
#pragma unroll
        for (int d = 0; d < (int)(sizeof(Vec) / 4); ++d)
          x[b][d] = out ? n[d] : (last ? t[d] : x[b][d]);
      }
    }
  };
  // (the max propagates NaN; a NaN or +inf chunk max makes the record NaN:
  // the row then has no distribution)
  auto step_max = [&]() {
    float lm = kNegInf;
#pragma unroll
    for (int b = 0; b < R; ++b) {
      float f[4];
      unpack<TI>(x[b], f);
      lm = max3_nan(max3_nan(lm, f[0], f[1]), f[2], f[3]);
    }
    return lm;
  };
  const double c2 = c2_reg();
  auto step_sum = [&](double md, double acc) {
#pragma unroll
    for (int b = 0; b < R; ++b) {
      float f[4];
      unpack<TI>(x[b], f);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc += term(f[e], md, tab, c2);
    }
    return acc;
  };
  float lm = kNegInf;
  if constexpr (!WIDE) {
    load_step(c0);
    lm = step_max();
  } else {
    for (uint32_t s0 = c0; s0 < c1; s0 += kSmpStepVecs) {
      load_step(s0);
      lm = max_nan(lm, step_max());
    }
  }
  const float mq = row16_max(lm);
  double ls = 0.0;
  if (mq != kNegInf) {  // an all -inf chunk has no mass
    const double md = (double)mq;
    if constexpr (!WIDE) {
      ls = step_sum(md, 0.0);
    } else {
      for (uint32_t s0 = c0; s0 < c1; s0 += kSmpStepVecs) {
        load_step(s0);
        ls = step_sum(md, ls);
      }
    }
  }
  const double sum = row16_sum(ls);
  mq_out = mq;
  sq_out = mq < __builtin_huge_valf() ? sum : __builtin_nan("");  // NaN or +inf max: NaN
}

// The outputs of a masked row (tid of T lanes).
template <int T>
__device__ __forceinline__ void sample_masked_row(const CacheArgs& a, int64_t row) {
  const int M = a.K;
  for (int i = threadIdx.x; i < M; i += T) {
    a.ids_out[row * M + i] = 0;
    if (a.logp) a.logp[row * M + i] = 0.f;
  }
  if (threadIdx.x == 0 && a.lse_out) a.lse_out[row] = 0.f;
}

// From the records of a row (visible to the workgroup) to its draws.  Md is
// the maximum that the terms are relative to.
template <class TI, int T, class Terms, class Lds>
__device__ __forceinline__ void sample_finish(const CacheArgs& a, int64_t row, const void* zrow,
                                              Lds& c, const Terms& terms, uint32_t CV,
                                              uint32_t nchunk, double Md) {
  constexpr int W = T / 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = a.K;
  const uint32_t nvec = (uint32_t)a.nvec;
  // wave w takes draws w, w + W, ... (at most 64: OPD_K_MAX / W), whose
  // uniforms are requested here, ahead of their use
  static_assert(kKMax <= 64 * W, "a wave's draws fit its lanes");
  const int mine = w + lane * W;
  const float my_u = mine < M ? a.u[row * M + mine] : 0.f;
  // records at the row max; runs of C consecutive chunks per thread
  const uint32_t C = (nchunk + T - 1) / T;
  {
    const uint32_t r0 = min((uint32_t)tid * C, nchunk), r1 = min(r0 + C, nchunk);
    double run = 0.0;
    for (uint32_t q = r0; q < r1; ++q) {
      const double sq = terms.record(q, c.s[q]);
      c.s[q] = sq;
      run += sq;
    }
    const double incl = wave_incl_scan_f64(run);
    if (lane == 63) c.wt[w] = incl;
    __syncthreads();
    double before = 0.0;
    for (int k = 0; k < w; ++k) before += c.wt[k];
    c.p[tid] = before + incl;
  }
  double S = 0.0;
#pragma unroll
  for (int k = 0; k < W; ++k) S += c.wt[k];  // equals p[T - 1] bit for bit
  __syncthreads();

  const double L = Md + log(S);
  if (tid == 0 && a.lse_out) a.lse_out[row] = (float)L;
  // a NaN or +inf logit, or a row of -inf, leaves S NaN or 0: no distribution
  const bool defined = S > 0.0 && S <= 1.7976931348623157e308;
  // one draw per wavefront at a time, the next one's chunk located and on its
  // way meanwhile; lane k keeps the wave's k-th draw
  int32_t my_id = -1;
  typename TI::Vec x[2], nx[2];
  auto locate = [&](int k, typename TI::Vec (&v)[2]) {
    DrawAt d{-1, 0.0, kLast};
    const float u = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_u), k));
    if (w + k * W < M && defined && u >= 0.f && u < 1.f)
      d = smp_locate<T>(c, nchunk, C, (double)u * S, S);
    if (d.q >= 0) {
      const uint32_t c0 = (uint32_t)d.q * CV;
      step_load<TI>(zrow, c0, min(c0 + CV, nvec), nvec, a.tail, v);
    }
    return d;
  };
  DrawAt d = locate(0, x);
#pragma unroll 1
  for (int k = 0; w + k * W < M; ++k) {
    DrawAt nd{-1, 0.0, kLast};
    if (k < 63) nd = locate(k + 1, nx);
    if (d.q >= 0) {
      int64_t id = -1;
      const uint32_t c0 = (uint32_t)d.q * CV;
      if (d.pick == kCross && CV == kSmpStepVecs) {
        const typename Terms::Chunk ck = terms.chunk(d.q);
        double wt[8], acc = 0.0;
        step_terms<TI>(x, c0, min(c0 + CV, nvec), terms, ck, wt);
        const int at = step_crossing(wt, d.r, ck.scale, acc);
        if (at >= 0) id = (int64_t)c0 * 4 + at;
      }
      if (id < 0) id = smp_element<TI>(d, terms, zrow, nvec, a.tail, CV);
      if (lane == k) my_id = (int32_t)id;
    }
    d = nd;
    x[0] = nx[0];
    x[1] = nx[1];
  }
  if (mine < M) {
    a.ids_out[row * M + mine] = my_id;
    if (a.logp)
      a.logp[row * M + mine] =
          my_id >= 0 ? (float)((double)load_elem<TI>(zrow, my_id) - L) : __builtin_nanf("");
  }
}

// One row by T lanes, from the double-precision exponential (c.tab is set).
template <class TI, bool WIDE, int T, int MAXC>
__device__ __forceinline__ void sample_row(const CacheArgs& a, int64_t row, const void* zrow,
                                           SmpLds<T, MAXC>& c) {
  constexpr int W = T / 64;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t nvec = (uint32_t)a.nvec;
  const uint32_t steps = (nvec + kSmpStepVecs - 1) / kSmpStepVecs;
  const uint32_t G = WIDE ? (steps + MAXC - 1) / MAXC : 1;  // steps per chunk
  const uint32_t CV = G * kSmpStepVecs;
  const uint32_t nchunk = (nvec + CV - 1) / CV;  // <= MAXC

  // one pass over the row: DPP row k of wave w takes chunks 4 w + k,
  // 4 w + k + 4 W, ...
  const uint32_t rowk = (uint32_t)lane >> 4, rl = (uint32_t)lane & 15;
  float lmax = kNegInf;
  for (uint32_t q0 = 4u * w; q0 < nchunk; q0 += 4u * W) {  // wave-uniform
    const uint32_t q = q0 + rowk;
    float mq;
    double sq;
    chunk_record<TI, WIDE>(zrow, q, q0, CV, nvec, a.tail, c.tab, mq, sq);
    if (rl == 15 && q < nchunk) {
      c.m[q] = mq;
      c.s[q] = sq;
    }
    if (q < nchunk) lmax = max_nan(lmax, mq);
  }
  const float Mx = block_max<W>(lmax, c.red);  // ends with a barrier: records visible
  const double Md = (double)Mx;
  sample_finish<TI, T>(a, row, zrow, c, ExpTerms{c.m, c.tab, Md}, CV, nchunk, Md);
}

template <class TI, bool WIDE>
__global__ void __launch_bounds__(kSmpThreads) k_sample(CacheArgs a) {
  __shared__ SmpLds<kSmpThreads, kSmpMaxChunks> c;
  const int64_t row = xcd_remap(blockIdx.x, gridDim.x);
  if (a.mask && a.mask[row] == 0) {
    sample_masked_row<kSmpThreads>(a, row);
    return;
  }
  for (int j = threadIdx.x; j < kExpTab; j += kSmpThreads) c.tab[j] = exp2((double)j / kExpTab);
  __syncthreads();
  sample_row<TI, WIDE>(a, row, (const char*)a.logits + row * a.ld * TI::BYTES, c);
}

// ---------------------------------------------------------------- draws of bf16 rows
// A bf16 logit has few values: those of magnitude [2^-17, 640), both signs, are
// 6,720.  k_sample_tab keeps exp(z) of each, in double, in LDS, so the term of an
// element is one LDS read, and the pass over the row one integer sequence and
// one double addition per element where the exponential takes sixteen
// double-precision instructions; and the terms exp(z), not exp(z - max), need no
// maximum.  The entries are within about 3.4e-16 relative (exp_reduced:
// 1.5e-15).  A tile that holds a value outside [2^-17, 352) classes its elements
// by their offsets, two to an instruction: logits below -820 (-inf among them) read
// the entry past the table, 0; zeros are counted; other magnitudes below 2^-17
// take exp's series.  A row with any other value ([640, inf), [-820, -640]), or
// whose sum is below exp(-60), is marked for k_sample_redo; one with a NaN or
// +inf has no distribution.  In the rows that stay the maximum is above -74 (the
// sum is at most V exp(max)), so a logit below -820 is 0 in double's exp(z - max)
// as well.  Where all magnitudes are below 352 no term that is not 0 would
// underflow there either; in the other ("far") rows one may, which can matter to
// a uniform of 0 only (any other is at least 2^-149 of the sum), so a far row that
// has one is marked too.
// Measured at 4,096 rows of V = 151,936, 16 draws each, against k_sample for every
// row: a tenth of the entries -inf 296 / 460 us, nine tenths 260 / 403, a tenth zeros
// 354 / 414, one entry of 400 in every row 217 / 435, one of NaN 195 / 388; but one of
// 700 in every row (both kernels read it) 600 / 430, and every entry below 2^-17
// and not 0 597 / 401.
//
// One 1,024-lane workgroup per CU stays for all its rows, so the table is set
// up once, and its 16 waves take work from one queue: for each row its tiles
// (four chunks, 2,048 elements), then the draws of the row before it, four to
// an item.  No wave waits for another's phase: rows stream while the last
// one's draws wait for memory.  Records and prefixes of the rows under way lie
// in a ring of slots.  A wave only ever waits for items before its own in the
// queue (a draw for its row's tiles, a tile for the draws of the row that held
// its slot), all of them held by running waves, so every wait ends.
// Bound by HBM and LDS together: 220 us at 4,096 rows of V = 151,936, 16 draws each
// (5.7 TB/s; a plain read of the rows takes 183), of which LDS bank
// conflicts take about a third, against 430-450 us for k_sample, and 258 us with
// a workgroup, and a table, per row; 256 rows 29.4 / 53.4, 2,048 rows of V = 20,000
// 42.3 / 65.6.  (The draws of chunks with unusual values are found one by one
// after the others, and the sums keep to the registers left: four copies of
// the former, or an element's rare term beside each read, spill into the stream.)
constexpr int kTabThreads = 1024;
constexpr int kTabRing = 2560;                  // records in the ring
constexpr int kTabMaxSlots = 8;
constexpr int kTabMaxChunks = kTabRing / 2;     // rows up to 655,360 entries
constexpr int kTabCus = 256;
// Draws per item.  Two cost 16 draws of 4,096 rows 229 against 219 us, 64 draws of
// 2,048 rows of V = 20,000 99 / 85 (256 rows 26.9 / 28.7); eight spill, 228 / 214 and
// 256 rows 36.0 / 28.7 (64 draws 300 / 318).
constexpr int kTabDraws = 4;
constexpr uint32_t kTabLoExp = 110;             // biased exponent of 2^-17
constexpr uint32_t kTabBase = kTabLoExp << 7;   // bf16 magnitude bits of 2^-17
constexpr uint32_t kTabEnd = 0x4420;            // of 640
constexpr uint32_t kTabFar = 0x43B0;            // and of 352
constexpr uint32_t kTabSize = 2 * (kTabEnd - kTabBase);
constexpr uint32_t kTabNear = 2 * (kTabFar - kTabBase);  // the fast path's entries
constexpr uint32_t kTabBinades = (kTabSize + 255) / 256;
static_assert(kTabSize % 32 == 0, "the table ends with a whole set of low factors");
static_assert((kTabSize + 1) * 8 <= 65536, "a table offset in bytes has 16 bits");
constexpr double kTabMinSum = 8.75651076269652e-27;  // exp(-60)
// ids_out[row * M] of a row left to k_sample_redo
constexpr int32_t kSampleRedo = -2;

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

struct TabLds {
  // exp(z), z's magnitude and sign bit (rotated to the lowest) as index; then 0
  double e[kTabSize + 2];
  union {
    struct {
      double s[kTabRing];  // chunk sums
      double p[kTabRing];  // their inclusive prefix
    };
    double lo[kTabBinades * 32];  // the table's low factors, while it is set up
  };
  uint32_t next;                   // the queue: the next item
  uint32_t done[kTabMaxSlots];     // tiles summed of the row in a slot
  uint32_t drawn[kTabMaxSlots];    // draw items ended in a slot, over all its rows
  uint32_t ready[kTabMaxSlots];    // 1 + the row whose prefix a slot holds
  uint32_t kind[kTabMaxSlots];     // kTabKinds (1 + the last unusual row of a slot) + its kind
};

// Sets up the table with one exponential for every five entries: a magnitude is
// (1 + h / 8 + l / 128) 2^x, so exp(z) is the entry at l = 0 times exp(+-l 2^(x
// - 7)).  Ends with a barrier.
__device__ __forceinline__ void tab_setup(TabLds& t) {
  constexpr uint32_t T = kTabThreads, kHi = kTabSize / 16, kLo = kTabBinades * 32;
  if (threadIdx.x < 2) t.e[kTabSize + threadIdx.x] = 0.0;
  for (uint32_t j = threadIdx.x; j < kHi + kLo; j += T) {
    const bool high = j < kHi;
    // the high entries by (binade, h, sign), the low factors by (binade, l, sign)
    const uint32_t i = high ? j : j - kHi, sign = i & 1u;
    const uint32_t x = high ? i >> 4 : i >> 5;
    const uint32_t bits = ((x + kTabLoExp) << 7) | (high ? ((i >> 1) & 7u) << 4 : 0u);
    const float m = __uint_as_float(bits << 16);  // 2^x for a low factor
    const double z = high ? (double)m : (double)m * ((double)((i >> 1) & 15u) / 128.0);
    const double v = exp(sign ? -z : z);
    if (high)
      t.e[(x << 8) | (((i >> 1) & 7u) << 5) | sign] = v;
    else
      t.lo[i] = v;
  }
  __syncthreads();
  for (uint32_t j = threadIdx.x; j < kTabSize; j += T) {
    const uint32_t l = (j >> 1) & 15u;
    if (l != 0u) t.e[j] = t.e[j & ~30u] * t.lo[((j >> 8) << 5) | (j & 31u)];
  }
  __syncthreads();
}

// Table offsets (in elements) of the two logits in a dword; kTabSize or more
// for a value that the table does not hold.  (Kept opaque, so that the range
// check and the reads share one copy.)
__device__ __forceinline__ u16x2 tab_index(uint32_t x) {
  const u16x2 h = __builtin_bit_cast(u16x2, x);
  uint32_t t = __builtin_bit_cast(
      uint32_t, (u16x2)(h * (uint16_t)2 + ((h >> 15) - (uint16_t)(2 * kTabBase))));
  asm("" : "+v"(t));
  return __builtin_bit_cast(u16x2, t);
}

// The logit of a table offset, and the offset of -inf.
__device__ __forceinline__ float tab_logit(uint32_t t) {
  const uint32_t r = t + 2 * kTabBase;  // (16 bits of it)
  return __uint_as_float(((r >> 1) & 0x7FFFu) << 16 | (r & 1u) << 31);
}
constexpr uint32_t kTabZeroAt = (2 * 0x7F80u + 1 - 2 * kTabBase) & 0xFFFFu;
// The first offset of a logit below -820, and the first of a magnitude below
// the table.
constexpr uint32_t kTabZeroFrom = 2 * (0x444Du + 1 - kTabBase) + 1;
constexpr uint32_t kTabTinyAt = 2 * (0x8000u - kTabBase);

// What a row's values make of it; of several the last counts.
enum TabKind : uint32_t { kTabUsual, kTabFarRow, kTabMarked, kTabUndef, kTabKinds };

// A pair of 16-bit constants, made where it is used: held in scalar registers
// across the kernel's loop they would push others out.
__device__ __forceinline__ u16x2 pair_of(uint32_t x) {
  return __builtin_bit_cast(u16x2, fresh_s(x * 0x10001u));
}
// Two offsets, those of the logits below -820 replaced by 0: the odd ones in
// [kTabZeroFrom, kTabZeroAt].  (Packed 16-bit operations.)
struct TabRare {
  u16x2 first = pair_of(kTabZeroFrom), n = pair_of(kTabZeroAt + 1 - kTabZeroFrom), one = pair_of(1);
  __device__ __forceinline__ u16x2 operator()(u16x2 t) const {
    const u16x2 past = __builtin_elementwise_sub_sat(n, (u16x2)(t - first));  // 0: outside
    const u16x2 zero = t & __builtin_elementwise_min(past, one);  // 1: odd, inside
    return t & (zero - one);
  }
};

// The term of such an offset past the near entries that the table does not hold
// (0 otherwise), and the row's kind as far as is known.  (By what the table
// holds, not by bounds of its own: a value is in the table, 0 in double, below
// the table, or one that no row that stays holds.)
__device__ __forceinline__ double tab_rare_term(uint32_t t, uint32_t& kind) {
  double w = 0.0;
  if (t >= kTabNear) {
    const float z = tab_logit(t);
    if (t >= kTabTinyAt) {
      const double d = (double)z;
      // the next term of the series, z^3 / 6, is below 7.5e-17
      w = fma(d, fma(d, 0.5, 1.0), 1.0);
    } else {
      kind = max(kind, (uint32_t)(t < kTabSize ? kTabFarRow
                                  : z < __builtin_huge_valf() ? kTabMarked : kTabUndef));
    }
  }
  return w;
}

// The larger of a kind and a wave's (wave-uniform).
__device__ __forceinline__ uint32_t tab_raise(uint32_t kind, uint32_t lane_kind) {
  for (uint32_t k = kTabUndef; k > kind; --k)
    if (__ballot(lane_kind == k) != 0) return k;
  return kind;
}

struct TabTerms {
  const double* e;
  struct Chunk {
    double scale;
  };
  __device__ __forceinline__ Chunk chunk(int64_t) const { return Chunk{1.0}; }
  __device__ __forceinline__ double operator()(float z, const Chunk&) const {
    const uint32_t b = __float_as_uint(z) >> 16;
    const uint32_t t = (((b << 1) | (b >> 15)) - 2 * kTabBase) & 0xFFFFu;
    uint32_t kind = kTabUsual;
    return e[min(t, kTabSize)] + (t >= kTabTinyAt ? tab_rare_term(t, kind) : 0.0);
  }
};

// The terms of two vectors per lane, if the table holds those of the whole
// wavefront or they are 0 (vectors outside the chunk read as -inf).
__device__ __forceinline__ bool tab_terms(const InBf16::Vec (&x)[2], const double* e,
                                          double (&w)[8]) {
  u16x2 t[4], top = {0, 0};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    t[k] = tab_index(x[k / 2][k & 1]);
    top = __builtin_elementwise_max(top, t[k]);
  }
  if (__ballot(top[0] >= kTabSize || top[1] >= kTabSize) != 0) {
    const TabRare rare;
    const u16x2 size = pair_of(kTabSize);
    top = (u16x2){0, 0};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      top = __builtin_elementwise_max(top, rare(t[k]));
      t[k] = __builtin_elementwise_min(t[k], size);
    }
    if (__ballot(top[0] >= kTabSize || top[1] >= kTabSize) != 0) return false;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    w[2 * k] = e[t[k][0]];
    w[2 * k + 1] = e[t[k][1]];
  }
  return true;
}

// LDS words that waves of the workgroup pass work by.  A wave's LDS operations
// complete in order; the fences keep the compiler to that order and wait for
// LDS only, so loads from memory stay in flight.
__device__ __forceinline__ uint32_t lds_peek(const uint32_t* p) {
  const uint32_t v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ void lds_release() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
}
__device__ __forceinline__ void lds_acquire() {
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// one addition per wave; the value before it
__device__ __forceinline__ uint32_t lds_count(uint32_t* p) {
  uint32_t v = 0;
  if ((threadIdx.x & 63) == 0)
    v = __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ void lds_post(uint32_t* p, uint32_t v) {
  if ((threadIdx.x & 63) == 0)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_raise(uint32_t* p, uint32_t v) {
  if ((threadIdx.x & 63) == 0)
    __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// (waits for a value, or for a count to reach one)
__device__ __forceinline__ void lds_wait(const uint32_t* p, uint32_t v) {
  while ((int32_t)(lds_peek(p) - v) < 0) __builtin_amdgcn_s_sleep(1);
}

__global__ void __launch_bounds__(kTabThreads) k_sample_tab(CacheArgs a) {
  typedef InBf16 TI;
  typedef TI::Vec Vec;
  constexpr int R = kSmpLoads;
  __shared__ TabLds sh;
  const int lane = threadIdx.x & 63;
  const uint32_t rowk = (uint32_t)lane >> 4, rl = (uint32_t)lane & 15;
  const uint32_t nvec = (uint32_t)a.nvec, N = (uint32_t)a.N, M = (uint32_t)a.K;
  const uint32_t nchunk = (nvec + kSmpStepVecs - 1) / kSmpStepVecs;  // <= kTabMaxChunks
  // tiles of four chunks; one that holds the row's end or a ragged last vector
  // takes the path of unusual values
  constexpr uint32_t TILE = 4 * kSmpStepVecs;
  const uint32_t nclean = a.tail == TI::EPV ? nvec : nvec - 1;
  const uint32_t ntile = (nvec + TILE - 1) / TILE, ndraw = (M + kTabDraws - 1) / kTabDraws;
  const uint32_t slots = min((uint32_t)kTabMaxSlots, (uint32_t)kTabRing / nchunk);  // >= 2
  // the workgroup's rows are b, b + G, ...; block j of its queue holds the
  // tiles of its row j and the draws of its row j - 1
  const uint32_t G = gridDim.x, b0 = blockIdx.x;
  const uint32_t rows = (N - b0 + G - 1) / G, per = ntile + ndraw, items = (rows + 1) * per;
  const uint32_t magic = 0xFFFFFFFFu / per + 1;  // i / per = mulhi(i, magic) for i per < 2^32

  for (int i = threadIdx.x; i < 1 + 4 * kTabMaxSlots; i += kTabThreads) (&sh.next)[i] = 0u;
  tab_setup(sh);

  // (blocks of 64 rows to each XCD, as xcd_remap, with constant divisors)
  auto row_of = [&](uint32_t j) -> int64_t {
    const uint32_t i = b0 + j * G, q = i >> 3;
    if (i >= (N & ~511u)) return (int64_t)i;
    return (int64_t)(((q >> 6) << 9) + ((i & 7u) << 6) + (q & 63u));
  };
  auto row_ptr = [&](int64_t row) { return (const char*)a.logits + row * a.ld * TI::BYTES; };
  auto valid = [&](int64_t row) { return !a.mask || a.mask[row] != 0; };

  // The draws [4 k, 4 k + 4) of the workgroup's row j.
  auto draws = [&](uint32_t j, uint32_t k) __attribute__((always_inline)) {
    const uint32_t slot = j % slots, base = slot * nchunk;
    const int64_t row = row_of(j);
    const uint32_t m = k * kTabDraws + (uint32_t)lane;  // this lane's draw
    const bool mine = lane < kTabDraws && m < M;
    int32_t id = 0;
    float lp = 0.f;
    if (!valid(row)) {
      if (k == 0 && lane == 0 && a.lse_out) a.lse_out[row] = 0.f;
      // (a slot's draw items are counted in the order of its rows)
      lds_wait(&sh.drawn[slot], j / slots * ndraw);
    } else {
      const char* zrow = row_ptr(row);
      const float u = mine ? a.u[row * M + m] : -1.f;
      lds_wait(&sh.ready[slot], j + 1);
      lds_acquire();
      const double* s = sh.s + base;
      const double* p = sh.p + base;
      const double S = p[nchunk - 1];
      const uint32_t seen = lds_peek(&sh.kind[slot]), own = kTabKinds * (j + 1);
      const bool undef = seen == own + kTabUndef;
      bool redo = !undef && (seen == own + kTabMarked || !(S >= kTabMinSum));
      if (seen == own + kTabFarRow) {  // (every item of the row decides alike)
        bool zero = false;
        for (uint32_t i = lane; i < M; i += 64) zero |= a.u[row * M + i] == 0.f;
        redo |= __ballot(zero) != 0;
      }
      if (redo || undef) {
        if (redo && k == 0 && lane == 0) a.ids_out[row * M] = kSampleRedo;
        lds_release();
        lds_count(&sh.drawn[slot]);
        if (undef) {
          if (k == 0 && lane == 0 && a.lse_out) a.lse_out[row] = __builtin_nanf("");
          if (mine) {
            a.ids_out[row * M + m] = -1;
            if (a.logp) a.logp[row * M + m] = __builtin_nanf("");
          }
        }
        return;
      }
      const double L = log(S);
      if (k == 0 && lane == 0 && a.lse_out) a.lse_out[row] = (float)L;
      // each lane's chunk: p[lo - 1] <= t < p[hi] throughout, so a crossing is
      // found even where rounding leaves p short of monotone
      const bool ok = u >= 0.f && u < 1.f;
      const double t = (double)u * S;
      uint32_t lo = 0, hi = nchunk - 1;
      while (__ballot(lo < hi) != 0) {
        const uint32_t mid = (lo + hi) >> 1;
        if (p[mid] > t) hi = mid;
        else if (lo < hi) lo = mid + 1;
      }
      // (t < S, as u <= 1 - 2^-24)
      const double r = fmax(t - (lo ? p[lo - 1] : 0.0), 0.0);
      id = -1;
      // the chunks of the item's draws, all on their way together
      Vec x[kTabDraws][2];
#pragma unroll
      for (int d = 0; d < kTabDraws; ++d) {
        const uint32_t c0 = (uint32_t)__builtin_amdgcn_readlane((int)lo, d) * kSmpStepVecs;
        step_load<TI>(zrow, c0, min(c0 + kSmpStepVecs, nvec), nvec, a.tail, x[d]);
      }
      const uint64_t oks = __ballot(ok);
      uint32_t left = 0;
#pragma unroll
      for (int d = 0; d < kTabDraws; ++d) {
        if (((oks >> d) & 1ull) == 0) continue;
        const uint32_t c0 = (uint32_t)__builtin_amdgcn_readlane((int)lo, d) * kSmpStepVecs;
        double w[8], acc = 0.0;
        int at = -1;
        if (tab_terms(x[d], sh.e, w)) at = step_crossing(w, from_lane(r, d), 1.0, acc);
        if (at < 0) left |= 1u << d;
        else if (lane == d) id = (int32_t)(c0 * 4 + (uint32_t)at);
      }
      // chunks with unusual values, and those where rounding left no crossing: the
      // chunk's last entry of mass then, or that of the nearest chunk that has any
#pragma unroll 1
      while (left != 0) {
        const int d = __builtin_ctz(left);
        left &= left - 1u;
        DrawAt da{__builtin_amdgcn_readlane((int)lo, d), from_lane(r, d), kCross};
        if (!(s[da.q] > 0.0)) {
          const int64_t q = da.q;
          da.q = chunk_positive(s, q + 1, nchunk, false);
          da.pick = kFirst;
          if (da.q < 0) {
            da.q = chunk_positive(s, 0, q, true);
            da.pick = kLast;
          }
        }
        const int64_t j_id = smp_element<TI>(da, TabTerms{sh.e}, zrow, nvec, a.tail, kSmpStepVecs);
        if (lane == d) id = (int32_t)j_id;
      }
      lp = mine && id >= 0 ? (float)((double)load_elem<TI>(zrow, id) - L) : __builtin_nanf("");
      lds_release();
    }
    lds_count(&sh.drawn[slot]);
    if (mine) {
      a.ids_out[row * M + m] = id;
      if (a.logp) a.logp[row * M + m] = lp;
    }
  };

  const uint32_t loff = (rowk * kSmpStepVecs + rl) * (uint32_t)sizeof(Vec);
  Vec x[R];
  bool have = false;        // a tile is in x (or on its way there)
  uint32_t tj = 0, tk = 0;  // its row and its place there
#pragma unroll 1
  for (;;) {
    u16x2 t[2 * R], top = {0, 0};
    if (have) {
#pragma unroll
      for (int i = 0; i < 2 * R; ++i) {
        t[i] = tab_index(x[i / 2][i & 1]);
        top = __builtin_elementwise_max(top, t[i]);
      }
    }
    // the next item; a tile's loads are issued before the current one is
    // summed, and take its registers.  (Draws are left until it has been: they
    // may wait for it.)
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t item = lds_count(&sh.next);
    const uint32_t nj = __umulhi(item, magic), nk = item - nj * per;
    const bool end = item >= items, draw = !end && nk >= ntile && nj > 0;
    const bool tile = !end && nk < ntile && nj < rows && valid(row_of(nj));
    if (tile) {
      const Rsrc r = slot_rsrc(row_ptr(row_of(nj)), nvec * (uint32_t)sizeof(Vec),
                               nk * TILE * (uint32_t)sizeof(Vec));
#pragma unroll
      for (int b = 0; b < R; ++b)
        x[b] = buf_ld<TI, kAuxNt>(r, loff + 16u * (uint32_t)sizeof(Vec) * b);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (have) {
      const uint32_t j = tj, k = tk, t0 = k * TILE, slot = j % slots;
      double s0 = 0.0, s1 = 0.0;
      uint32_t kind = kTabUsual;
      if (t0 + TILE > nclean || __ballot(top[0] >= kTabNear || top[1] >= kTabNear) != 0) {
        if (t0 + TILE > nclean) {  // (what is past the row's end reads as -inf)
          const int left = (int)((uint32_t)a.V - 4u * (t0 + fresh_v(rowk * kSmpStepVecs + rl)));
#pragma unroll
          for (int i = 0; i < 2 * R; ++i) {
            const int at = 64 * (i / 2) + 2 * (i & 1);
            if (left <= at) t[i][0] = (uint16_t)kTabZeroAt;
            if (left <= at + 1) t[i][1] = (uint16_t)kTabZeroAt;
          }
        }
        if (__ballot(top[0] >= kTabTinyAt || top[1] >= kTabTinyAt) != 0) {
          // zeros: counted (their terms are 1), then as good as -inf
          const u16x2 tiny = pair_of(kTabTinyAt), none = pair_of(kTabZeroAt), one = pair_of(1);
          u16x2 n = {0, 0};
#pragma unroll
          for (int i = 0; i < 2 * R; ++i) {
            // (1, and then all bits, where an offset is not a zero's)
            const u16x2 not0 = __builtin_elementwise_min((u16x2)((t[i] ^ tiny) >> 1), one);
            const u16x2 keep = 0 - not0;
            n += not0;
            t[i] = (t[i] & keep) | (none & ~keep);
          }
          n = (uint16_t)(2 * R) - n;
          s0 = (double)(uint16_t)(n[0] + n[1]);
        }
        const TabRare rare;
        const u16x2 size = pair_of(kTabSize);
#pragma unroll
        for (int i = 0; i < 2 * R; ++i) {
          const u16x2 r = rare(t[i]);
          if (__ballot(r[0] >= kTabNear || r[1] >= kTabNear) != 0) {
            uint32_t k2 = kTabUsual;
            s0 += tab_rare_term(r[0], k2);
            s1 += tab_rare_term(r[1], k2);
            if (__ballot(k2 != kTabUsual) != 0) kind = tab_raise(kind, k2);
          }
          t[i] = __builtin_elementwise_min(t[i], size);
        }
      }
      // (eight reads in flight: the scheduling barriers keep each batch whole)
#pragma unroll
      for (int h = 0; h < 2 * R; h += 4) {
        double v[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          // offsets in bytes, both in 16 bits
          const uint32_t o = __builtin_bit_cast(uint32_t, (u16x2)(t[h + i] << 3));
          v[2 * i] = *(const double*)((const char*)sh.e + (o & 0xFFFFu));
          v[2 * i + 1] = *(const double*)((const char*)sh.e + (o >> 16));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          s0 += v[2 * i];
          s1 += v[2 * i + 1];
        }
      }
      const double sum = row16_sum(s0 + s1);
      // the slot's last row has been drawn from (see `draws`); until then its
      // mark and its records are still read
      lds_wait(&sh.drawn[slot], j / slots * ndraw);
      if (kind != kTabUsual) lds_raise(&sh.kind[slot], kTabKinds * (j + 1) + kind);
      const uint32_t q = k * 4 + rowk;
      if (rl == 15 && q < nchunk) sh.s[slot * nchunk + q] = sum;
      lds_release();
      if (lds_count(&sh.done[slot]) + 1 == ntile) {
        // the row's last tile: its prefix, runs of C chunks per lane
        lds_acquire();
        const double* s = sh.s + slot * nchunk;
        double* p = sh.p + slot * nchunk;
        const uint32_t C = (nchunk + 63) / 64;
        const uint32_t r0 = min((uint32_t)lane * C, nchunk), r1 = min(r0 + C, nchunk);
        double run = 0.0;
        for (uint32_t i = r0; i < r1; ++i) run += s[i];
        double at = wave_incl_scan_f64(run) - run;
        if (lane == 0) at = 0.0;
        for (uint32_t i = r0; i < r1; ++i) {
          at += s[i];
          p[i] = at;
        }
        lds_post(&sh.done[slot], 0u);  // for the slot's next row, which waits for this one's draws
        lds_release();
        lds_post(&sh.ready[slot], j + 1);
      }
    }
    if (draw) {
      draws(nj - 1, nk - ntile);
      // vmcnt(0): left to the compiler, the loads of a draw that was skipped
      // would be waited for, and the next tile's with them, where their
      // registers are used again in the sums
      __builtin_amdgcn_s_waitcnt(0x0F70);
    }
    if (end) break;
    have = tile;
    tj = nj;
    tk = nk;
  }
}

// The rows that k_sample_tab left, a workgroup each, five to a CU as in k_sample;
// the usual case, none, costs a grid of workgroups that read a mark and end.
// (One workgroup taking several rows would hold 161 registers, three to a CU.)
__global__ void __launch_bounds__(kSmpThreads) k_sample_redo(CacheArgs a) {
  __shared__ SmpLds<kSmpThreads, kSmpMaxChunks> c;
  const int64_t row = xcd_remap(blockIdx.x, gridDim.x);
  // (a masked row's ids are 0; every lane has read the mark before one overwrites
  // it: sample_row has barriers)
  if (a.ids_out[row * a.K] != kSampleRedo) return;
  for (int j = threadIdx.x; j < kExpTab; j += kSmpThreads) c.tab[j] = exp2((double)j / kExpTab);
  __syncthreads();
  sample_row<InBf16, false>(a, row, (const char*)a.logits + row * a.ld * InBf16::BYTES, c);
}

// ---------------------------------------------------------------- top-k

// Sort key: the IEEE-754 total order of the fp32 bits (bf16 widened), with
// -0 taken as +0.  Larger key = larger value.
__device__ __forceinline__ uint32_t order_key(uint32_t bits) {
  bits = bits == 0x80000000u ? 0u : bits;
  return (bits & 0x80000000u) ? ~bits : (bits | 0x80000000u);
}
__device__ __forceinline__ float key_value(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

__device__ __forceinline__ uint32_t shfl_xor_u32(uint32_t v, int m) {
  return (uint32_t)__shfl_xor((int)v, m, 64);
}
__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  const uint32_t lo = shfl_xor_u32((uint32_t)v, m), hi = shfl_xor_u32((uint32_t)(v >> 32), m);
  return ((uint64_t)hi << 32) | lo;
}

// Bitonic sort of one value per lane over the workgroup, descending: lane i
// ends with the i-th largest.  Exchanges within a wavefront use lane
// shuffles; wider ones go through LDS (two buffers, one barrier each).
// Only the first P lanes (P a power of two) take part; the others keep their
// values.
template <class T, int NTH = NT>
__device__ T block_sort_desc(T v, T (*buf)[NTH], int P = NTH) {
  const int tid = threadIdx.x;
  int ping = 0;
#pragma unroll 1
  for (int size = 2; size <= P; size <<= 1) {
#pragma unroll 1
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      T pv;
      if (stride >= 64) {
        buf[ping][tid] = v;
        __syncthreads();
        pv = buf[ping][tid ^ stride];
        ping ^= 1;
      } else if constexpr (sizeof(T) == 8) {
        pv = shfl_xor_u64(v, stride);
      } else {
        pv = shfl_xor_u32(v, stride);
      }
      const bool take_max = ((tid & size) == 0) == ((tid & stride) == 0);
      v = take_max ? (v > pv ? v : pv) : (v < pv ? v : pv);
    }
  }
  return v;
}

// Bitonic sort of one value per lane within a wavefront, descending.
__device__ __forceinline__ uint32_t wave_sort_desc(uint32_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int size = 2; size <= 64; size <<= 1) {
#pragma unroll
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      const uint32_t pv = shfl_xor_u32(v, stride);
      const bool take_max = ((lane & size) == 0) == ((lane & stride) == 0);
      v = take_max ? max(v, pv) : min(v, pv);
    }
  }
  return v;
}

// Bitonic sort, descending, of P entries held in LDS (P a power of two).
__device__ void lds_sort_desc(uint64_t* s, uint32_t P) {
  for (uint32_t size = 2; size <= P; size <<= 1) {
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (uint32_t i = threadIdx.x; i < P / 2; i += NT) {
        const uint32_t lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
        const uint64_t x = s[lo], y = s[hi];
        if ((lo & size) == 0 ? x < y : x > y) {
          s[lo] = y;
          s[hi] = x;
        }
      }
      __syncthreads();
    }
  }
}

struct TopkLds {
  uint64_t sbuf[2][NT];
  uint64_t cand[kTopkCand];
  uint32_t cnt;
  uint32_t wbound[NW];
  uint32_t ured[NW];
  float red[NW];
  Stats st[NW];
};

// Calls f(key, j) for every element j of the row this lane holds (the
// resident slots, or a streamed pass).  The resident registers pass through
// an empty barrier first, so keys are recomputed in each pass rather than
// kept live from an earlier one.
template <class TI, int NSLOT, class F>
__device__ __forceinline__ void each_key(typename TI::Vec (&x)[NSLOT > 0 ? NSLOT : 1],
                                         const void* zrow, uint32_t nvec, int64_t V, int tail,
                                         int tid, F&& f) {
  const uint32_t V32 = (uint32_t)V;
  if constexpr (NSLOT > 0) {
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) keep_packed(x[s]);
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
      const uint32_t b = slot_base<NT>(s, nvec);
      if ((uint32_t)(s * NT + NT) <= nvec || slot_owns<NT>(s, b, tid, nvec)) {
        const uint32_t v = b + (uint32_t)tid;
        float fv[4];
        unpack<TI>(x[s], fv);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t j = v * 4u + (uint32_t)e;
          if (tail == TI::EPV || j < V32) f(order_key(__float_as_uint(fv[e])), j);
        }
      }
    }
  } else {
    for (uint32_t v = tid; v < nvec; v += NT) {
      float fv[4];
      unpack<TI>(ld_cached<TI>(zrow, v), fv);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t j = v * 4u + (uint32_t)e;
        if (j < V32) f(order_key(__float_as_uint(fv[e])), j);
      }
    }
  }
}

// One row (every return below is workgroup-uniform).
template <class TI, int NSLOT, bool LSE>
__device__ __forceinline__ void topk_row(const CacheArgs& a, int64_t row, TopkLds& sh) {
  const int tid = threadIdx.x;
  const int k = a.K;
  if (a.mask && a.mask[row] == 0) {
    for (int i = tid; i < k; i += NT) {
      a.ids_out[row * k + i] = 0;
      if (a.logp) a.logp[row * k + i] = 0.f;
    }
    if (tid == 0 && a.lse_out) a.lse_out[row] = 0.f;
    return;
  }
  const void* zrow = (const char*)a.logits + row * a.ld * TI::BYTES;
  const uint32_t nvec = (uint32_t)a.nvec;
  const int64_t V = a.V;
  typename TI::Vec x[NSLOT > 0 ? NSLOT : 1];
  if constexpr (NSLOT > 0) load_row<TI, NSLOT>(zrow, nvec, a.tail, tid, x);

  // Each lane's largest value (NaN ignored), which also starts the
  // log-partition; a lane with no element reports -inf.
  float lmx = kNegInf, L = 0.f;
  if constexpr (NSLOT > 0) {
    lmx = lane_max<TI, NSLOT>(x);
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) keep_packed(x[s]);
    if constexpr (LSE) {
      const float m = block_max<NW>(lmx, sh.red);
      L = m + logf(block_sum<NW>(lane_sumexp<TI, NSLOT>(x, -m * kLog2e), sh.red));
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) keep_packed(x[s]);
    }
  } else {
    if constexpr (LSE) {
      Stats st = stats_empty();
      for (uint32_t v = tid; v < nvec; v += NT) {
        const typename TI::Vec xv = load_vec<TI>(zrow, v, nvec, a.tail);
        stats_add<TI, false>(st, xv, xv);
      }
      lmx = st.mz;
      st = block_merge<false, NW>(st, sh.st);
      L = st.mz + logf(st.sz);
    } else {
      for (uint32_t v = tid; v < nvec; v += NT) {
        float f[4];
        unpack<TI>(load_vec<TI>(zrow, v, nvec, a.tail), f);
#pragma unroll
        for (int e = 0; e < 4; ++e) lmx = fmaxf(lmx, f[e]);
      }
    }
  }

  // A lower bound on the k-th largest key: in every wave, r = ceil(k / 16)
  // lanes hold a value at least that wave's r-th largest lane maximum, so
  // 16 r >= k elements are at least the smallest of those 16 values.  A lane
  // whose maximum overstates its elements (none, or only NaN) can only
  // lower the bound to -inf or below, where every element is collected.
  {
    const uint32_t lkey = (uint32_t)tid < nvec ? order_key(__float_as_uint(lmx)) : 0u;
    const uint32_t srt = wave_sort_desc(lkey);
    const int r = (k + NW - 1) / NW;
    const uint32_t wb = (uint32_t)__shfl((int)srt, r - 1, 64);
    if ((tid & 63) == 0) sh.wbound[tid >> 6] = wb;
    if (tid == 0) sh.cnt = 0u;
  }
  __syncthreads();
  uint32_t bound = sh.wbound[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) bound = min(bound, sh.wbound[w]);
  // Candidates: every element not below the bound's value, and every NaN
  // (!(v < b) holds for both); their exact keys decide the order.
  const float bval = key_value(bound);
  auto take = [&](float v, uint32_t j) {
    if (!(v < bval)) {
      const uint32_t pos = atomicAdd(&sh.cnt, 1u);
      if (pos < (uint32_t)kTopkCand)
        sh.cand[pos] = ((uint64_t)order_key(__float_as_uint(v)) << 32) | (0xFFFFFFFFu - j);
    }
  };
  if constexpr (NSLOT > 0) {
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
      const uint32_t b = slot_base<NT>(s, nvec);
      if ((uint32_t)(s * NT + NT) <= nvec || slot_owns<NT>(s, b, tid, nvec)) {
        const uint32_t v = b + (uint32_t)tid;
        float f[4];
        unpack<TI>(x[s], f);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (a.tail == TI::EPV || v * 4u + e < (uint32_t)V) take(f[e], v * 4u + e);
      }
    }
  } else {
    for (uint32_t v = tid; v < nvec; v += NT) {
      float f[4];
      unpack<TI>(ld_cached<TI>(zrow, v), f);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (v * 4u + e < (uint32_t)V) take(f[e], v * 4u + e);
    }
  }
  __syncthreads();
  const uint32_t cnt = sh.cnt;

  uint64_t mine = 0;  // after sorting: this lane's rank in the support
  if (cnt >= (uint32_t)k && cnt <= (uint32_t)NT) {
    int P = 2;
    while (P < (int)cnt) P <<= 1;
    mine = block_sort_desc<uint64_t>(tid < (int)cnt ? sh.cand[tid] : 0ull, sh.sbuf, P);
  } else if (cnt >= (uint32_t)k && cnt <= (uint32_t)kTopkCand) {
    uint32_t P = NT;
    while (P < cnt) P <<= 1;
    for (uint32_t i = cnt + tid; i < P; i += NT) sh.cand[i] = 0ull;
    __syncthreads();
    lds_sort_desc(sh.cand, P);
    mine = sh.cand[tid];
  } else {
    // Too many candidates (a row with many equal large values): find the
    // k-th largest key th by bisection over key bits, then the need-th
    // lowest index among the elements equal to th, by counting passes.
    // These passes re-read the row from memory (a rare path; compact code).
    typename TI::Vec none[1];
    auto count = [&](auto&& pred) {
      uint32_t n = 0;
      each_key<TI, 0>(none, zrow, nvec, V, a.tail, tid, [&](uint32_t key, uint32_t j) { n += pred(key, j) ? 1u : 0u; });
      return block_add_u32(n, sh.ured);
    };
    uint32_t th = 0;
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t t = th | (1u << bit);
      if (count([&](uint32_t key, uint32_t) { return key >= t; }) >= (uint32_t)k) th = t;
    }
    const uint32_t gt = th == 0xFFFFFFFFu ? 0u : count([&](uint32_t key, uint32_t) { return key > th; });
    const uint32_t need = (uint32_t)k - gt;
    uint32_t y = 0;
    for (int bit = 30; bit >= 0; --bit) {
      const uint32_t t = y | (1u << bit);
      if (count([&](uint32_t key, uint32_t j) { return key == th && j < t; }) < need) y = t;
    }
    if (tid == 0) sh.cnt = 0u;
    __syncthreads();
    each_key<TI, 0>(none, zrow, nvec, V, a.tail, tid, [&](uint32_t key, uint32_t j) {
      if (key > th || (key == th && j <= y)) {
        const uint32_t pos = atomicAdd(&sh.cnt, 1u);
        if (pos < (uint32_t)kTopkCand) sh.cand[pos] = ((uint64_t)key << 32) | (0xFFFFFFFFu - j);
      }
    });
    __syncthreads();
    mine = block_sort_desc<uint64_t>(tid < k ? sh.cand[tid] : 0ull, sh.sbuf);
  }

  if (tid < k) {
    const uint32_t j = 0xFFFFFFFFu - (uint32_t)mine;
    a.ids_out[row * k + tid] = (int32_t)j;
    if (a.logp) a.logp[row * k + tid] = key_value((uint32_t)(mine >> 32)) - L;
  }
  if (tid == 0 && a.lse_out) a.lse_out[row] = L;
}

// The top-k of a row per workgroup (register-resident for NSLOT > 0); and,
// after the streamed kernel, a short grid whose workgroups walk the rows and
// redo only those the streamed kernel marked (reading them from memory), so
// that the usual case, no marked row, costs a few hundred workgroups rather
// than one per row.
constexpr int kTopkRedoGroups = 512;
template <class TI, int NSLOT, bool LSE>
__global__ void __launch_bounds__(NT) k_topk(CacheArgs a) {
  __shared__ TopkLds sh;
  topk_row<TI, NSLOT, LSE>(a, xcd_remap(blockIdx.x, gridDim.x), sh);
}
template <class TI, int NSLOT, bool LSE>
__global__ void __launch_bounds__(NT) k_topk_redo(CacheArgs a) {
  __shared__ TopkLds sh;
  __shared__ uint32_t s_n;
  __shared__ int64_t s_rows[NT];
  const int64_t stride = (int64_t)gridDim.x;
  // the workgroup's rows are blockIdx.x + i * stride; a lane reads one row's
  // mark, so a batch of NT rows costs one round trip, and only the marked
  // rows are redone
  for (int64_t base = blockIdx.x; base < a.N; base += stride * NT) {  // workgroup-uniform
    if (threadIdx.x == 0) s_n = 0u;
    __syncthreads();
    const int64_t row = base + (int64_t)threadIdx.x * stride;
    if (row < a.N && a.ids_out[row * a.K] == kTopkRedo) s_rows[atomicAdd(&s_n, 1u)] = row;
    __syncthreads();
    const uint32_t n = s_n;
    for (uint32_t i = 0; i < n; ++i) {
      topk_row<TI, NSLOT, LSE>(a, s_rows[i], sh);
      __syncthreads();  // the next row's writes to LDS wait for this row's reads
    }
  }
}

// ---------------------------------------------------------------- top-k, streamed

// The top-k support of rows of at least 16,384 entries, for k <= 64, reads
// each row once: 256-lane workgroups with about 34 KiB of LDS, four per CU.
// Each lane keeps the running maximum of the values it has seen.  After each
// tile of 8 coalesced loads per lane, and before any of the tile's elements
// is kept, the wave recomputes the ceil(k / 4)-th largest of its 64 running
// maxima (a radix select over order keys with ballots, 16 key bits for bf16
// rows) and publishes it in LDS; the bound in use is the smallest of the
// four waves' published values (on a wave's first tile, the k-th largest of
// its own maxima), a lower bound on the row's k-th largest, and it only
// rises.  Only lanes whose tile maximum reaches the bound look at the tile
// again, vector by vector, and keep the elements at or above it in their
// own LDS slots: no cross-lane compaction in the stream.  The next tile's
// loads are issued before the current tile is processed.  Since no bound
// exceeded the row's k-th largest key, the slots hold every element at or
// above it; at the end the largest known bound filters them, and a block
// sort of those (at most 256) gives the support.  A row
// whose lane slots overflow (many equal large values), that leaves more
// than 256 candidates, or that holds a NaN is marked, and a second launch
// runs the resident kernel on the marked rows only.
constexpr int kTkThreads = 256;
constexpr int kTkWaves = kTkThreads / 64;
constexpr int kTkLoads = 8;    // vector loads per lane per tile
constexpr int kTkSlots = 16;   // candidate slots per lane (a power of two)
constexpr int kTkMaxK = 64;    // one running maximum per lane bounds k
constexpr int64_t kTkMinVec = 4096;

struct TkLds {
  uint64_t buf[kTkSlots][kTkThreads];  // lane-private candidates: (value bits, ~index)
  uint64_t sel[kTkThreads];            // survivors: (order key, ~index)
  uint32_t theta[kTkWaves];            // published wave bounds (order keys)
  uint32_t nsel;
  uint32_t over;
  Stats st[kTkWaves];
};

// The largest key t (low KEEP bits zero) with at least k of the wave's rk
// >= t: the k-th largest rk, rounded down to the key bits that vary.
template <int LOWBITS>
__device__ __forceinline__ uint32_t wave_kth_key(uint32_t rk, int k) {
  uint32_t t = 0;
#pragma unroll
  for (int bit = 31; bit >= LOWBITS; --bit) {
    const uint32_t c = t | (1u << bit);
    if ((uint32_t)__popcll(__ballot(rk >= c)) >= (uint32_t)k) t = c;
  }
  return t;
}

template <class TI, bool LSE>
__global__ void __launch_bounds__(kTkThreads) k_topk_stream(CacheArgs a) {
  constexpr int T = kTkThreads, W = kTkWaves, B = kTkLoads;
  // bf16 values widened to fp32 have 16 zero low bits, so their order keys
  // vary in the top 16 bits only (a negative value's low key bits are ones,
  // which a threshold with zero low bits still admits)
  constexpr int LOWBITS = TI::BYTES == 2 ? 16 : 0;
  typedef typename TI::Vec Vec;
  __shared__ TkLds sh;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t row = xcd_remap(blockIdx.x, gridDim.x);
  const int k = a.K;  // <= kTkMaxK
  if (a.mask && a.mask[row] == 0) {
    for (int i = tid; i < k; i += T) {
      a.ids_out[row * k + i] = 0;
      if (a.logp) a.logp[row * k + i] = 0.f;
    }
    if (tid == 0 && a.lse_out) a.lse_out[row] = 0.f;
    return;
  }
  if (lane == 0) sh.theta[w] = 0u;
  if (tid == 0) {
    sh.nsel = 0u;
    sh.over = 0u;
  }
  __syncthreads();
  const void* zrow = (const char*)a.logits + row * a.ld * TI::BYTES;
  const uint32_t nvec = (uint32_t)a.nvec;  // >= kTkMinVec: every wave's first tile is full
  const uint32_t V32 = (uint32_t)a.V;
  constexpr uint32_t TILE = 64u * B, STRIDE = W * TILE;
  // tiles wholly inside the row (and clear of a ragged last vector) take
  // the path without per-element checks
  const uint32_t nclean = a.tail == TI::EPV ? nvec : nvec - 1;
  const uint32_t nfull = nclean / TILE * TILE;
  float run = kNegInf;  // this lane's running maximum (NaN ignored)
  // The bound.  Each wave publishes the ceil(k / 4)-th largest of its 64
  // running maxima (as an order key): that many of its lanes have each seen
  // an element at least that large, so the smallest of the four published
  // values has k distinct elements at or above it and is a lower bound on
  // the row's k-th largest.  Published values only rise, so a stale read
  // is still a lower bound.
  const int kq = (k + W - 1) / W;
  uint32_t qown = 0;    // this wave's published value (wave-uniform)
  uint32_t theta = 0;   // the bound in use (wave-uniform)
  bool first = true;    // this wave's first tile
  uint32_t cnt = 0;     // this lane's candidates so far
  float m = kNegInf, sum = 0.f, chk = 0.f;
  uint32_t bare = 0;    // this lane's first tiles that hold -inf and NaN only

  // One tile of B vectors per lane at vector t0 (lane l holds t0 + 64 b + l).
  // Pass A, for every lane: the tile's maximum (and its share of the
  // log-partition); then the bound; then pass B, in the lanes whose tile
  // maximum reaches the bound only, the elements kept.  A NaN anywhere in
  // the row (and, when the log-partition is wanted, a lane that sees no
  // finite value) sends the row to the exact fallback, so the bound and the
  // comparisons here need only order the numbers.
  auto process = [&](const Vec (&x)[B], uint32_t t0, auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    auto vals = [&](int b, float (&f)[4]) {
      unpack<TI>(x[b], f);
      if constexpr (!FULL) {
        const uint32_t v = t0 + 64u * b + lane;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!(v < nvec && v * 4u + e < V32)) f[e] = kNegInf;
      }
    };
    // the tile's maximum; with LSE (registers to spare) each vector's
    // maximum is also kept, so pass B skips vectors below the bound unread
    static_assert(B == 8, "the tile maximum below folds eight vectors");
    float vmx[B];
    float tmx = kNegInf;
#pragma unroll
    for (int b = 0; b < B; ++b) {
      float f[4];
      vals(b, f);
      if constexpr (LSE) {
        vmx[b] = max3_raw(max3_raw(f[0], f[1], f[2]), f[3], f[3]);
      } else {
        tmx = max3_raw(max3_raw(tmx, f[0], f[1]), f[2], f[3]);
        chk += (f[0] + f[1]) + (f[2] + f[3]);
      }
    }
    if constexpr (LSE)
      tmx = max3_raw(max3_raw(vmx[0], vmx[1], vmx[2]), max3_raw(vmx[3], vmx[4], vmx[5]),
                     max3_raw(vmx[6], vmx[7], vmx[7]));
    if constexpr (LSE) {
      const float mn = fmaxf(m, tmx);
      if (mn != kNegInf) {  // (a lane that never sees a finite value sends its row to the fallback)
        const float nm = -mn * kLog2e;
        float ex[B * 4];
#pragma unroll
        for (int b = 0; b < B; ++b) {
          float f[4];
          vals(b, f);
#pragma unroll
          for (int e = 0; e < 4; ++e) ex[4 * b + e] = fast_exp2(fmaf(f[e], kLog2e, nm));
        }
#pragma unroll
        for (int h = B * 2; h >= 1; h >>= 1)
#pragma unroll
          for (int i = 0; i < h; ++i) ex[i] += ex[i + h];
        sum = fmaf(sum, rescale(m, mn), ex[0]);  // NaN from a NaN element
        m = mn;
      } else {
        ++bare;
      }
    }
    run = fmaxf(run, tmx);
    // raise the bound before keeping any of the tile's elements
    const uint32_t rk = order_key(__float_as_uint(run));
    if ((uint32_t)__popcll(__ballot(rk > qown)) >= (uint32_t)kq) {  // wave-uniform
      qown = wave_kth_key<LOWBITS>(rk, kq);
      if (lane == 0) sh.theta[w] = qown;
    }
    if (first) {  // until the other waves have published: the k-th of this wave's maxima
      theta = wave_kth_key<LOWBITS>(rk, k);
      first = false;
    }
    uint32_t pub = sh.theta[0];
#pragma unroll
    for (int q = 1; q < W; ++q) pub = min(pub, sh.theta[q]);
    theta = max(theta, (uint32_t)__builtin_amdgcn_readfirstlane(pub));
    const float thf = key_value(theta);
    // for numbers, f >= thf exactly when order_key(f) >= theta (a bf16
    // bound's zero low key bits sit below every widened value's)
    if (__ballot(tmx >= thf) != 0) {  // wave-uniform
      // the lane's vectors whose maximum reaches the bound, one bit each
      uint32_t rm = 0u;
      if (tmx >= thf) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
          bool reach;
          if constexpr (LSE) {
            reach = vmx[b] >= thf;
          } else {
            Vec xv = x[b];
            keep_packed(xv);  // unpacked again here rather than held since pass A
            float f[4];
            unpack<TI>(xv, f);
            reach = max3_raw(max3_raw(f[0], f[1], f[2]), f[3], f[3]) >= thf;
          }
          rm |= reach ? 1u << b : 0u;
        }
      }
      // One reaching vector per lane per round, in index order within the
      // lane, for as many rounds as the busiest lane needs (usually one):
      // a body per vector position instead would run whenever any lane's
      // vector at that position reaches.
      while (__ballot(rm != 0u) != 0) {  // wave-uniform
        if (rm != 0u) {
          const int b = __builtin_ctz(rm);
          rm &= rm - 1u;
          Vec xv = x[0];
#pragma unroll
          for (int j = 1; j < B; ++j) xv = b == j ? x[j] : xv;
          keep_packed(xv);  // selected packed, then unpacked
          float f[4];
          unpack<TI>(xv, f);
          const uint32_t v = t0 + 64u * (uint32_t)b + lane;
          // each element is written to the lane's next free slot, which
          // only a kept element then claims (a lane that reaches the last
          // slot overflows, and its row goes to the fallback)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool keep = f[e] >= thf && (FULL || (v < nvec && v * 4u + e < V32));
            sh.buf[cnt & (kTkSlots - 1)][tid] =
                ((uint64_t)__float_as_uint(f[e]) << 32) | (0xFFFFFFFFu - (v * 4u + e));
            cnt += keep ? 1u : 0u;
          }
        }
      }
    }
  };
  // full tiles through a buffer resource that starts at the tile (scalar
  // arithmetic): the lane offset is fixed and each load's step an immediate
  const uint32_t loff = (uint32_t)lane * (uint32_t)sizeof(Vec);
  auto load = [&](Vec (&x)[B], uint32_t t0) {
    const uint64_t off = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)t0) * sizeof(Vec);
    const Rsrc r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>((const char*)zrow + off), 0,
                                                     (int)(TILE * sizeof(Vec)), kRsrcWord3);
#pragma unroll
    for (int b = 0; b < B; ++b) {
      if constexpr (TI::BYTES == 2)
        x[b] = __builtin_amdgcn_raw_buffer_load_b64(r, (int)(loff + 64u * sizeof(Vec) * b), 0,
                                                    kAuxNt);
      else
        x[b] = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(loff + 64u * sizeof(Vec) * b), 0,
                                                     kAuxNt);
    }
  };
  typedef std::integral_constant<bool, true> Full;
  typedef std::integral_constant<bool, false> Partial;
  // the wave's full tiles, two buffers: the next tile's loads are in flight
  // while the current one is processed
  Vec xa[B], xb[B];
  uint32_t t0 = (uint32_t)w * TILE;
  if (t0 < nfull) {  // wave-uniform
    load(xa, t0);
    while (t0 + 2 * STRIDE < nfull) {
      load(xb, t0 + STRIDE);
      process(xa, t0, Full());
      load(xa, t0 + 2 * STRIDE);
      process(xb, t0 + STRIDE, Full());
      t0 += 2 * STRIDE;
    }
    if (t0 + STRIDE < nfull) {
      load(xb, t0 + STRIDE);
      process(xa, t0, Full());
      process(xb, t0 + STRIDE, Full());
      t0 += 2 * STRIDE;
    } else {
      process(xa, t0, Full());
      t0 += STRIDE;
    }
  }
  // the one tile that reaches past the clean vectors (the wave whose turn it is)
  if (t0 < nvec) {
#pragma unroll
    for (int b = 0; b < B; ++b) xa[b] = ld_nt<TI>(zrow, min(t0 + 64u * b + lane, nvec - 1));
    process(xa, t0, Partial());
  }
  // the tiles that were not summed, for NaN (usually none; read again here,
  // which keeps the test out of the loop's registers)
  if constexpr (LSE) {
    const uint32_t v0 = (uint32_t)w * TILE + lane;
    for (uint32_t i = 0; i < bare; ++i)
#pragma unroll 1
      for (uint32_t v = v0 + i * STRIDE; v < min(v0 + i * STRIDE + TILE, nvec); v += 64) {
        float f[4];
        unpack<TI>(load_vec<TI>(zrow, v, nvec, a.tail), f);
        sum += (f[0] == f[0] && f[1] == f[1] && f[2] == f[2] && f[3] == f[3])
                   ? 0.f
                   : __builtin_nanf("");
      }
  }
  bool nan_seen;
  if constexpr (LSE) nan_seen = sum != sum || m == kNegInf;
  else nan_seen = chk != chk;
  if (cnt >= (uint32_t)kTkSlots || nan_seen) sh.over = 1u;
  float L = 0.f;
  if constexpr (LSE) {
    Stats st = stats_empty();
    st.mz = m;
    st.sz = sum;
    st = block_merge<false, W>(st, sh.st);  // barriers: bounds and slots visible
    L = st.mz + logf(st.sz);
  } else {
    __syncthreads();
  }
  // every bound in use was at most the row's k-th largest key, so the slots
  // hold every element at or above it; the largest bound known filters them
  uint32_t tstar = sh.theta[0];
#pragma unroll
  for (int q = 1; q < W; ++q) tstar = min(tstar, sh.theta[q]);
  tstar = max(tstar, theta);
  const bool overflow = sh.over != 0u;
  if (!overflow) {
    for (uint32_t i = 0; i < cnt; ++i) {
      const uint64_t e = sh.buf[i][tid];  // (value bits, ~index)
      const uint32_t key = order_key((uint32_t)(e >> 32));
      if (key >= tstar) {
        const uint32_t pos = atomicAdd(&sh.nsel, 1u);
        if (pos < (uint32_t)T) sh.sel[pos] = ((uint64_t)key << 32) | (uint32_t)e;
      }
    }
  }
  __syncthreads();
  const uint32_t nsel = sh.nsel;
  if (overflow || nsel > (uint32_t)T || nsel < (uint32_t)k) {  // workgroup-uniform
    if (tid == 0) a.ids_out[row * k] = kTopkRedo;
    return;
  }
  // Each survivor's rank is the number of survivors above it (the entries
  // are distinct); the k of rank below k are the top k, each written at its
  // rank.  Every lane reads the same entry at a time (an LDS broadcast), and
  // the reads do not depend on each other, unlike the exchanges of a sort.
  if (tid < (int)nsel) {
    const uint64_t mine = sh.sel[tid];
    uint32_t rank = 0;
#pragma unroll 8
    for (uint32_t i = 0; i < nsel; ++i) rank += sh.sel[i] > mine ? 1u : 0u;
    if (rank < (uint32_t)k) {
      const uint32_t j = 0xFFFFFFFFu - (uint32_t)mine;
      a.ids_out[row * k + rank] = (int32_t)j;
      if (a.logp) a.logp[row * k + rank] = key_value((uint32_t)(mine >> 32)) - L;
    }
  }
  if (tid == 0 && a.lse_out) a.lse_out[row] = L;
}

// ---------------------------------------------------------------- scoring

// Scoring reads each row once and writes a handful of values, so it is
// organised for overlap rather than residency: 256-lane workgroups with a
// small register footprint (several per CU), each lane loading batches of
// kScoreBatch vectors and folding them into a running (max, sum-exp) with
// one rescale per batch.
constexpr int kScoreThreads = 256;
constexpr int kScoreBatch = 8;

template <class TI>
__global__ void __launch_bounds__(kScoreThreads) k_score(CacheArgs a) {
  constexpr int T = kScoreThreads, W = T / 64, B = kScoreBatch;
  typedef typename TI::Vec Vec;
  __shared__ Stats s_st[W];
  const int tid = threadIdx.x;
  const int64_t row = xcd_remap(blockIdx.x, gridDim.x);
  const int K = a.K;  // <= OPD_K_MAX == T: one id per lane
  if (a.mask && a.mask[row] == 0) {
    if (tid < K) a.logp[row * K + tid] = 0.f;
    if (tid == 0 && a.lse_out) a.lse_out[row] = 0.f;
    return;
  }
  const void* zrow = (const char*)a.logits + row * a.ld * TI::BYTES;
  const uint32_t nvec = (uint32_t)a.nvec;
  const bool ragged = a.tail != TI::EPV;
  // the ids are requested before the row, so the gather does not wait behind it
  const int32_t id = tid < K ? a.ids[row * K + tid] : 0;
  float m = kNegInf, sum = 0.f;
  for (uint32_t v0 = 0; v0 < nvec; v0 += T * B) {
    Vec xb[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const uint32_t v = v0 + (uint32_t)(b * T + tid);
      xb[b] = ld_nt<TI>(zrow, min(v, nvec - 1));  // clamped: every lane loads
    }
    float f[B][4];
    float bm = kNegInf;
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const uint32_t v = v0 + (uint32_t)(b * T + tid);
      Vec xv = xb[b];
      if (v >= nvec) xv = neg_inf_vec<TI>();
      else if (ragged && v == nvec - 1) xv = tail_masked<TI>(xv, a.tail);
      unpack<TI>(xv, f[b]);
#pragma unroll
      for (int e = 0; e < 4; ++e) bm = fmaxf(bm, f[b][e]);
    }
    // (as stats_add: a block of NaN has no maximum either, and is summed)
    const float mn = fmaxf(m, bm);
    float acc = sum * rescale(m, mn);
    const float nm = mn != kNegInf ? -mn * kLog2e : 0.f;
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc += ez(f[b][e], nm);
    sum = acc;
    m = mn;
  }
  Stats st = stats_empty();
  st.mz = m;
  st.sz = sum;
  st = block_merge<false, W>(st, s_st);
  const float L = st.mz + logf(st.sz);
  if (tid < K) {
    const bool ok = id >= 0 && (int64_t)id < a.V;
    a.logp[row * K + tid] = ok ? load_elem<TI>(zrow, id) - L : __builtin_nanf("");
  }
  if (tid == 0 && a.lse_out) a.lse_out[row] = L;
}

// ---------------------------------------------------------------- dispatch

template <class TI, int NSLOT>
hipError_t launch_op(const CacheArgs& a, CacheOp op, hipStream_t stream) {
  const dim3 grid((unsigned)a.N), block(NT);
  const dim3 rgrid((unsigned)min(a.N, (int64_t)kTopkRedoGroups));
  switch (op) {
    case CacheOp::Sample:
      break;
    case CacheOp::Topk:
      if constexpr (NSLOT == 0) {
        if (a.redo) {
          if (a.logp || a.lse_out)
            hipLaunchKernelGGL((k_topk_redo<TI, 0, true>), rgrid, block, 0, stream, a);
          else
            hipLaunchKernelGGL((k_topk_redo<TI, 0, false>), rgrid, block, 0, stream, a);
          break;
        }
      }
      if (a.logp || a.lse_out) {
        hipLaunchKernelGGL((k_topk<TI, NSLOT, true>), grid, block, 0, stream, a);
      } else {
        hipLaunchKernelGGL((k_topk<TI, NSLOT, false>), grid, block, 0, stream, a);
      }
      break;
    case CacheOp::Score:
      break;
  }
  return hipGetLastError();
}

// Whether bf16 rows are drawn from the table.  Setting it up, and the draws of an
// item one after the other, cost what k_sample's double-precision terms cost on
// few narrow rows with few draws.  Measured, table against k_sample: 64 rows of V =
// 16,384, M = 1 12.1 / 10.2 us, M = 4 1.32 times, M = 8 1.07 times; 24,576 M = 1 1.01, M = 4
// 1.09; 32,000 M = 4 1.04 times; 512 rows of 22,000 M = 1 1.07, M = 4 1.12 times, of 24,576
// 0.91 and 1.02; 1,024 rows of 16,384 (eight whole tiles) M = 1 0.92, of 18,000 1.06, of
// 20,000 0.99; 16 draws 0.97 and less everywhere.
bool draws_from_table(const CacheArgs& a) {
  if (a.nvec < 4096 || a.nvec > (int64_t)kTabMaxChunks * kSmpStepVecs) return false;
  if (a.N <= 256) return a.K > 8 || a.nvec >= (a.K > 4 ? 5600 : 5600 + 1100 * a.K);
  if (a.K > 4 || a.N > 1024) return true;
  return a.N <= 640 ? a.nvec >= 5800 : a.nvec == 4096 || a.nvec >= 5000;
}

template <class TI>
hipError_t launch_dt(const CacheArgs& a, CacheOp op, bool resident, hipStream_t stream) {
  if (op == CacheOp::Sample) {
    if constexpr (TI::BYTES == 2) {
      if (draws_from_table(a)) {
        hipLaunchKernelGGL(k_sample_tab, dim3((unsigned)min(a.N, (int64_t)kTabCus)),
                           dim3(kTabThreads), 0, stream, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_sample_redo, dim3((unsigned)a.N), dim3(kSmpThreads), 0, stream, a);
        return hipGetLastError();
      }
    }
    // more than one 128-vector step per chunk above 2048 steps per row
    if ((a.nvec + kSmpStepVecs - 1) / kSmpStepVecs <= (int64_t)kSmpMaxChunks)
      hipLaunchKernelGGL((k_sample<TI, false>), dim3((unsigned)a.N), dim3(kSmpThreads), 0,
                         stream, a);
    else
      hipLaunchKernelGGL((k_sample<TI, true>), dim3((unsigned)a.N), dim3(kSmpThreads), 0,
                         stream, a);
    return hipGetLastError();
  }
  if (op == CacheOp::Score) {
    hipLaunchKernelGGL((k_score<TI>), dim3((unsigned)a.N), dim3(kScoreThreads), 0, stream, a);
    return hipGetLastError();
  }
  if (op == CacheOp::Topk && a.K <= kTkMaxK && a.nvec >= kTkMinVec) {
    if (a.logp || a.lse_out)
      hipLaunchKernelGGL((k_topk_stream<TI, true>), dim3((unsigned)a.N), dim3(kTkThreads), 0,
                         stream, a);
    else
      hipLaunchKernelGGL((k_topk_stream<TI, false>), dim3((unsigned)a.N), dim3(kTkThreads), 0,
                         stream, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    CacheArgs b = a;
    b.redo = 1;  // the rows the streamed kernel left (rare: re-read, not held in registers)
    return launch_op<TI, 0>(b, op, stream);
  }
  if (!resident) return launch_op<TI, 0>(a, op, stream);
  constexpr int big = TI::BYTES == 2 ? 38 : 19, small = TI::BYTES == 2 ? 16 : 8;
  if (a.nvec <= (int64_t)small * NT) return launch_op<TI, small>(a, op, stream);
  return launch_op<TI, big>(a, op, stream);
}

}  // namespace

hipError_t launch_cache(const CacheArgs& a, CacheOp op, int in_dt, bool resident,
                        hipStream_t stream) {
  if (a.N == 0) return hipSuccess;
  return in_dt == BF16 ? launch_dt<InBf16>(a, op, resident, stream)
                       : launch_dt<InF32>(a, op, resident, stream);
}

}  // namespace opd
