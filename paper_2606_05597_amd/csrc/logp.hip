// Forward only: the sampled action's log-prob and the policy entropy of each
// token row (the proximal log-probs recomputed before an update, Table 5, and
// the per-token entropy of Sec. 5), one workgroup per row.  The same kernels
// also reduce one shard of a vocabulary split over devices to its per-token
// record (max, sum exp, action logit; grpo_vocab_shard_stats).
//
// A row is read once.  Each thread walks its 16-byte vectors U at a time (all U
// loads in flight together) and keeps, relative to its running shift m,
//   s = sum e^(z - m)   and   t = sum e^(z - m) (z - m),
// rescaling both when a chunk raises m.  For any shift m >= max z the row's
// log-sum-exp is m + log s and its entropy -sum p log p = log s - t / s; both
// terms of the entropy are >= 0, so it has no cancellation even when small.
#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>

#include "device.h"
#include "host.h"
#include "launch.h"

namespace grpo {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct LogpArgs {
  const void* logits;
  int64_t ld, V;
  int64_t v_begin;  // global id of column 0 (a shard's first column; 0 otherwise)
  int T;
  const int32_t* actions;
  float* logp;      // nullable
  float* entropy;   // nullable
  int32_t* flags;   // nullable
  grpo_vocab_stats* stats;  // non-null: write each row's shard record instead of logp / entropy
};

// One element folded into (s, t) at the current shift m: s = sum e^(z - m), t = sum e^(z - m) w with
// w = (z - m) log2(e), the argument the exp2 takes anyway (t is in log2 units; row_out converts).  A -inf logit (a
// masked column) has e = 0 and adds no term (0 log 0 = 0): its w = -inf is clamped to -FLT_MAX in the product,
// which is then 0, not NaN.  A NaN logit still makes e, and so s and t, NaN.
// ENT = false: s only (t stays 0), for the calls that want no entropy.
template <bool ENT = true>
__device__ __forceinline__ void fold(float z, float nmb, float& s, float& t) {
  const float w = fmaf(z, kLog2e, nmb);
  const float e = __builtin_amdgcn_exp2f(w);
  s += e;
  if constexpr (ENT) t = fmaf(e, fmaxf(w, -FLT_MAX), t);
}

// Raises the shift m >= kShiftMin to mn: s and t are re-expressed relative to mn.  Where nothing is left of the old sum
// (f = 0) its moment is 0 too: -dl s may then be infinite.
template <bool ENT = true>
__device__ __forceinline__ void rescale(float& m, float mn, float& s, float& t) {
  if (mn > m) {
    const float dl = (mn - m) * kLog2e, f = __builtin_amdgcn_exp2f(-dl);
    if constexpr (ENT) t = f == 0.f ? 0.f : f * fmaf(-dl, s, t);
    s *= f;
    m = mn;
  }
}

// Combines every thread's (m, s, t) into the row's (M, S, T) in fp64, valid in thread 0 (t and T in log2 units):
// within each wave (DPP within rows of 16 lanes, then the four rows), then across the NW <= 16 waves by the first
// 16 lanes of wave 0.  Every lane of the workgroup takes part.
template <int NW>
__device__ __forceinline__ void block_combine3(float m, float s, float t, float* sh_m, double* sh_s, double* sh_t,
                                               double& M_out, double& S_out, double& T_out) {
  static_assert(NW >= 1 && NW <= 16, "one wave partial per lane of a 16-lane row");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const double L = (double)kLog2e;
  const float mw = wave_max_dpp(m);
  const double f = (double)__builtin_amdgcn_exp2f((m - mw) * kLog2e);
  const double sw = wave_sum_dpp(f * (double)s);
  const double tw = wave_sum_dpp(f * ((double)t + ((double)m - (double)mw) * L * (double)s));
  if (lane == 0) {
    sh_m[wv] = mw;
    sh_s[wv] = sw;
    sh_t[wv] = tw;
  }
  __syncthreads();
  if (wv == 0) {
    const float mq = lane < NW ? sh_m[lane] : -INFINITY;
    const float M = row16_max(mq);
    const double g = (mq == -INFINITY) ? 0.0 : exp((double)mq - (double)M);
    const int q = lane < NW ? lane : 0;
    const double S = row16_sum(g * sh_s[q]);
    const double T = row16_sum(mq == -INFINITY ? 0.0 : g * (sh_t[q] + ((double)mq - (double)M) * L * sh_s[q]));
    M_out = (double)M;
    S_out = S;
    T_out = T;
  }
}

// Element e of a 16-byte vector (8 bf16 or 4 fp32), widened to fp32.
template <typename Tin>
__device__ __forceinline__ float elem(const u32x4& x, int e) {
  if constexpr (sizeof(Tin) == 2) {
    const uint32_t w = x[e >> 1];
    return (e & 1) ? bf16_hi(w) : bf16_lo(w);
  } else {
    return __uint_as_float(x[e]);
  }
}

template <typename Tin>
__device__ __forceinline__ void row_out(const LogpArgs& a, int t, double M, double S, double Tsum, double za,
                                        bool act_ok) {
  if (a.stats) {
    grpo_vocab_stats r;
    r.m = (M == (double)kShiftMin && S == 0.0) ? -INFINITY : M;  // the maximum of stored values: exact
    r.s = S;
    r.z_a = act_ok ? za : -INFINITY;
    a.stats[t] = r;
    if (a.flags && (isnan(M) || isnan(S) || M == INFINITY)) atomicOr(a.flags, GRPO_FLAG_NONFINITE);
    return;
  }
  const double lse = M + log(S);
  const bool masked = lse == -INFINITY && za > -INFINITY && za <= (double)kShiftMin;  // throughout, as in token_eval
  if (a.logp) a.logp[t] = !act_ok ? 0.f : masked ? -INFINITY : (float)(za - lse);
  // Tsum is in log2 units: sum e^(z - M) (z - M) = Tsum / log2(e)
  if (a.entropy) a.entropy[t] = (float)(log(S) - Tsum / ((double)kLog2e * S));
  if (a.flags) {
    if (!act_ok) atomicOr(a.flags, GRPO_FLAG_ACTION);
    if (!isfinite(lse)) atomicOr(a.flags, GRPO_FLAG_NONFINITE);
  }
}

// ENT: the entropy moment is accumulated (not for a shard's records or a call without an entropy output).  RAG: rows
// that are not whole aligned vectors (RowSplit); an edge element is folded after its thread's vectors.
template <typename Tin, int NT, int U, bool ENT, bool RAG>
__global__ __launch_bounds__(NT) void k_logp_vec(const LogpArgs a) {
  constexpr int EPV = 16 / sizeof(Tin), NW = NT / 64;
  __shared__ float sh_m[NW];
  __shared__ double sh_s[NW], sh_t[NW];
  __shared__ float sh_za;
  const int t = blockIdx.x, tid = threadIdx.x;
  const Tin* row0 = static_cast<const Tin*>(a.logits) + (int64_t)t * a.ld;
  const RowSplit sp = row_split<Tin, RAG>(row0, a.V);
  const int nvec = sp.nvec;
  const u32x4* row = reinterpret_cast<const u32x4*>(row0 + sp.head);
  const int64_t act64 = (int64_t)a.actions[t] - a.v_begin;
  const bool act_ok = act64 >= 0 && act64 < a.V;
  const int act = act_ok ? (int)act64 : -1;
  int act_lane;
  const int act_vec = vec_of<Tin>(sp, act, act_lane);
  float m = kShiftMin, s = 0.f, tt = 0.f;
  const int ecol = RAG ? edge_col<Tin>(sp, tid) : -1;
  float ez = -INFINITY;
  if (RAG && ecol >= 0) ez = load_elem(row0 + ecol);
  for (int base = tid; base < nvec; base += NT * U) {
    u32x4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int vi = base + u * NT;
      if (vi < nvec) x[u] = __builtin_nontemporal_load(row + vi);
    }
    float cm = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int vi = base + u * NT;
      if (vi < nvec) {
        cm = vec_max<Tin>(x[u], cm);
        if (vi == act_vec) sh_za = elem<Tin>(x[u], act_lane);
      }
    }
    rescale<ENT>(m, cm, s, tt);
    const float nmb = -m * kLog2e;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int vi = base + u * NT;
      if (vi < nvec) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) fold<ENT>(elem<Tin>(x[u], e), nmb, s, tt);
      }
    }
  }
  if (RAG && ecol >= 0) {
    rescale<ENT>(m, fmaxf(m, ez), s, tt);
    fold<ENT>(ez, -m * kLog2e, s, tt);
    if (ecol == act) sh_za = ez;
  }
  double M, S, Tsum;
  block_combine3<NW>(m, s, tt, sh_m, sh_s, sh_t, M, S, Tsum);  // its barrier publishes sh_za
  if (tid == 0) row_out<Tin>(a, t, M, S, Tsum, act_ok ? (double)sh_za : 0.0, act_ok);
}

// ---- loss and dlogits of rows that no kernel holds -------------------------------
struct TwiceArgs {
  const void* logits;
  void* dlogits;
  int64_t ld;
  int T;
  TokenArgs tok;
};

// One workgroup per row of whole aligned vectors: the row's sum as k_logp_vec forms it for a record (the same terms in
// the same order, so that the results are those of the two launches to the bit), the token epilogue, then dlogits.  A
// thread's first HR vectors stay in registers and the next HL in LDS (rows have more than that); the rest is read a
// second time, backwards, the end of the row from the L2 and, at two workgroups per CU, which the registers and the LDS
// are sized for, as much more from the memory-side cache as its 256 MB hold of the rows in flight: 512 rows of up to
// 0.5 MB (131,072 columns) beside what is held, less of longer ones.
// HBM-bound.  fp32 loss and dlogits, in two launches / here: 6,000 x 151,936 2.01 / 1.48 ms (4.9 TB/s of the row read and
// written once), 8,000 x 100,000 1.68 / 1.22, 3,000 x 262,144 1.62 / 1.32, 800 x 1,000,000 1.89 / 1.78, 64 x 151,936
// 0.078 / 0.042; with nothing held 1.60 at 151,936, with more workgroups per CU 1.66 to 2.0.
template <typename Tin, int NT, int U, int HR, int HL>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_rows_twice(const TwiceArgs a) {
  constexpr int EPV = 16 / sizeof(Tin), NW = NT / 64, H = HR + HL;
  static_assert(HR % U == 0 && HL % U == 0, "whole chunks");
  __shared__ u32x4 stage[HL * NT];
  __shared__ float sh_m[NW];
  __shared__ double sh_s[NW], sh_t[NW];
  __shared__ float sh_za;
  __shared__ RowScale sh_rs;
  const int t = blockIdx.x, tid = threadIdx.x;
  const int nvec = (int)(a.tok.V / EPV);
  constexpr int VB = NT * 16;
  const int voff = tid * 16;
  const char* row = reinterpret_cast<const char*>(static_cast<const Tin*>(a.logits) + (int64_t)t * a.ld);
  // a vector of the row; past its end, the last one, which is then left out
  auto at = [&](int vi) { return reinterpret_cast<const u32x4*>(row + (uint32_t)min(vi, nvec - 1) * 16u); };
  const TokenIn in = token_load(a.tok, t);
  const bool act_ok = in.act >= 0 && in.act < a.tok.V;
  const RowSplit sp{0, nvec, 0};
  int act_lane;
  const int act_vec = vec_of<Tin>(sp, act_ok ? in.act : -1, act_lane);
  float m = kShiftMin, s = 0.f, tt = 0.f;
  u32x4 hold[HR], x[U], y[U];
#pragma unroll
  for (int q = 0; q < HR; ++q) 
    hold[q] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(row + q * VB + (uint32_t)voff));
  auto load = [&](u32x4 (&v)[U], int q) {  // vectors q .. q + U - 1 of the thread
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = *at((q + u) * NT + tid);
  };
  auto sum = [&](const u32x4* v, int q, bool whole) {
    const int base = q * NT + tid;
    float cm = -INFINITY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int vi = base + u * NT;
      if (whole || vi < nvec) {
        cm = vec_max<Tin>(v[u], cm);
        if (vi == act_vec) sh_za = elem<Tin>(v[u], act_lane);
      }
    }
    rescale<false>(m, cm, s, tt);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int vi = base + u * NT;
      if (whole || vi < nvec) {
#pragma unroll
        for (int e = 0; e < EPV; ++e) fold<false>(elem<Tin>(v[u], e), -m * kLog2e, s, tt);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  load(x, HR);
#pragma unroll
  for (int q = 0; q < HR; q += U) sum(hold + q, q, true);
#pragma unroll 1
  for (int q = 0; q < HL; q += 2 * U) {  // two chunks in flight, in turn
    load(y, HR + q + U);
#pragma unroll
    for (int u = 0; u < U; ++u) stage[(q + u) * NT + tid] = x[u];
    sum(x, HR + q, true);
    load(x, HR + q + 2 * U);
#pragma unroll
    for (int u = 0; u < U; ++u) stage[(q + U + u) * NT + tid] = y[u];
    sum(y, HR + q + U, true);
  }
  const int nv = (nvec + NT - 1) / NT;
#pragma unroll 1
  for (int q = H; q < nv; q += 2 * U) {
    load(y, q + U);
    sum(x, q, false);
    load(x, q + 2 * U);
    sum(y, q + U, false);
  }
  double M, S, Tsum;
  block_combine3<NW>(m, s, tt, sh_m, sh_s, sh_t, M, S, Tsum);  // its barrier publishes sh_za
  if (tid == 0) {
    if (isnan(M) || isnan(S) || M == INFINITY) atomicOr(&a.tok.hdr->flags, GRPO_FLAG_NONFINITE);
    sh_rs = token_finish(a.tok, t, in, row_lse(M, S), act_ok ? (double)sh_za : 0.0);
  }
  __syncthreads();
  if (!a.dlogits) return;
  const RowScale rs = sh_rs;
  const uint32_t smask = sign_mask<Tin>(rs);
  int act_l;
  const int act_v = vec_of<Tin>(sp, rs.act, act_l);
  const __amdgpu_buffer_rsrc_t dst = row_rsrc(static_cast<Tin*>(a.dlogits) + (int64_t)t * a.ld, nvec * 16);
  auto put = [&](const u32x4& v, int q) {
    __builtin_amdgcn_raw_buffer_store_b128(vec_dlogits<Tin>(v, rs, smask, q * NT + tid == act_v, act_l), dst, voff,
                                           q * VB, kStream);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1" ::: "memory");  // the store has read its data before its registers are reused
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr int U2 = 8;
#pragma unroll 1
  for (int q = H + (nv - H + U2 - 1) / U2 * U2 - U2; q >= H; q -= U2) {
    u32x4 z[U2];
#pragma unroll
    for (int u = 0; u < U2; ++u) z[u] = __builtin_nontemporal_load(at((q + u) * NT + tid));
#pragma unroll
    for (int u = 0; u < U2; ++u) put(z[u], q + u);
  }
#pragma unroll 1
  for (int q = 0; q < HL; ++q) put(stage[q * NT + tid], HR + q);
#pragma unroll
  for (int q = 0; q < HR; ++q) put(hold[q], q);
}

hipError_t launch_rows_twice(const void* logits, void* dlogits, int64_t T, int64_t ld, const TokenArgs& tok,
                             hipStream_t s) {
  const TwiceArgs a{logits, dlogits, ld, (int)T, tok};
  hipLaunchKernelGGL((k_rows_twice<float, 256, 4, 36, 16>), dim3((unsigned)T), dim3(256), 0, s, a);
  return hipGetLastError();
}

__global__ void k_clear_flag(int32_t* f) { *f = 0; }

// Ragged rows of up to 8 KB go to one wave each: a workgroup of four took the log-probs of 20,000 rows of 101 columns in
// 24.4 us (bf16; 22.6 fp32), longer than reading them element by element, one wave 14.1 (12.8); 1,003 columns 27.9 and
// 15.7, 4,001 37.6 and 26.9; fp32 2,003 31.0 and 25.6.
constexpr int64_t kOneWaveBytes = 8192;
typedef void (*LogpKernel)(const LogpArgs);
template <typename Tin, int NT, bool RAG>
static LogpKernel logp_kernel(bool ent) {
  return ent ? k_logp_vec<Tin, NT, 4, true, RAG> : k_logp_vec<Tin, NT, 4, false, RAG>;
}
template <typename Tin>
static void launch_logp_rows(const LogpArgs& a, bool rag, hipStream_t s) {
  const bool ent = a.entropy && !a.stats;
  const bool one_wave = rag && a.V * (int64_t)sizeof(Tin) <= kOneWaveBytes;
  const LogpKernel k = one_wave ? logp_kernel<Tin, 64, true>(ent)
                       : rag    ? logp_kernel<Tin, 256, true>(ent)
                                : logp_kernel<Tin, 256, false>(ent);
  hipLaunchKernelGGL(k, dim3((unsigned)a.T), dim3(one_wave ? 64 : 256), 0, s, a);
}

// One workgroup per row.
static void launch_logp(const LogpArgs& a, grpo_dtype dt, hipStream_t s) {
  const bool rag = row_form(a.logits, nullptr, a.V, a.ld, dt == GRPO_BF16 ? 2 : 4) == RowForm::kRagged;
  if (dt == GRPO_BF16) launch_logp_rows<uint16_t>(a, rag, s);
  else launch_logp_rows<float>(a, rag, s);
}

hipError_t launch_vocab_records(const void* logits, grpo_dtype dt, int64_t T, int64_t V, int64_t ld,
                                int64_t v_begin, const int32_t* actions, grpo_vocab_stats* stats, int32_t* flags,
                                hipStream_t s) {
  if (T > 0) {
    LogpArgs a{logits, ld, V, v_begin, (int)T, actions, nullptr, nullptr, flags, stats};
    launch_logp(a, dt, s);
  }
  return hipGetLastError();
}

}  // namespace grpo

using namespace grpo;

extern "C" int grpo_token_logp(const void* logits, int32_t dtype, int64_t T, int64_t V, int64_t ld,
                               const int32_t* actions, float* token_logp, float* token_entropy, int32_t* error_flags,
                               hipStream_t s) {
  if (T < 0 || T >= ((int64_t)1 << 31) || V < 1 || ld < V) return GRPO_ERR_SHAPE;
  if (T > 0 && (!logits || !actions)) return GRPO_ERR_ARG;
  if (dtype != GRPO_F32 && dtype != GRPO_BF16) return GRPO_ERR_DTYPE;
  const grpo_dtype dt = static_cast<grpo_dtype>(dtype);
  const int esz = (dt == GRPO_BF16) ? 2 : 4;
  if (!aligned(logits, esz)) return GRPO_ERR_ALIGN;
  if (error_flags) hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, s, error_flags);
  if (T > 0) {
    LogpArgs a{logits, ld, V, 0, (int)T, actions, token_logp, token_entropy, error_flags, nullptr};
    launch_logp(a, dt, s);
  }
  return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

extern "C" int grpo_vocab_shard_stats(const void* logits, int32_t dtype, int64_t T, int64_t V_shard, int64_t ld,
                                      int64_t v_begin, const int32_t* actions, grpo_vocab_stats* stats,
                                      int32_t* error_flags, hipStream_t s) {
  constexpr int64_t kLim = (int64_t)1 << 31;  // v_begin + V_shard < 2^31, tested without forming the sum first
  if (T < 0 || T >= kLim || V_shard < 1 || V_shard >= kLim || ld < V_shard || v_begin < 0 ||
      v_begin >= kLim - V_shard)
    return GRPO_ERR_SHAPE;
  if (T > 0 && (!logits || !actions || !stats)) return GRPO_ERR_ARG;
  if (dtype != GRPO_F32 && dtype != GRPO_BF16) return GRPO_ERR_DTYPE;
  const grpo_dtype dt = static_cast<grpo_dtype>(dtype);
  const int esz = (dt == GRPO_BF16) ? 2 : 4;
  if (!aligned(logits, esz) || !aligned(stats, 8)) return GRPO_ERR_ALIGN;
  if (error_flags) hipLaunchKernelGGL(k_clear_flag, dim3(1), dim3(1), 0, s, error_flags);
  if (T > 0) {
    LogpArgs a{logits, ld, V_shard, v_begin, (int)T, actions, nullptr, nullptr, error_flags, stats};
    launch_logp(a, dt, s);
  }
  return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}
