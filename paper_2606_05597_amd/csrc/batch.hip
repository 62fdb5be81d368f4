// Batch bookkeeping kernels: segment validation, group advantages, and the
// deterministic loss reduction.  All are small next to the row pass.
#include <hip/hip_runtime.h>
#include <math.h>

#include "device.h"
#include "launch.h"

namespace grpo {

// ---- segments ----------------------------------------------------------------
// One workgroup.  Checks the CSR offsets of Eq. 1's trajectory/step/token
// sums, writes traj_tok_off[i] = step_tok_off[traj_step_off[i]] and the
// per-trajectory weight w_i = 1/(n_groups * G * |tau_i| or k).
struct SegArgs {
  const int32_t* sto;  // [n_steps+1]
  const int32_t* tso;  // [n_traj+1]
  int32_t n_steps, n_traj, G, norm;
  int64_t T;
  double n_groups, k;
  WsHeader* hdr;
  int32_t* traj_tok_off;  // ws [n_traj+1]
  double* w;              // ws [n_traj]
  int32_t* aux_traj_tok_off;
};

__global__ __launch_bounds__(256) void k_segments(const SegArgs a) {
  const int tid = threadIdx.x;
  int bad = 0;
  for (int j = tid; j < a.n_steps; j += 256)
    if (a.sto[j + 1] < a.sto[j]) bad = 1;
  for (int i = tid; i < a.n_traj; i += 256)
    if (a.tso[i + 1] <= a.tso[i]) bad = 1;
  if (tid == 0) {
    if (a.sto[0] != 0 || (int64_t)a.sto[a.n_steps] != a.T) bad = 1;
    if (a.tso[0] != 0 || a.tso[a.n_traj] != a.n_steps) bad = 1;
  }
  bad = __syncthreads_or(bad);
  for (int i = tid; i <= a.n_traj; i += 256) {
    int off;
    if (i == a.n_traj) {
      off = (int)a.T;
    } else {
      int st = min(max(a.tso[i], 0), a.n_steps);  // clamped: offsets may be malformed
      off = a.sto[st];
      int steps = a.tso[i + 1] - a.tso[i];
      double den = (a.norm == GRPO_NORM_CONST_K) ? a.k : (double)steps;
      a.w[i] = 1.0 / (a.n_groups * (double)a.G * den);
    }
    a.traj_tok_off[i] = off;
    if (a.aux_traj_tok_off) a.aux_traj_tok_off[i] = bad ? -1 : off;
  }
  if (tid == 0) {
    a.hdr->flags = bad ? GRPO_FLAG_OFFSETS : 0;
    a.hdr->done = 0;
    a.hdr->counts[0] = a.hdr->counts[1] = 0;
  }
}

// The trajectory of every token, found by binary search over the trajectory
// starts, and what the token epilogue needs from it (advantage, normaliser
// weight), so that the row passes read per-token values only.  Also the
// optional token outputs that need no logits.  One thread per token.
__global__ __launch_bounds__(256) void k_tok_traj(int64_t T, int32_t n_traj, const int32_t* traj_tok_off,
                                                  const WsHeader* hdr, const int32_t* actions, int64_t ld,
                                                  const float* adv, const double* w, float* tok_adv, double* tok_w,
                                                  int32_t* aux_tok_traj, int64_t* aux_gather) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= T) return;
  const int i = find_traj(traj_tok_off, n_traj, (int)t);
  tok_adv[t] = adv[i];
  tok_w[t] = w[i];
  if (aux_tok_traj) aux_tok_traj[t] = (hdr->flags & GRPO_FLAG_OFFSETS) ? -1 : i;
  if (aux_gather) aux_gather[t] = t * ld + actions[t];
}

// k_segments and k_tok_traj in one launch, for batches whose tables fit one workgroup's LDS: every workgroup of 256
// tokens makes the tables itself (the offsets come from the L2), workgroup 0 writes them out.  A launch and a gap
// less: at T = 30,000 9.7 us before, 5.1 now, and the gap.  Up to kSegTraj trajectories and kSegSteps steps, beyond which the tables cost every workgroup
// more than the launch does.
constexpr int kSegTraj = 1024, kSegSteps = 16384;
struct SegTokArgs {
  SegArgs s;
  const int32_t* actions;
  int64_t ld;
  const float* adv;
  float* tok_adv;
  double* tok_w;
  int32_t* aux_tok_traj;
  int64_t* aux_gather;
};
__global__ __launch_bounds__(256) void k_segments_tok(const SegTokArgs p) {
  __shared__ int sh_off[kSegTraj];
  __shared__ double sh_w[kSegTraj];
  const SegArgs& a = p.s;
  const int tid = threadIdx.x;
  const bool lead = blockIdx.x == 0;
  int bad = 0;
  for (int j = tid; j < a.n_steps; j += 256)
    if (a.sto[j + 1] < a.sto[j]) bad = 1;
  for (int i = tid; i < a.n_traj; i += 256) {
    const int s0 = a.tso[i], s1 = a.tso[i + 1];
    if (s1 <= s0) bad = 1;
    const int off = a.sto[min(max(s0, 0), a.n_steps)];  // clamped: offsets may be malformed
    const double den = (a.norm == GRPO_NORM_CONST_K) ? a.k : (double)(s1 - s0);
    const double w = 1.0 / (a.n_groups * (double)a.G * den);
    sh_off[i] = off;
    sh_w[i] = w;
    if (lead) {
      a.traj_tok_off[i] = off;
      a.w[i] = w;
    }
  }
  if (tid == 0) {
    if (a.sto[0] != 0 || (int64_t)a.sto[a.n_steps] != a.T) bad = 1;
    if (a.tso[0] != 0 || a.tso[a.n_traj] != a.n_steps) bad = 1;
  }
  bad = __syncthreads_or(bad);
  if (lead) {
    if (a.aux_traj_tok_off) {
      for (int i = tid; i < a.n_traj; i += 256) a.aux_traj_tok_off[i] = bad ? -1 : sh_off[i];
      if (tid == 0) a.aux_traj_tok_off[a.n_traj] = bad ? -1 : (int)a.T;
    }
    if (tid == 0) {
      a.traj_tok_off[a.n_traj] = (int)a.T;
      a.hdr->flags = bad ? GRPO_FLAG_OFFSETS : 0;
      a.hdr->done = 0;
      a.hdr->counts[0] = a.hdr->counts[1] = 0;
    }
  }
  const int64_t t = (int64_t)blockIdx.x * 256 + tid;
  if (t >= a.T) return;
  const int i = find_traj(sh_off, a.n_traj, (int)t);
  p.tok_adv[t] = p.adv[i];
  p.tok_w[t] = sh_w[i];
  if (p.aux_tok_traj) p.aux_tok_traj[t] = bad ? -1 : i;
  if (p.aux_gather) p.aux_gather[t] = t * p.ld + p.actions[t];
}

hipError_t launch_segments(const grpo_segments* seg, int64_t T, int64_t ld, const int32_t* actions,
                           const float* adv, const grpo_loss_params* p, char* ws, const LossWs& L,
                           const grpo_aux* aux, hipStream_t s) {
  int32_t* aux_traj_tok_off = aux ? aux->traj_tok_off : nullptr;
  SegArgs a;
  a.sto = seg->step_tok_off;
  a.tso = seg->traj_step_off;
  a.n_steps = seg->n_steps;
  a.n_traj = seg->n_traj;
  a.G = seg->group_size;
  a.norm = p->norm;
  a.T = T;
  a.n_groups = n_groups_of(seg, p);
  a.k = (double)p->k;
  a.hdr = reinterpret_cast<WsHeader*>(ws + L.hdr);
  a.traj_tok_off = reinterpret_cast<int32_t*>(ws + L.traj_tok_off);
  a.w = reinterpret_cast<double*>(ws + L.w);
  a.aux_traj_tok_off = aux_traj_tok_off;
  if (a.n_traj <= kSegTraj && a.n_steps <= kSegSteps) {
    const SegTokArgs p{a, actions, ld, adv, reinterpret_cast<float*>(ws + L.tok_adv),
                       reinterpret_cast<double*>(ws + L.tok_w), aux ? aux->tok_traj : nullptr,
                       aux ? aux->gather_idx : nullptr};
    hipLaunchKernelGGL(k_segments_tok, dim3((unsigned)(T > 0 ? (T + 255) / 256 : 1)), dim3(256), 0, s, p);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_segments, dim3(1), dim3(256), 0, s, a);
  if (T > 0)
    hipLaunchKernelGGL(k_tok_traj, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, s, T, seg->n_traj,
                       a.traj_tok_off, a.hdr, actions, ld, adv, a.w, reinterpret_cast<float*>(ws + L.tok_adv),
                       reinterpret_cast<double*>(ws + L.tok_w), aux ? aux->tok_traj : nullptr,
                       aux ? aux->gather_idx : nullptr);
  return hipGetLastError();
}

TokenArgs make_token_args(int64_t V, const int32_t* actions, const float* behave, const float* prox,
                          const float* adv, const grpo_loss_params* p, char* ws, const LossWs& L,
                          const grpo_aux* aux) {
  TokenArgs a;
  a.V = V;
  a.actions = actions;
  a.behave = behave;
  a.prox = prox;
  a.tok_adv = reinterpret_cast<const float*>(ws + L.tok_adv);
  a.tok_w = reinterpret_cast<const double*>(ws + L.tok_w);
  a.hdr = reinterpret_cast<WsHeader*>(ws + L.hdr);
  a.contrib = reinterpret_cast<double*>(ws + L.contrib);
  a.state = reinterpret_cast<int8_t*>(ws + L.state);
  a.tok_ratio = reinterpret_cast<double2*>(ws + L.tok_ratio);
  a.token_logp = aux ? aux->token_logp : nullptr;
  a.lo = 1.0 - (double)p->eps_low;
  a.hi = 1.0 + (double)p->eps_high;
  a.c = (double)p->dual_clip_c;
  a.grad_scale = (double)p->grad_scale;
  return a;
}

// ---- reduction -----------------------------------------------------------------
// One workgroup per trajectory sums its tokens' contributions in a fixed
// order; the last workgroup to finish sums the trajectories in index order.
struct ReduceArgs {
  int64_t T;
  int32_t n_traj;
  WsHeader* hdr;
  const int32_t* traj_tok_off;
  const double* contrib;
  const int8_t* state;
  const double2* tok_ratio;  // ws [T]: (r, rho), NaN outside the loss
  double* traj_loss;         // ws
  double* traj_rstats;       // ws [n_traj][6]: sum r, min r, max r, sum rho, min rho, max rho
  double* loss_out;
  double* aux_traj_loss;
  int64_t* aux_clip_counts;
  double* aux_ratio_stats;
  int32_t* aux_error_flags;
};

template <int NT>
__device__ __forceinline__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) sh[wv] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int q = 0; q < NT / 64; ++q) r += sh[q];
  __syncthreads();
  return r;  // valid in thread 0
}

template <int NT, bool MAX>
__device__ __forceinline__ double block_ext(double v, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double u = __shfl_xor(v, o, 64);
    v = MAX ? fmax(v, u) : fmin(v, u);
  }
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) sh[wv] = v;
  __syncthreads();
  double r = v;
  if (threadIdx.x == 0)
    for (int q = 0; q < NT / 64; ++q) r = MAX ? fmax(r, sh[q]) : fmin(r, sh[q]);
  __syncthreads();
  return r;  // valid in thread 0
}

// Latency-bound: a few hundred tokens per workgroup, then one workgroup over the trajectories.  Clip counts and ratio
// statistics are formed for the calls that ask for them only, and a workgroup's four counts go into the header as two
// 64-bit atomics (every count is below 2^31).  With four atomics from every wave, all on one line, and every statistic
// reduced whether wanted or not, the launch took 32 us at T = 32,411 (every output asked for) and 27 at 30,000 (the
// loss alone; 7 now).  Every output is gathered in one walk over the tokens, four at a time: the whole loss call on
// rows of 64 with every output took 69 us at 30,000 tokens in 8 trajectories and 492 at 100,000 in one with a walk for
// each kind of output, and takes 37 and 125.
__global__ __launch_bounds__(256) void k_reduce(const ReduceArgs a) {
  __shared__ double sh[4];
  __shared__ int64_t shc[4][2];
  __shared__ int is_last;
  const int i = blockIdx.x, tid = threadIdx.x;
  const bool ratios = a.aux_ratio_stats != nullptr, counts = ratios || a.aux_clip_counts != nullptr;
  const int64_t t0 = min(max((int64_t)a.traj_tok_off[i], (int64_t)0), a.T);
  const int64_t t1 = min(max((int64_t)a.traj_tok_off[i + 1], t0), a.T);
  double acc = 0.0;
  double sr = 0.0, srho = 0.0;
  double rmin = INFINITY, rmax = -INFINITY, pmin = INFINITY, pmax = -INFINITY;
  int64_t c0 = 0, c1 = 0;  // eps-clip cut and dual-clip cut, ratio outside and valid: low and high halves
  if (!counts) {
    for (int64_t t = t0 + tid; t < t1; t += 256) acc += a.contrib[t];
  } else {  // one walk: a trajectory's tokens are a chain of memory latencies, of which three walks take three
    auto add = [&](double c, int st) {
      acc += c;
      c0 += (int64_t)((st & kStateEpsCut) != 0) | ((int64_t)((st & kStateDualCut) != 0) << 32);
      c1 += (int64_t)((st & kStateOutside) != 0) | ((int64_t)((st & kStateValid) != 0) << 32);
    };
    auto add_ratios = [&](double2 q, int st) {
      if (!(st & kStateValid)) return;
      sr += q.x;
      srho += q.y;
      rmin = fmin(rmin, q.x);
      rmax = fmax(rmax, q.x);
      pmin = fmin(pmin, q.y);
      pmax = fmax(pmax, q.y);
    };
    constexpr int U = 4;  // tokens in flight
    int64_t t = t0 + tid;
    for (; t + (U - 1) * 256 < t1; t += U * 256) {
      double c[U];
      double2 q[U];
      int st[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        c[u] = a.contrib[t + u * 256];
        st[u] = a.state[t + u * 256];
        if (ratios) q[u] = a.tok_ratio[t + u * 256];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        add(c[u], st[u]);
        if (ratios) add_ratios(q[u], st[u]);
      }
    }
    for (; t < t1; t += 256) {
      const int st = a.state[t];
      add(a.contrib[t], st);
      if (ratios) add_ratios(a.tok_ratio[t], st);
    }
  }
  const double tot = block_sum<256>(acc, sh);
  if (counts) {
    c0 = wave_sum_i64(c0);
    c1 = wave_sum_i64(c1);
    if ((tid & 63) == 0) {
      shc[tid >> 6][0] = c0;
      shc[tid >> 6][1] = c1;
    }
    __syncthreads();
    if (tid < 2) {
      const int64_t c = shc[0][tid] + shc[1][tid] + shc[2][tid] + shc[3][tid];
      if (c) atomicAdd((unsigned long long*)&a.hdr->counts[tid], (unsigned long long)c);
    }
  }
  if (ratios) {
    const double tsr = block_sum<256>(sr, sh), tsrho = block_sum<256>(srho, sh);
    const double trmin = block_ext<256, false>(rmin, sh), trmax = block_ext<256, true>(rmax, sh);
    const double tpmin = block_ext<256, false>(pmin, sh), tpmax = block_ext<256, true>(pmax, sh);
    if (tid == 0) {
      double* rs = a.traj_rstats + 6 * (int64_t)i;
      rs[0] = tsr;
      rs[1] = trmin;
      rs[2] = trmax;
      rs[3] = tsrho;
      rs[4] = tpmin;
      rs[5] = tpmax;
    }
  }
  __syncthreads();  // the counter updates are performed before the block reports done
  if (tid == 0) {
    a.traj_loss[i] = tot;
    __threadfence();
    const unsigned prev = atomicAdd(&a.hdr->done, 1u);
    is_last = (prev == (unsigned)gridDim.x - 1);
  }
  __syncthreads();
  if (!is_last) return;
  __threadfence();
  double part = 0.0;
  for (int q = tid; q < a.n_traj; q += 256)
    part += __hip_atomic_load(&a.traj_loss[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const double loss = block_sum<256>(part, sh);
  const int flags = __hip_atomic_load(&a.hdr->flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const bool bad = flags & GRPO_FLAG_OFFSETS;
  if (a.aux_traj_loss)
    for (int q = tid; q < a.n_traj; q += 256)
      a.aux_traj_loss[q] =
          bad ? (double)NAN : __hip_atomic_load(&a.traj_loss[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (a.aux_ratio_stats) {
    // per-trajectory partials in index order (sums through the same fixed-shape tree as the loss)
    auto ld = [&](int q, int k) {
      return __hip_atomic_load(&a.traj_rstats[6 * (int64_t)q + k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    double p_sr = 0.0, p_srho = 0.0, p_rmin = INFINITY, p_rmax = -INFINITY, p_pmin = INFINITY, p_pmax = -INFINITY;
    for (int q = tid; q < a.n_traj; q += 256) {
      p_sr += ld(q, 0);
      p_rmin = fmin(p_rmin, ld(q, 1));
      p_rmax = fmax(p_rmax, ld(q, 2));
      p_srho += ld(q, 3);
      p_pmin = fmin(p_pmin, ld(q, 4));
      p_pmax = fmax(p_pmax, ld(q, 5));
    }
    const double v0 = block_sum<256>(p_sr, sh), v3 = block_sum<256>(p_srho, sh);
    const double v1 = block_ext<256, false>(p_rmin, sh), v2 = block_ext<256, true>(p_rmax, sh);
    const double v4 = block_ext<256, false>(p_pmin, sh), v5 = block_ext<256, true>(p_pmax, sh);
    if (tid == 0) {
      double* o = a.aux_ratio_stats;
      const double nan = (double)NAN;
      o[0] = bad ? nan : v0;
      o[1] = bad ? nan : v1;
      o[2] = bad ? nan : v2;
      o[3] = bad ? nan : v3;
      o[4] = bad ? nan : v4;
      o[5] = bad ? nan : v5;
      const int64_t c = __hip_atomic_load(&a.hdr->counts[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      o[6] = (double)(c & 0xffffffff);
      o[7] = (double)(c >> 32);
    }
  }
  if (tid == 0) {
    *a.loss_out = bad ? (double)NAN : loss;
    if (a.aux_clip_counts) {
      const int64_t c = __hip_atomic_load(&a.hdr->counts[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      a.aux_clip_counts[0] = c & 0xffffffff;
      a.aux_clip_counts[1] = c >> 32;
    }
    if (a.aux_error_flags) *a.aux_error_flags = flags;
  }
}

hipError_t launch_reduce(int64_t T, int32_t n_traj, char* ws, const LossWs& L, double* loss_out,
                         const grpo_aux* aux, hipStream_t s) {
  ReduceArgs a;
  a.T = T;
  a.n_traj = n_traj;
  a.hdr = reinterpret_cast<WsHeader*>(ws + L.hdr);
  a.traj_tok_off = reinterpret_cast<const int32_t*>(ws + L.traj_tok_off);
  a.contrib = reinterpret_cast<const double*>(ws + L.contrib);
  a.state = reinterpret_cast<const int8_t*>(ws + L.state);
  a.tok_ratio = reinterpret_cast<const double2*>(ws + L.tok_ratio);
  a.traj_loss = reinterpret_cast<double*>(ws + L.traj_loss);
  a.traj_rstats = reinterpret_cast<double*>(ws + L.traj_rstats);
  a.loss_out = loss_out;
  a.aux_traj_loss = aux ? aux->traj_loss : nullptr;
  a.aux_clip_counts = aux ? aux->clip_counts : nullptr;
  a.aux_ratio_stats = aux ? aux->ratio_stats : nullptr;
  a.aux_error_flags = aux ? aux->error_flags : nullptr;
  hipLaunchKernelGGL(k_reduce, dim3(n_traj), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ---- group advantages (Sec. 3.2) -------------------------------------------------
// One workgroup per group; the moments are summed serially in fp64 so the
// result does not depend on the launch shape.
// mode GRPO_ADV_SUCCESS_FILTER: A_i = 1[r_i > 0] (RAFT++, Sec. 3.2 / Table 5).
// mixed (nullable): 1 when the group's rewards are not all equal (DAPO dynamic
// sampling, Sec. 3.2); n_mixed (nullable, cleared beforehand) counts them.
__global__ __launch_bounds__(64) void k_advantages(const float* __restrict__ r, int G, int mode, int ddof,
                                                   double std_eps, float* __restrict__ adv,
                                                   int32_t* __restrict__ mixed, int32_t* __restrict__ n_mixed) {
  __shared__ double sh_mean, sh_den;
  const int64_t base = (int64_t)blockIdx.x * G;
  if (threadIdx.x == 0 && (mixed || n_mixed)) {
    int m = 0;
    for (int q = 1; q < G; ++q) m |= (r[base + q] != r[base]);
    if (mixed) mixed[blockIdx.x] = m;
    if (n_mixed && m) atomicAdd(n_mixed, 1);
  }
  if (mode == GRPO_ADV_SUCCESS_FILTER) {
    for (int q = threadIdx.x; q < G; q += 64) adv[base + q] = (r[base + q] > 0.f) ? 1.f : 0.f;
    return;
  }
  if (threadIdx.x == 0) {
    double mean = 0.0;
    for (int q = 0; q < G; ++q) mean += (double)r[base + q];
    mean /= (double)G;
    double ss = 0.0;
    for (int q = 0; q < G; ++q) {
      const double d = (double)r[base + q] - mean;
      ss += d * d;
    }
    const double sd = (G - ddof > 0) ? sqrt(ss / (double)(G - ddof)) : 0.0;
    sh_mean = mean;
    sh_den = sd + std_eps;
  }
  __syncthreads();
  const double mean = sh_mean, den = sh_den;
  for (int q = threadIdx.x; q < G; q += 64)
    adv[base + q] = (den == 0.0) ? 0.f : (float)(((double)r[base + q] - mean) / den);
}

}  // namespace grpo

namespace grpo {
__global__ void k_clear_i32(int32_t* p) { *p = 0; }

// dst = src * *scale, in fp32, rounded to nearest even bf16; 8 elements a step and thread.  HBM-bound: 6 bytes per
// element.  At 3,584 x 151,936 0.62 ms (5.3 TB/s); the two passes it replaces (an fp32 product, then the rounding) took
// 1.26 ms and moved 14 bytes.
__global__ __launch_bounds__(256) void k_scale_to_bf16(const float* __restrict__ src, const float* __restrict__ scale,
                                                       uint16_t* __restrict__ dst, int64_t n) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  const float g = *scale;
  const int64_t step = (int64_t)gridDim.x * 256 * 8;
  for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8; i < n; i += step) {
    if (i + 8 <= n) {
      const f32x4 a = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + i));
      const f32x4 b = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + i) + 1);
      const u32x4 o = {pack_bf16(a[0] * g, a[1] * g), pack_bf16(a[2] * g, a[3] * g), pack_bf16(b[0] * g, b[1] * g),
                       pack_bf16(b[2] * g, b[3] * g)};
      __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(dst + i));
    } else {
      for (int64_t j = i; j < n; ++j) dst[j] = (uint16_t)(pack_bf16(src[j] * g, 0.f) & 0xffffu);
    }
  }
}
}  // namespace grpo

// For the torch binding's autograd wrappers, not part of the ABI of grpo.h: dst[i] = bf16(src[i] * *scale), i < n.  src
// (fp32) and dst (bf16) 16-byte aligned device arrays that don't overlap, scale a device fp32 scalar.
extern "C" int grpo_binding_scale_to_bf16(const float* src, const float* scale, void* dst, int64_t n, hipStream_t s) {
  if (n < 0) return GRPO_ERR_SHAPE;
  if (!scale || (n > 0 && (!src || !dst))) return GRPO_ERR_ARG;
  if (!grpo::aligned(src, 16) || !grpo::aligned(dst, 16) || !grpo::aligned(scale, 4)) return GRPO_ERR_ALIGN;
  if (n == 0) return GRPO_OK;
  const int64_t blocks = (n + 2047) / 2048;
  hipLaunchKernelGGL(grpo::k_scale_to_bf16, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, s, src,
                     scale, static_cast<uint16_t*>(dst), n);
  return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

extern "C" int grpo_advantages_ex(const float* rewards, int32_t n_traj, int32_t group_size, int32_t mode,
                                  int32_t ddof, float std_eps, float* adv_out, int32_t* group_mixed,
                                  int32_t* n_mixed, hipStream_t s) {
  if (!rewards || !adv_out) return GRPO_ERR_ARG;
  if (mode != GRPO_ADV_GROUP_NORM && mode != GRPO_ADV_SUCCESS_FILTER) return GRPO_ERR_ARG;
  if (ddof != 0 && ddof != 1) return GRPO_ERR_ARG;
  if (!(std_eps >= 0.f) || !isfinite(std_eps)) return GRPO_ERR_ARG;
  if (n_traj < 1 || group_size < 1 || n_traj % group_size != 0) return GRPO_ERR_SHAPE;
  if (n_mixed) hipLaunchKernelGGL(grpo::k_clear_i32, dim3(1), dim3(1), 0, s, n_mixed);
  hipLaunchKernelGGL(grpo::k_advantages, dim3(n_traj / group_size), dim3(64), 0, s, rewards, group_size, mode, ddof,
                     (double)std_eps, adv_out, group_mixed, n_mixed);
  return hipGetLastError() == hipSuccess ? GRPO_OK : GRPO_ERR_HIP;
}

extern "C" int grpo_advantages(const float* rewards, int32_t n_traj, int32_t group_size, int32_t ddof,
                               float std_eps, float* adv_out, hipStream_t s) {
  return grpo_advantages_ex(rewards, n_traj, group_size, GRPO_ADV_GROUP_NORM, ddof, std_eps, adv_out, nullptr,
                            nullptr, s);
}

extern "C" const char* grpo_status_str(int status) {
  switch (status) {
    case GRPO_OK: return "GRPO_OK";
    case GRPO_ERR_ARG: return "GRPO_ERR_ARG: a required pointer is NULL or a scalar is out of range";
    case GRPO_ERR_SHAPE: return "GRPO_ERR_SHAPE: inconsistent sizes";
    case GRPO_ERR_DTYPE: return "GRPO_ERR_DTYPE: unsupported dtype";
    case GRPO_ERR_WORKSPACE: return "GRPO_ERR_WORKSPACE: workspace missing or too small";
    case GRPO_ERR_ALIGN: return "GRPO_ERR_ALIGN: a device pointer is misaligned";
    case GRPO_ERR_HIP: return "GRPO_ERR_HIP: a HIP launch failed";
    default: return "unknown grpo status";
  }
}
