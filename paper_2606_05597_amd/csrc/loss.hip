// The logits path: streaming log-softmax + gather, the per-token surrogate of
// Eq. 1 (dual clip of Eq. 2), and dlogits, one workgroup per token row.
//
// Every row is read from HBM once with 16-byte loads (a wavefront covers 1 KiB
// contiguous per instruction), reduced to (max, sum exp) per thread, combined
// across the workgroup, and dlogits are formed from the same registers and
// written once: V*s bytes read and V*s written per token.
//
//  k_rows_pipe      long bf16 rows (81,920 < V <= 188,416): persistent, one
//                   workgroup of 1024 threads per CU.  Row t+G streams in
//                   while row t's dlogits are written: part of each row lives
//                   in LDS (global_load_lds), the rest in registers.
//  k_rows_resident  shorter rows: one workgroup per row, several per CU.
//  bf16 rows that are not whole 16-byte vectors (odd vocabularies, strides or
//  addresses) take the same kernels, split at the 16-byte boundaries into
//  vectors and at most 14 edge elements (device.h RowSplit).
//  k_rows_stream    bf16 rows that one CU cannot hold (beyond 188,416 columns), up
//                   to 4 MiB: persistent, most of the row held, the rest read a
//                   second time from the caches.
//  k_rows_twice     (logp.hip) fp32 rows beyond 77,824 columns (rows_twice): one
//                   workgroup per row, part of it held, the rest read a second time.
//  two passes       longer rows, and long rows without dlogits: each row reduced
//                   to a record (logp.hip), then the record turned into the token
//                   epilogue and the row's dlogits (vocab.hip), which reads the
//                   row again.
//  k_rows_elements  fp32 rows that are not whole 16-byte vectors, and rows whose
//                   dlogits lie at another distance from a 16-byte boundary than
//                   their logits: element loads.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "device.h"
#include "launch.h"

namespace grpo {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Row-pass arguments: the logits, the dlogits destination and the token epilogue.
struct RowArgs {
  const void* logits;
  void* dlogits;  // nullable: forward only
  int64_t ld;     // row stride in elements
  int T;
  int chunk;      // k_rows_pipe: consecutive rows a workgroup takes at a time (>= 1) in rows [0, r0)
  int r0;         // k_rows_pipe: a multiple of chunk * gridDim.x
  int chunk2;     // k_rows_pipe: rows [r0, T) go chunk2 at a time, one chunk per workgroup (>= 1)
  bool staged;    // k_rows_elements: the dynamic LDS holds a row
  TokenArgs tok;
};

// Element e of a 16-byte vector (8 bf16 or 4 fp32), widened to fp32.
template <typename Tin>
__device__ __forceinline__ float vec_elem(const u32x4& x, int e) {
  if constexpr (sizeof(Tin) == 2) {
    uint32_t w = x[0];
#pragma unroll
    for (int q = 1; q < 4; ++q)
      if ((e >> 1) == q) w = x[q];
    return (e & 1) ? bf16_hi(w) : bf16_lo(w);
  } else {
    uint32_t w = x[0];
#pragma unroll
    for (int q = 1; q < 4; ++q)
      if (e == q) w = x[q];
    return __uint_as_float(w);
  }
}

// sum of exp(z - m) over the vector, with nmb = -m*log2(e)
template <typename Tin>
__device__ __forceinline__ float vec_sumexp(const u32x4& x, float nmb) {
  float s = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if constexpr (sizeof(Tin) == 2) {
      s += __builtin_amdgcn_exp2f(fmaf(bf16_lo(x[q]), kLog2e, nmb)) +
           __builtin_amdgcn_exp2f(fmaf(bf16_hi(x[q]), kLog2e, nmb));
    } else {
      s += __builtin_amdgcn_exp2f(fmaf(__uint_as_float(x[q]), kLog2e, nmb));
    }
  }
  return s;
}

// The LDS part of a k_rows_pipe row keeps its terms: the sum pass overwrites each vector of 8 bf16 logits in the
// thread's own LDS slot with its terms e = exp(z - m) as fp16 pairs (round to nearest even), and the dlogits pass
// forms d = g exp(z - lse) = c e with one multiply, c = g exp(m - lse), instead of a second exponential.  The terms
// are <= 1: relative error at most 2^-11 for e >= 2^-14, absolute at most 2^-25 below, before the bf16 rounding of
// d.  The sum is formed from the fp32 terms in vec_sumexp's order.  (Not the register part: kept there, the
// compiler issued all of the part's exponentials ahead of their packs and spilled the fp32 terms; and with three
// register vectors' terms parked in the LDS left free, the kernel ran no faster.)
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_f16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, f16x2));
}
__device__ __forceinline__ f32x2 unpack_f16(uint32_t w) {
  return __builtin_convertvector(__builtin_bit_cast(f16x2, w), f32x2);
}
__device__ __forceinline__ float vec_sumexp_keep(u32x4& x, float nmb) {
  float s = 0.f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float lo = __builtin_amdgcn_exp2f(fmaf(bf16_lo(x[q]), kLog2e, nmb));
    const float hi = __builtin_amdgcn_exp2f(fmaf(bf16_hi(x[q]), kLog2e, nmb));
    s += lo + hi;
    x[q] = pack_f16(lo, hi);
  }
  return s;
}
// dlogits of a vector of kept terms, bf16 round to nearest even; c carries the row's sign; the action column (when
// it falls in this vector) replaced by d_a.
__device__ __forceinline__ u32x4 vec_dlogits_kept(const u32x4& e, float c, bool has_act, int act_lane, float d_a) {
  u32x4 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x2 f = unpack_f16(e[q]);
    o[q] = pack_bf16(f[0] * c, f[1] * c);
  }
  if (has_act) {
    const uint32_t da = pack_bf16(d_a, 0.f) & 0xffffu;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((act_lane >> 1) == q) o[q] = (act_lane & 1) ? ((o[q] & 0xffffu) | (da << 16)) : ((o[q] & 0xffff0000u) | da);
  }
  return o;
}

// Combines every thread's (shift m >= kShiftMin, sum s of exp(z - m)) into the row's (M, S),
// valid in thread 0: within each wave (DPP within rows of 16 lanes, then the
// four rows), then across the NW <= 16 waves by the first 16 lanes of wave 0,
// one wave partial per lane.  The rescale factors exp(m - M) <= 1 are fp32 and
// the sums fp64.  Every lane of the workgroup takes part.  Ends with every wave
// past a barrier.
template <int NW>
__device__ __forceinline__ void block_combine(float m, float s, float* sh_m, double* sh_s, double& M_out,
                                              double& S_out) {
  static_assert(NW >= 1 && NW <= 16, "one wave partial per lane of a 16-lane row");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const float mw = wave_max_dpp(m);
  const double sw = wave_sum_dpp((double)s * (double)__builtin_amdgcn_exp2f((m - mw) * kLog2e));
  if (lane == 0) {
    sh_m[wv] = mw;
    sh_s[wv] = sw;
  }
  __syncthreads();
  if (wv == 0) {
    const float mq = lane < NW ? sh_m[lane] : -INFINITY;
    const float M = row16_max(mq);
    const double S =
        row16_sum(mq == -INFINITY ? 0.0 : sh_s[lane < NW ? lane : 0] * (double)__builtin_amdgcn_exp2f((mq - M) * kLog2e));
    M_out = (double)M;
    S_out = S;
  }
}

// As block_combine, but every wave reads the NW wave partials and forms the row's (M, S) itself, so that every
// lane of the workgroup holds them after the one barrier (each 16-lane row of a wave reduces the same partials).
template <int NW>
__device__ __forceinline__ void block_combine_all(float m, float s, float* sh_m, double* sh_s, double& M_out,
                                                  double& S_out) {
  static_assert(NW >= 1 && NW <= 16, "one wave partial per lane of a 16-lane row");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, r = lane & 15;
  const float mw = wave_max_dpp(m);
  const double sw = wave_sum_dpp((double)s * (double)__builtin_amdgcn_exp2f((m - mw) * kLog2e));
  if (lane == 0) {
    sh_m[wv] = mw;
    sh_s[wv] = sw;
  }
  __syncthreads();
  const float mq = r < NW ? sh_m[r] : -INFINITY;
  const float M = row16_max(mq);
  M_out = (double)M;
  S_out = row16_sum(mq == -INFINITY ? 0.0 : sh_s[r < NW ? r : 0] * (double)__builtin_amdgcn_exp2f((mq - M) * kLog2e));
}

// ---- persistent pipelined kernel for long bf16 rows ----------------------------
// 16 bytes per lane from the buffer (rsrc, voff + soff) into LDS at lds_base + 16 * lane, non-temporal.
// Inline asm: the compiler's own handling of LDS DMA would hold every LDS read back until all LDS DMA in
// flight has landed; the kernel orders them with explicit waits instead.  M0 carries the LDS address;
// nothing else in this kernel uses it.  An LDS DMA must not follow the write of M0 directly: one wait state
// between them (the compiler inserts the same for its own LDS DMA; it cannot see inside this asm).
__device__ __forceinline__ void dma16_nt(uint32_t lds_base, uint32_t voff, uint32_t soff, u32x4 rsrc) {
  lds_base = __builtin_amdgcn_readfirstlane(lds_base);
  soff = __builtin_amdgcn_readfirstlane(soff);
#pragma unroll
  for (int k = 0; k < 4; ++k) rsrc[k] = __builtin_amdgcn_readfirstlane(rsrc[k]);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds" ::"s"(lds_base), "v"(voff), "s"(rsrc),
               "s"(soff)
               : "memory", "m0");
}
__device__ __forceinline__ u32x4 row_rsrc_words(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  u32x4 r = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, bytes, kRsrcWord3};
  return r;
}
// waits until at most N vector-memory operations of this wave are outstanding (they complete in order)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Hides the register vectors' values from the optimiser, so that the widened
// bf16 of one pass is recomputed in the next instead of kept live across it.
template <int N>
__device__ __forceinline__ void fresh(u32x4 (&v)[N]) {
#pragma unroll
  for (int q = 0; q < N; ++q) asm volatile("" : "+v"(v[q]));
}

// Each thread owns NV vectors of 8 bf16, with (NV-1)*1024 < V/8 <= NV*1024 so
// that only the last vector can be partial.  RAG: rows that are not whole aligned
// vectors (RowSplit).  A row then has floor(V/8) or floor(V/8) - 1 vectors, so all
// but the last are still whole; a thread's edge element travels in a register, loaded
// before the next row's LDS part is staged, so that the waits count the same
// operations; and the LDS part keeps its logits, not their fp16 terms, so that
// dlogits are formed in fp32 throughout (the terms are worth 0.3%).  The first NP live in LDS (staged
// with buffer loads straight to LDS and read back in every pass), the other
// NR = NV - NP in registers.  Once the row's lse is known, dlogits are written
// first for the LDS part, which is then re-staged with the next row, and then
// for the register part, whose registers are then reloaded with the next
// row's vectors.
template <int NV, int NP, bool RAG>
__global__ __launch_bounds__(1024) void k_rows_pipe(const RowArgs a) {
  constexpr int NT = 1024, NW = NT / 64, NR = NV - NP, VB = NT * 16;  // VB: bytes per vector slot
  __shared__ __attribute__((aligned(16))) u32x4 stage[NP * NT];
  __shared__ float sh_m[NW];
  __shared__ double sh_s[NW];
  __shared__ float sh_za;
  __shared__ TokenIn sh_in;  // inputs of the row about to start (wave 1 loads them during the previous row)
  const int wv = threadIdx.x >> 6;
  const uint16_t* logits = static_cast<const uint16_t*>(a.logits);
  uint16_t* dlogits = static_cast<uint16_t*>(a.dlogits);
  auto split = [&](int r) { return row_split<uint16_t, RAG>(logits + (int64_t)r * a.ld, a.tok.V); };

  const uint32_t lds_stage =
      (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) u32x4*)stage) + wv * 64 * 16;
  auto stage_row = [&](int r, int voff) {  // vectors 0..NP-1 of row r -> LDS, asynchronously
    const RowSplit sp = split(r);
    const u32x4 src = row_rsrc_words(logits + (int64_t)r * a.ld + sp.head, (uint32_t)sp.nvec * 16u);
#pragma unroll
    for (int j = 0; j < NP; ++j) dma16_nt(lds_stage + j * NT * 16, voff, j * VB, src);
  };
  auto load_regs = [&](u32x4 (&dst)[NR], int r, int voff) {
    const RowSplit sp = split(r);
    const __amdgpu_buffer_rsrc_t src = row_rsrc(logits + (int64_t)r * a.ld + sp.head, sp.nvec * 16);
#pragma unroll
    for (int q = 0; q < NR; ++q) dst[q] = __builtin_amdgcn_raw_buffer_load_b128(src, voff, (NP + q) * VB, kStream);
  };

  // Rows [0, r0) go to workgroups in chunks of `chunk` consecutive rows, chunk c to workgroup c mod gridDim.x;
  // the rest, fewer than chunk * gridDim.x rows, in one chunk of chunk2 rows per workgroup, so that no workgroup
  // has more than chunk2 rows beyond the others.  A workgroup walks its chunks in order, so the row it stages
  // next is usually the one after the row it writes.  Past its last row, next_row returns T.
  const int C = a.chunk, R0 = a.r0, C2 = a.chunk2;
  auto next_row = [&](int r) {
    const int q = r + 1;
    if (r < R0) {
      if (q % C != 0) return q;
      const int nq = q + ((int)gridDim.x - 1) * C;
      return nq < R0 ? nq : min(R0 + (int)blockIdx.x * C2, a.T);
    }
    return ((q - R0) % C2 != 0 && q < a.T) ? q : a.T;
  };
  int t = R0 > 0 ? (int)blockIdx.x * C : R0 + (int)blockIdx.x * C2;
  if (t >= a.T) return;
  u32x4 reg[NR];
  float ez = -INFINITY;  // RAG: the thread's edge element of row t
  auto load_edge = [&](int r, int tid) {
    const int c = edge_col<uint16_t>(split(r), tid);
    return c >= 0 ? load_elem(logits + (int64_t)r * a.ld + c) : -INFINITY;
  };
  if constexpr (RAG) ez = load_edge(t, threadIdx.x);
  if (threadIdx.x == 64) sh_in = token_load(a.tok, t);
  stage_row(t, threadIdx.x * 16);
  load_regs(reg, t, threadIdx.x * 16);
  wait_vmcnt<NR>();  // this wave's LDS part of row t has landed; the register loads may still be in flight

  for (int t_next = 0; t < a.T; t = t_next) {
    // The thread index is laundered per row so that nothing derived from it
    // is hoisted out of the row loop and kept live across it.
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int voff = tid * 16;
    const RowSplit sp = split(t);
    const bool last_full = tid < sp.nvec - (NV - 1) * NT;
    const int tn = next_row(t);
    t_next = tn;
    lds_barrier();  // every wave's LDS part of row t has landed, and sh_in holds row t's inputs
    const TokenIn in = sh_in;
    const bool act_ok = in.act >= 0 && in.act < a.tok.V;
    int act_lane;
    const int act_vec = vec_of<uint16_t>(sp, act_ok ? in.act : -1, act_lane);
    const int ecol = RAG ? edge_col<uint16_t>(sp, tid) : -1;

    // (max, sum exp) over the LDS part first, while the register part is still landing
    float m1 = kShiftMin;
#pragma unroll 1
    for (int j = 0; j < NP; ++j) {
      const u32x4 x = stage[j * NT + tid];
      m1 = vec_max<uint16_t>(x, m1);
      if (j * NT + tid == act_vec) sh_za = vec_elem<uint16_t>(x, act_lane);
    }
    const float nmb1 = -m1 * kLog2e;
    float s1 = 0.f;
#pragma unroll 1
    for (int j = 0; j < NP; ++j) {  // the terms replace the logits in the thread's own LDS slots
      u32x4 x = stage[j * NT + tid];
      if constexpr (RAG) {
        s1 += vec_sumexp<uint16_t>(x, nmb1);
      } else {
        s1 += vec_sumexp_keep(x, nmb1);
        stage[j * NT + tid] = x;
      }
    }
    float m = m1;
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int j = NP + q;
      if (j < NV - 1 || last_full) {
        m = vec_max<uint16_t>(reg[q], m);
        if (j * NT + tid == act_vec) sh_za = vec_elem<uint16_t>(reg[q], act_lane);
      }
    }
    if constexpr (RAG) {
      m = fmaxf(m, ez);
      if (act_ok && ecol == in.act) sh_za = ez;
    }
    const float nmb = -m * kLog2e;
    float s = s1 * __builtin_amdgcn_exp2f((m1 - m) * kLog2e);
    if constexpr (RAG) s += __builtin_amdgcn_exp2f(fmaf(ez, kLog2e, nmb));  // no edge: exp2(-inf) = 0
    fresh(reg);
#pragma unroll
    for (int q = 0; q < NR; ++q)
      if (NP + q < NV - 1 || last_full) s += vec_sumexp<uint16_t>(reg[q], nmb);

    double M, S;
    block_combine_all<NW>(m, s, sh_m, sh_s, M, S);  // barrier: sh_za is visible, every lane holds (M, S)
    // every wave forms the row's scale itself (no second barrier, no one-lane section); thread 0 writes the
    // token's outputs
    TokenEval ev;
    const RowScale rs = token_eval(a.tok, in, row_lse(M, S), (double)sh_za, ev);
    if (tid == 0) token_store(a.tok, t, in, ev);
    // wave 1 fetches the next row's token inputs meanwhile (every wave read this row's from sh_in before the
    // barrier above; the next row reads them after its first barrier)
    if (tid == 64) sh_in = token_load(a.tok, tn < a.T ? tn : t);

    const uint32_t smask = sign_mask<uint16_t>(rs);
    const float c1 = rs.sign * __builtin_amdgcn_exp2f(rs.nc - nmb1);  // the LDS part's terms: d = c1 e
    int act_l;
    const int act_v = vec_of<uint16_t>(sp, rs.act, act_l);
    fresh(reg);
    // forward only: a zero-sized destination, so the range check drops every store
    const bool write = dlogits != nullptr;
    const __amdgpu_buffer_rsrc_t dst = row_rsrc(write ? dlogits + (int64_t)t * a.ld + sp.head : logits, write ? sp.nvec * 16 : 0);
#pragma unroll 1
    for (int j = 0; j < NP; ++j) {
      u32x4 d;
      if constexpr (RAG) d = vec_dlogits<uint16_t>(stage[j * NT + tid], rs, smask, j * NT + tid == act_v, act_l);
      else d = vec_dlogits_kept(stage[j * NT + tid], c1, j * NT + tid == act_v, act_l, rs.d_a);
      __builtin_amdgcn_raw_buffer_store_b128(d, dst, voff, j * VB, kStream);
    }
    if constexpr (RAG) {
      if (write && ecol >= 0) store_elem(dlogits + (int64_t)t * a.ld + ecol, elem_dlogits(ez, rs, ecol, rs.act));
      ez = load_edge(tn < a.T ? tn : t, tid);
    }
    lds_barrier();  // every wave is done reading stage[] (the stores read registers)
    if (tn < a.T) stage_row(tn, voff);
    // past the last row: a zero-sized source, every load returns 0
    const RowSplit spn = split(tn < a.T ? tn : t);
    const __amdgpu_buffer_rsrc_t nxt =
        row_rsrc(logits + (int64_t)(tn < a.T ? tn : t) * a.ld + spn.head, tn < a.T ? spn.nvec * 16 : 0);
    // All of the register part's stores, then all of its loads: a burst in each direction per wave runs 7-8%
    // faster than alternating store and load per vector.  Each store is followed by two wait states: the compiler
    // reuses a store's data registers in the very next instruction (it inserts no wait for a 16-byte buffer store
    // with a register offset), and when it did, the store wrote the overwritten values.
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const int j = NP + q;
      __builtin_amdgcn_raw_buffer_store_b128(
          vec_dlogits<uint16_t>(reg[q], rs, smask, j * NT + tid == act_v, act_l), dst, voff, j * VB, kStream);
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_nop 1" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < NR; ++q) reg[q] = __builtin_amdgcn_raw_buffer_load_b128(nxt, voff, (NP + q) * VB, kStream);
    // the 2 NR register stores and loads were issued after the LDS part of row tn, so this returns once
    // that part has landed
    wait_vmcnt<2 * NR>();
  }
}

// ---- persistent kernel for rows that one CU cannot hold --------------------------
// As k_rows_pipe (one workgroup of 1024 threads per CU, 16-byte vectors j * 1024 + tid), with the row in three parts:
// vectors 0 .. NP-1 in LDS, the next NR in registers, and the rest streamed, U at a time, through one more set of
// registers.  The streamed part is read twice: forwards for (max, sum exp), then, beginning with the last U vectors,
// which are still there, backwards for dlogits.  HBM-bound.  What the second read finds in the memory-side cache depends
// on how much all CUs together have read in between: up to rows of about 1 MB (256 CUs, 256 MB) most of it, of longer
// rows their ends; the third of a MB per row that the CU holds is saved in any case.
// A row fills the first two parts (at least NP + NR vectors and one element more per thread).
// Every load and store is issued whatever the row's length (stores past it are dropped by the range check of the row's
// descriptor), so that the wait for the LDS part counts the same operations on every row.
template <typename Tin, int NP, int NR, int U, bool RAG>
__global__ __launch_bounds__(1024) void k_rows_stream(const RowArgs a) {
  constexpr int NT = 1024, NW = NT / 64, VB = NT * 16, NH = NP + NR;
  __shared__ __attribute__((aligned(16))) u32x4 stage[NP * NT];
  __shared__ float sh_m[NW];
  __shared__ double sh_s[NW];
  __shared__ float sh_za;
  __shared__ TokenIn sh_in;  // inputs of the row about to start (wave 1 loads them during the previous row)
  const int wv = threadIdx.x >> 6;
  const Tin* logits = static_cast<const Tin*>(a.logits);
  Tin* dlogits = static_cast<Tin*>(a.dlogits);
  auto split = [&](int r) { return row_split<Tin, RAG>(logits + (int64_t)r * a.ld, a.tok.V); };
  auto source = [&](int r, const RowSplit& sp) { return row_rsrc(logits + (int64_t)r * a.ld + sp.head, sp.nvec * 16); };
  const uint32_t lds_stage =
      (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) u32x4*)stage) + wv * 64 * 16;
  auto stage_row = [&](int r, const RowSplit& sp, int voff) {
    const u32x4 src = row_rsrc_words(logits + (int64_t)r * a.ld + sp.head, (uint32_t)sp.nvec * 16u);
#pragma unroll
    for (int j = 0; j < NP; ++j) dma16_nt(lds_stage + j * NT * 16, voff, j * VB, src);
  };
  u32x4 reg[NR], x[U];
  auto load_batch = [&](int r, const RowSplit& sp, int b, int tid) {  // past the row's end: the last vector, left out
    const char* row = reinterpret_cast<const char*>(logits + (int64_t)r * a.ld + sp.head);
#pragma unroll
    for (int u = 0; u < U; ++u)
      x[u] = *reinterpret_cast<const u32x4*>(row + (uint32_t)min((NH + b * U + u) * NT + tid, sp.nvec - 1) * 16u);
  };
  const int nb = (int)((a.tok.V / (16 / (int)sizeof(Tin)) + NT - 1) / NT - NH + U - 1) / U;  // batches, at least one

  // rows to workgroups as in k_rows_pipe
  const int C = a.chunk, R0 = a.r0, C2 = a.chunk2;
  auto next_row = [&](int r) {
    const int q = r + 1;
    if (r < R0) {
      if (q % C != 0) return q;
      const int nq = q + ((int)gridDim.x - 1) * C;
      return nq < R0 ? nq : min(R0 + (int)blockIdx.x * C2, a.T);
    }
    return ((q - R0) % C2 != 0 && q < a.T) ? q : a.T;
  };
  int t = R0 > 0 ? (int)blockIdx.x * C : R0 + (int)blockIdx.x * C2;
  if (t >= a.T) return;
  float ez = -INFINITY;  // RAG: the thread's edge element of row t
  auto load_edge = [&](int r, const RowSplit& sp, int tid) {
    const int c = edge_col<Tin>(sp, tid);
    return c >= 0 ? load_elem(logits + (int64_t)r * a.ld + c) : -INFINITY;
  };
  {
    const RowSplit sp = split(t);
    const __amdgpu_buffer_rsrc_t src = source(t, sp);
    const int voff = threadIdx.x * 16;
    if constexpr (RAG) ez = load_edge(t, sp, threadIdx.x);
    if (threadIdx.x == 64) sh_in = token_load(a.tok, t);
    stage_row(t, sp, voff);
#pragma unroll
    for (int q = 0; q < NR; ++q) reg[q] = __builtin_amdgcn_raw_buffer_load_b128(src, voff, (NP + q) * VB, kStream);
    load_batch(t, sp, 0, threadIdx.x);
    wait_vmcnt<NR + U>();  // this wave's LDS part of row t has landed; the others may still be in flight
  }

  for (int t_next = 0; t < a.T; t = t_next) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // nothing derived from it is hoisted out of the row loop
    const int voff = tid * 16;
    const RowSplit sp = split(t);
    const int tn = next_row(t);
    t_next = tn;
    lds_barrier();  // every wave's LDS part of row t has landed, and sh_in holds row t's inputs
    const TokenIn in = sh_in;
    const bool act_ok = in.act >= 0 && in.act < a.tok.V;
    int act_lane;
    const int act_vec = vec_of<Tin>(sp, act_ok ? in.act : -1, act_lane);
    const int ecol = RAG ? edge_col<Tin>(sp, tid) : -1;

    // (max, sum exp) over the LDS part, then the register part, each with a shift of its own, then the batches
    float m = kShiftMin, s = 0.f;
    auto raise = [&](float mn) {
      s *= __builtin_amdgcn_exp2f((m - mn) * kLog2e);
      m = mn;
    };
    {
      float mn = m;
#pragma unroll 1
      for (int j = 0; j < NP; ++j) {
        const u32x4 v = stage[j * NT + tid];
        mn = vec_max<Tin>(v, mn);
        if (j * NT + tid == act_vec) sh_za = vec_elem<Tin>(v, act_lane);
      }
      m = mn;
#pragma unroll 1
      for (int j = 0; j < NP; ++j) s += vec_sumexp<Tin>(stage[j * NT + tid], -m * kLog2e);
    }
    {
      float mn = m;
#pragma unroll
      for (int q = 0; q < NR; ++q)
      {
        mn = vec_max<Tin>(reg[q], mn);
        if ((NP + q) * NT + tid == act_vec) sh_za = vec_elem<Tin>(reg[q], act_lane);
      }
      if constexpr (RAG) {
        mn = fmaxf(mn, ez);
        if (act_ok && ecol == in.act) sh_za = ez;
      }
      raise(mn);
      fresh(reg);
#pragma unroll
      for (int q = 0; q < NR; ++q)
      {
        s += vec_sumexp<Tin>(reg[q], -m * kLog2e);
        __builtin_amdgcn_sched_barrier(0);  // else every exponential is issued first and its results spill
      }
      if constexpr (RAG) s += __builtin_amdgcn_exp2f(fmaf(ez, kLog2e, -m * kLog2e));  // no edge: exp2(-inf) = 0
    }
#pragma unroll 1
    for (int b = 0; b < nb; ++b) {
      if (b > 0) load_batch(t, sp, b, tid);
      float mn = m;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int vi = (NH + b * U + u) * NT + tid;
        if (vi < sp.nvec) {
          mn = vec_max<Tin>(x[u], mn);
          if (vi == act_vec) sh_za = vec_elem<Tin>(x[u], act_lane);
        }
      }
      raise(mn);
      fresh(x);
#pragma unroll
      for (int u = 0; u < U; ++u)
      {
        if ((NH + b * U + u) * NT + tid < sp.nvec) s += vec_sumexp<Tin>(x[u], -m * kLog2e);
        __builtin_amdgcn_sched_barrier(0);
      }
    }

    double M, S;
    block_combine_all<NW>(m, s, sh_m, sh_s, M, S);  // barrier: sh_za is visible, every lane holds (M, S)
    TokenEval ev;
    const RowScale rs = token_eval(a.tok, in, row_lse(M, S), (double)sh_za, ev);
    if (tid == 0) token_store(a.tok, t, in, ev);
    if (tid == 64) sh_in = token_load(a.tok, tn < a.T ? tn : t);

    const uint32_t smask = sign_mask<Tin>(rs);
    int act_l;
    const int act_v = vec_of<Tin>(sp, rs.act, act_l);
    // forward only: a zero-sized destination, so the range check drops every store
    const bool write = dlogits != nullptr;
    Tin* drow = write ? dlogits + (int64_t)t * a.ld : nullptr;
    const __amdgpu_buffer_rsrc_t dst = row_rsrc(write ? (const void*)(drow + sp.head) : (const void*)logits, write ? sp.nvec * 16 : 0);
    // each store is followed by two wait states, as in k_rows_pipe
    auto put = [&](const u32x4& v, int j) {
      __builtin_amdgcn_raw_buffer_store_b128(vec_dlogits<Tin>(v, rs, smask, j * NT + tid == act_v, act_l), dst, voff,
                                             j * VB, kStream);
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_nop 1" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    fresh(x);
#pragma unroll 1
    for (int b = nb - 1; b >= 0; --b) {
      if (b < nb - 1) load_batch(t, sp, b, tid);
#pragma unroll
      for (int u = 0; u < U; ++u) put(x[u], NH + b * U + u);
    }
#pragma unroll 1
    for (int j = 0; j < NP; ++j)
      __builtin_amdgcn_raw_buffer_store_b128(
          vec_dlogits<Tin>(stage[j * NT + tid], rs, smask, j * NT + tid == act_v, act_l), dst, voff, j * VB, kStream);
    const RowSplit spn = split(tn < a.T ? tn : t);
    if constexpr (RAG) {
      if (write && ecol >= 0) store_elem(drow + ecol, elem_dlogits(ez, rs, ecol, rs.act));
      ez = load_edge(tn < a.T ? tn : t, spn, tid);
    }
    lds_barrier();  // every wave is done reading stage[] (the stores read registers)
    // past the last row: a zero-sized source, every load returns 0
    if (tn < a.T) stage_row(tn, spn, voff);
    const __amdgpu_buffer_rsrc_t nxt =
        row_rsrc(logits + (int64_t)(tn < a.T ? tn : t) * a.ld + spn.head, tn < a.T ? spn.nvec * 16 : 0);
    fresh(reg);
#pragma unroll
    for (int q = 0; q < NR; ++q) put(reg[q], NP + q);
#pragma unroll
    for (int q = 0; q < NR; ++q) reg[q] = __builtin_amdgcn_raw_buffer_load_b128(nxt, voff, (NP + q) * VB, kStream);
    load_batch(tn < a.T ? tn : t, spn, 0, tid);
    // 2 NR + U operations were issued after the LDS part of row tn: this returns once that part has landed
    wait_vmcnt<2 * NR + U>();
  }
}

// ---- register-resident row kernel -------------------------------------------
// NT threads per row, NV 16-byte vectors per thread: V/EPV <= NT*NV.  RAG: rows that
// are not whole aligned vectors (RowSplit), otherwise they are (checked on the host).
// 8 vectors: at least 4 waves per SIMD (128 registers).  Without the bound the compiler joins 8 fp32 vectors'
// exponentials into one wide operation that takes 239: 30,000 x 6,000 459 us, now 279 (5.2 TB/s), 60,000 x 1,504 244,
// now 141.  4 fp32 vectors are 1.5% faster without it.
template <typename Tin, int NT, int NV, bool RAG>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NV == 8 ? 4 : 1))) void k_rows_resident(const RowArgs a) {
  constexpr int NW = NT / 64;
  __shared__ float sh_m[NW];
  __shared__ double sh_s[NW];
  __shared__ float sh_za;

  const int t = blockIdx.x;
  const int tid = threadIdx.x;
  const Tin* row = static_cast<const Tin*>(a.logits) + (int64_t)t * a.ld;
  const RowSplit sp = row_split<Tin, RAG>(row, a.tok.V);
  const int nvec = sp.nvec;
  const u32x4* src = reinterpret_cast<const u32x4*>(row + sp.head);
  const TokenIn in = token_load(a.tok, t);
  const bool act_ok = in.act >= 0 && in.act < a.tok.V;
  int act_lane;
  const int act_vec = vec_of<Tin>(sp, act_ok ? in.act : -1, act_lane);
  const int ecol = RAG ? edge_col<Tin>(sp, tid) : -1;
  float ez = -INFINITY;
  if (RAG && ecol >= 0) ez = load_elem(row + ecol);

  u32x4 buf[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int vi = j * NT + tid;
    if (vi < nvec) buf[j] = __builtin_nontemporal_load(src + vi);
  }
  float m = kShiftMin;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int vi = j * NT + tid;
    if (vi < nvec) {
      m = vec_max<Tin>(buf[j], m);
      if (vi == act_vec) sh_za = vec_elem<Tin>(buf[j], act_lane);
    }
  }
  if constexpr (RAG) {
    m = fmaxf(m, ez);
    if (act_ok && ecol == in.act) sh_za = ez;
  }
  const float nmb = -m * kLog2e;
  float s = RAG ? __builtin_amdgcn_exp2f(fmaf(ez, kLog2e, nmb)) : 0.f;  // no edge: exp2(-inf) = 0
#pragma unroll
  for (int j = 0; j < NV; ++j)
    if (j * NT + tid < nvec) s += vec_sumexp<Tin>(buf[j], nmb);

  double M, S;
  block_combine_all<NW>(m, s, sh_m, sh_s, M, S);  // barrier: sh_za is visible, every lane holds (M, S)
  // every wave forms the row's scale itself; thread 0 writes the token's outputs
  TokenEval ev;
  const RowScale rs = token_eval(a.tok, in, row_lse(M, S), (double)sh_za, ev);
  if (tid == 0) token_store(a.tok, t, in, ev);
  if (!a.dlogits) return;

  const uint32_t smask = sign_mask<Tin>(rs);
  Tin* drow = static_cast<Tin*>(a.dlogits) + (int64_t)t * a.ld;
  u32x4* dst = reinterpret_cast<u32x4*>(drow + sp.head);
  int act_l;
  const int act_v = vec_of<Tin>(sp, rs.act, act_l);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int vi = j * NT + tid;
    if (vi < nvec)
      __builtin_nontemporal_store(vec_dlogits<Tin>(buf[j], rs, smask, vi == act_v, act_l), dst + vi);
  }
  if (RAG && ecol >= 0) store_elem(drow + ecol, elem_dlogits(ez, rs, ecol, rs.act));
}

// ---- element row kernel --------------------------------------------------------
// Any V, ld and element alignment, thread k of 256 on columns k, k + 256, ...: fp32 rows that are not whole aligned
// vectors, and rows whose dlogits lie at another distance from a 16-byte boundary than their logits.  Three sweeps
// (max, sum, dlogits) with U elements in flight.  HELD: the row has at most U elements a thread, which stay in
// registers; otherwise a row that fits the workgroup's dynamic LDS (stage_row) is read from memory once and from there
// afterwards.  A thread's terms are summed one after the other in column order in every form.
// Bound by the element accesses' rate and, unstaged, by the re-reads.  fp32 loss and dlogits with one element in flight
// and every sweep from memory / here: 30,000 x 9,001 0.94 / 0.41 ms (5.3 TB/s), 20,000 x 19,003 1.32 / 0.71, 10,000 x
// 32,003 1.26 / 0.80, 6,000 x 151,669 3.77 / 3.23; of rows held, 20,000 x 101 50 / 34 us, x 1,003 78 / 48, x 2,003 165 /
// 80.
template <typename Tin, int U, bool HELD>
__global__ __launch_bounds__(256) void k_rows_elements(const RowArgs a) {
  constexpr int NT = 256, NW = NT / 64;
  extern __shared__ __attribute__((aligned(16))) char dyn[];
  Tin* stage = reinterpret_cast<Tin*>(dyn);
  __shared__ float sh_m[NW];
  __shared__ double sh_s[NW];
  __shared__ RowScale sh_rs;
  const int t = blockIdx.x, tid = threadIdx.x;
  const int64_t V = a.tok.V;
  const Tin* row = static_cast<const Tin*>(a.logits) + (int64_t)t * a.ld;
  const bool staged = !HELD && a.staged;
  Tin z[U];
  if constexpr (HELD) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (tid + u * NT < V) z[u] = row[tid + u * NT];
  }
  const TokenIn in = token_load(a.tok, t);
  // f(column, logit) for the thread's columns in order
  auto sweep = [&](auto from_lds, auto f) {
    for (int64_t base = tid; base < (HELD ? NT : V); base += NT * U) {
      if constexpr (!HELD) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int64_t v = base + u * NT;
          if (v < V) z[u] = from_lds ? stage[v] : row[v];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t v = base + u * NT;
        if (v < V) f(v, z[u]);
      }
    }
  };
  float m = kShiftMin;
  if (staged)
    sweep(std::false_type(), [&](int64_t v, Tin z) {
      stage[v] = z;  // read back by the same thread
      m = fmaxf(m, load_elem(&z));
    });
  else
    sweep(std::false_type(), [&](int64_t, Tin z) { m = fmaxf(m, load_elem(&z)); });
  const float nmb = -m * kLog2e;
  float s = 0.f;
  auto add = [&](int64_t, Tin z) { s += __builtin_amdgcn_exp2f(fmaf(load_elem(&z), kLog2e, nmb)); };
  if (staged) sweep(std::true_type(), add);
  else sweep(std::false_type(), add);
  double M, S;
  block_combine<NW>(m, s, sh_m, sh_s, M, S);
  if (tid == 0) {
    const bool ok = in.act >= 0 && (int64_t)in.act < V;
    sh_rs = token_finish(a.tok, t, in, row_lse(M, S), ok ? (double)load_elem(row + in.act) : 0.0);
  }
  __syncthreads();
  if (!a.dlogits) return;
  const RowScale rs = sh_rs;
  Tin* drow = static_cast<Tin*>(a.dlogits) + (int64_t)t * a.ld;
  auto put = [&](int64_t v, Tin z) { store_elem(drow + v, elem_dlogits(load_elem(&z), rs, (int)v, rs.act)); };
  if (staged) sweep(std::true_type(), put);
  else sweep(std::false_type(), put);
}

// ---- dispatch ------------------------------------------------------------------
typedef void (*RowKernel)(const RowArgs);

struct Variant {
  int nt, nv;
  RowKernel bf16[2], f32;  // bf16: whole aligned vectors, ragged; none where the persistent kernels come first
};

#define GRPO_VARIANT(NT, NV)                                                                     \
  {                                                                                              \
    NT, NV, {k_rows_resident<uint16_t, NT, NV, false>, k_rows_resident<uint16_t, NT, NV, true>}, \
        k_rows_resident<float, NT, NV, false>                                                    \
  }
#define GRPO_VARIANT_F32(NT, NV) \
  { NT, NV, {nullptr, nullptr}, k_rows_resident<float, NT, NV, false> }

// Searched in order; the first that holds the row is used.  Rows of 3,073 to 4,096 vectors (a bf16 vocabulary of
// 32,000 among them) take 1024 threads x 4 vectors: 6% faster there than 256 x 16 (0.707 against 0.752 ms at
// 32,411 x 32,000), 5% faster than 512 x 8.
static const Variant kVariants[] = {
    GRPO_VARIANT(64, 1),    GRPO_VARIANT(64, 2),    GRPO_VARIANT(64, 4),    GRPO_VARIANT(64, 8),
    GRPO_VARIANT(256, 4),   GRPO_VARIANT(256, 8),   GRPO_VARIANT(256, 12),  GRPO_VARIANT(1024, 4),
    GRPO_VARIANT(256, 20),  GRPO_VARIANT(256, 24),  GRPO_VARIANT(1024, 8),  GRPO_VARIANT(1024, 12),
    GRPO_VARIANT_F32(1024, 16), GRPO_VARIANT_F32(1024, 19),
};  // 1024 threads x 19 vectors is the largest that does not spill

// The persistent kernels for long bf16 rows, one per NV = ceil(V/8/1024) so
// that only each thread's last vector can be partial; NP vectors in LDS.
#define GRPO_PIPE(NV, NP) {k_rows_pipe<NV, NP, false>, k_rows_pipe<NV, NP, true>}
static const RowKernel kPipe[][2] = {
    GRPO_PIPE(11, 6), GRPO_PIPE(12, 6), GRPO_PIPE(13, 7), GRPO_PIPE(14, 7), GRPO_PIPE(15, 1), GRPO_PIPE(16, 2),
    GRPO_PIPE(17, 3), GRPO_PIPE(18, 4),
    GRPO_PIPE(19, 6), GRPO_PIPE(20, 9), GRPO_PIPE(21, 9), GRPO_PIPE(22, 9), GRPO_PIPE(23, 9),
};  // from 15 vectors on, 14 in registers and the rest in LDS, except 19 (V = 151,936): 13 and 6, 0.3% faster
   // than 15 and 4 and 0.4% faster than 14 and 5, with 12 and 7 or 11 and 8 within 0.1% of it (before the LDS
   // part kept its terms, 15 and 4 was 0.4% faster than 14 and 5)
// The streaming kernel: 9 LDS vectors and 12 in registers, whole aligned vectors or ragged.  Loss and dlogits in two
// passes / here: bf16 10,000 x 262,144 2.72 / 1.89 ms (5.6 TB/s of the row read and written once), 12,000 x 200,000
// 2.56 / 1.80.  13 + 5 and 14 + 6 register vectors, which spill, are 1 to 3% slower, a first read past the caches 11%.
static const RowKernel kStreamRows[2] = {k_rows_stream<uint16_t, 9, 12, 4, false>,
                                         k_rows_stream<uint16_t, 9, 12, 4, true>};
// Rows of up to 4 MiB, where the second read misses most of a row and the gain runs out: bf16 in two passes / here, 2,000 x
// 1,048,576 2.23 / 1.90 ms, 1,000 x 2,097,152 2.26 / 2.12, 700 1.56 / 1.48.
constexpr int64_t kStreamMaxRow = (int64_t)1 << 22;
// k_rows_twice: rows addressed with 32-bit offsets, of up to 8 MB, or longer ones while there are too few to fill the
// chip.  Loss and dlogits in two passes / here, ms: 8 MB a row, 600 rows 2.64 / 2.60, 2,100 9.40 / 9.48; 16 MB, 300 rows
// 3.35 / 3.10, 600 5.41 / 5.58; 32 MB, 300 rows 6.66 / 6.26, 600 11.4 / 11.7.
constexpr int64_t kTwiceMaxRow = (int64_t)1 << 30;
static bool rows_twice(int64_t T, int64_t V, int n_cu) {
  return V * 4 <= kTwiceMaxRow && (V * 4 <= (int64_t)8 << 20 || T <= n_cu + n_cu / 2);
}
// Rows without dlogits: a record pass reads a row once, at eight workgroups to a CU, where the kernels that hold most of
// a row read its end a second time and form dlogits for nobody.  They pay while the rows are too few to fill the chip.
// The loss alone, record pass and epilogue / the kernel that holds the row, in us, on 256 CUs:
//   bf16 (k_rows_stream) 200,000 columns, 128 rows 41 / 37, 300 44 / 64, 3,000 195 / 316; 2,097,152 columns, 128 rows
//   308 / 240, 300 331 / 534
//   fp32 (k_rows_twice) 151,936 columns, 400 rows 54 / 45, 520 60 / 68, 3,000 281 / 286; 1,000,000 columns, 400 rows
//   280 / 273, 520 319 / 436, 3,000 1,792 / 1,916; up to 512 KB a row 100,000 columns, 700 rows 53 / 51, 3,000 192 / 190
static bool records_without_dlogits(grpo_dtype dt, int64_t T, int64_t V, int n_cu) {
  return dt == GRPO_BF16 ? T > n_cu / 2 : T > n_cu + n_cu / 2 && V > 131072;
}
// Up to 10 vectors the resident kernel is faster: persistent / resident, 30,000 x 50,000 1.34 / 1.15 ms, 20,000 x 60,000
// 0.98 / 0.91, 20,000 x 80,000 1.24 / 1.18; at 11 and 12 1.09 / 1.10 (15,000 x 90,000), at 13 and 14 5% slower.
constexpr int kPipeMinNV = 11, kPipeMaxNV = 23;  // at most 15 register vectors and 9 LDS vectors per thread
constexpr int64_t kPipeMaxT = (int64_t)1 << 30;  // t + (gridDim.x - 1) * chunk + 1 stays far below 2^31

// Rows of up to kHeldElements elements a thread stay in registers, with no more in flight than the row has: a row of 101
// or 1,003 staged in LDS with 16 in flight a thread took 64 and 74 us (fp32, 20,000 rows), longer than element by
// element from memory.  Held / staged beyond, 16 a thread: bf16 4,093 / 4,097 columns 154 / 126 us, fp32 137 / 146.
constexpr int kHeldElements = 8;
template <typename Tin>
static RowKernel element_kernel(int64_t V) {
  if (V <= 256) return k_rows_elements<Tin, 1, true>;
  if (V <= 1024) return k_rows_elements<Tin, 4, true>;
  if (V <= 256 * kHeldElements) return k_rows_elements<Tin, kHeldElements, true>;
  return k_rows_elements<Tin, 16, false>;
}

struct Launch {
  RowKernel k;
  int nt;
  unsigned grid;
  int chunk = 1, r0 = 0, chunk2 = 1;
  unsigned lds = 0;    // dynamic LDS bytes: k_rows_elements with its rows staged
  bool twice = false;  // without k: k_rows_twice
};

static Launch pick_row_kernel(grpo_dtype dt, int64_t T, int64_t V, int64_t ld, const void* logits,
                              const void* dlogits, hipStream_t s) {
  const int epv = (dt == GRPO_BF16) ? 8 : 4;
  // fp32 rows that are not whole aligned vectors keep the element kernel and with it the order of their fp32 sums (column
  // classes modulo 256).  The ragged vector kernels' order is no less exact, but it moves the small dlogits of a
  // near-certain token by up to 5e-4 of the root mean square; nothing here reads such rows by vectors in the old order.
  RowForm form = row_form(logits, dlogits, V, ld, 16 / epv);
  if (dt == GRPO_F32 && form == RowForm::kRagged) form = RowForm::kElements;
  const int rag = form == RowForm::kRagged;
  if (form != RowForm::kElements) {
    const int64_t nvec = V / epv;  // the most a row has
    const int64_t nv = (nvec + 1023) / 1024;
    RowKernel k = nullptr;
    int n_cu = stream_cu_count(s);  // of the stream's device
    if (n_cu < 1) n_cu = 256;
    if (T <= kPipeMaxT) {
      if (dt == GRPO_BF16 && nv >= kPipeMinNV && nv <= kPipeMaxNV) k = kPipe[nv - kPipeMinNV][rag];
      else if (dt == GRPO_BF16 && nv > kPipeMaxNV && nvec * 16 <= kStreamMaxRow &&
               (dlogits || !records_without_dlogits(dt, T, V, n_cu)))
        k = kStreamRows[rag];
    }
    if (k) {
      // chunks of up to 8 rows (1.6-2.5% faster than single rows at 120,000 x 151,936), but at least four chunks
      // per CU, so that small batches still spread over the chip
      const int64_t chunk = std::max<int64_t>(1, std::min<int64_t>(8, T / (4 * (int64_t)n_cu)));
      const int64_t n_chunks = (T + chunk - 1) / chunk;
      const int64_t g = n_chunks < n_cu ? n_chunks : n_cu;  // one workgroup per CU (LDS bound)
      // whole rounds of chunks, then the remaining rows split evenly: at T = 120,000 the busiest workgroup has
      // 469 rows instead of 472
      const int64_t r0 = T / (chunk * g) * (chunk * g);
      const int64_t chunk2 = std::max<int64_t>(1, (T - r0 + g - 1) / g);
      return Launch{k, 1024, (unsigned)g, (int)chunk, (int)r0, (int)chunk2};
    }
    for (const Variant& v : kVariants) {
      const RowKernel fits = dt == GRPO_BF16 ? v.bf16[rag] : v.f32;
      if (fits && (int64_t)v.nt * v.nv >= nvec) return Launch{fits, v.nt, (unsigned)T};
    }
    Launch l{nullptr, 0, 0};  // two passes, or fp32 rows in one
    l.twice = dt == GRPO_F32 && rows_twice(T, V, n_cu) && (dlogits || !records_without_dlogits(dt, T, V, n_cu));
    return l;
  }
  // staged in LDS where two workgroups fit a CU: alone on its CU, 256 threads took 0.96 ms at fp32 10,000 x 32,003
  // against 0.80 with every sweep from memory
  const int64_t bytes = V * (16 / epv);
  const bool staged = V > 256 * kHeldElements && bytes <= 79 * 1024;
  Launch l{dt == GRPO_BF16 ? element_kernel<uint16_t>(V) : element_kernel<float>(V), 256, (unsigned)T};
  if (staged) l.lds = (unsigned)bytes;
  return l;
}

}  // namespace grpo

using namespace grpo;

extern "C" size_t grpo_loss_workspace_bytes(int64_t T, int32_t n_traj) {
  if (T < 0 || T >= ((int64_t)1 << 31) || n_traj < 1) return 0;  // the loss entry points refuse T >= 2^31
  return loss_ws_layout(T, n_traj).total;
}

// Argument checks of the logits path other than the workspace's (GRPO_OK or the error).
static int check_logits_call(const void* logits, int32_t dt, int64_t T, int64_t V, int64_t ld,
                             const int32_t* actions, const float* behave_logp, const float* adv,
                             const grpo_segments* seg, const grpo_loss_params* p, const double* loss_out,
                             const void* dlogits) {
  int st = check_loss_common(T, actions, behave_logp, adv, seg, p, loss_out);
  if (st != GRPO_OK) return st;
  if (dt != GRPO_BF16 && dt != GRPO_F32) return GRPO_ERR_DTYPE;
  if (T > 0 && !logits) return GRPO_ERR_ARG;
  if (V < 1 || ld < V || V >= ((int64_t)1 << 31)) return GRPO_ERR_SHAPE;
  const size_t esz = (dt == GRPO_BF16) ? 2 : 4;
  if (!aligned(logits, esz) || !aligned(dlogits, esz)) return GRPO_ERR_ALIGN;
  return GRPO_OK;
}

extern "C" int grpo_loss_fwd_bwd(const void* logits, int32_t dtype, int64_t T, int64_t V, int64_t ld,
                                 const int32_t* actions, const float* behave_logp, const float* prox_logp,
                                 const float* adv, const grpo_segments* seg, const grpo_loss_params* p,
                                 double* loss_out, void* dlogits, grpo_aux* aux, void* ws, size_t ws_bytes,
                                 hipStream_t s) {
  const int st = check_logits_call(logits, dtype, T, V, ld, actions, behave_logp, adv, seg, p, loss_out, dlogits);
  if (st != GRPO_OK) return st;
  const grpo_dtype dt = static_cast<grpo_dtype>(dtype);
  const LossWs L = loss_ws_layout(T, seg->n_traj);
  if (!ws || ws_bytes < L.total) return GRPO_ERR_WORKSPACE;
  if (!aligned(ws, kAlign)) return GRPO_ERR_ALIGN;
  char* w = static_cast<char*>(ws);

  if (launch_segments(seg, T, ld, actions, adv, p, w, L, aux, s) != hipSuccess) return GRPO_ERR_HIP;
  if (T > 0) {
    RowArgs a;
    a.logits = logits;
    a.dlogits = dlogits;
    a.ld = ld;
    a.T = (int)T;
    a.tok = make_token_args(V, actions, behave_logp, prox_logp, adv, p, w, L, aux);
    const Launch k = pick_row_kernel(dt, T, V, ld, logits, dlogits, s);
    a.chunk = k.chunk;
    a.r0 = k.r0;
    a.chunk2 = k.chunk2;
    a.staged = k.lds > 0;
    const bool timed = aux && aux->hot_begin && aux->hot_end;
    if (timed && hipEventRecord(aux->hot_begin, s) != hipSuccess) return GRPO_ERR_HIP;
    if (k.k) {
      hipLaunchKernelGGL(k.k, dim3(k.grid), dim3(k.nt), k.lds, s, a);
      if (hipGetLastError() != hipSuccess) return GRPO_ERR_HIP;
    } else if (k.twice) {
      if (launch_rows_twice(logits, dlogits, T, ld, a.tok, s) != hipSuccess) return GRPO_ERR_HIP;
    } else {
      // the whole vocabulary as one shard: its records, then the merge (trivial), epilogue and dlogits
      grpo_vocab_stats* rec = reinterpret_cast<grpo_vocab_stats*>(w + L.records);
      int32_t* flags = &reinterpret_cast<WsHeader*>(w + L.hdr)->flags;
      if (launch_vocab_records(logits, dt, T, V, ld, 0, actions, rec, flags, s) != hipSuccess) return GRPO_ERR_HIP;
      if (launch_shard_rows(logits, dlogits, dt, T, V, ld, 0, rec, 1, a.tok, s) != hipSuccess) return GRPO_ERR_HIP;
    }
    if (timed && hipEventRecord(aux->hot_end, s) != hipSuccess) return GRPO_ERR_HIP;
  }
  if (launch_reduce(T, seg->n_traj, w, L, loss_out, aux, s) != hipSuccess) return GRPO_ERR_HIP;
  return GRPO_OK;
}

// ---- the logits path without a caller workspace ------------------------------------
// For callers that cannot allocate device memory, the workspace is a file-scope device array of fixed size.
// Each device the library runs on holds its own copy until the process ends; host code reaches it only through
// the address hipGetSymbolAddress returns on that device, looked up once per device and kept.
static __device__ __align__(256) char scratch[GRPO_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch[kMaxDevices];  // device address of `scratch` per device (nullptr until its first call)
}  // namespace

// The scratch array's address on the stream's device: looked up with that device current on the device's first
// call, then read from the table.
static int scratch_of_stream(hipStream_t s, char** out) {
  hipDevice_t dev = 0;
  if (hipStreamGetDevice(s, &dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return GRPO_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess) return GRPO_ERR_HIP;
    if (cur != dev && hipSetDevice(dev) != hipSuccess) return GRPO_ERR_HIP;
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != dev && hipSetDevice(cur) != hipSuccess) return GRPO_ERR_HIP;
    if (e != hipSuccess || !ptr) return GRPO_ERR_HIP;
    g_scratch[dev] = static_cast<char*>(ptr);
  }
  *out = g_scratch[dev];
  return GRPO_OK;
}

extern "C" int grpo_loss_fwd_bwd_noalloc(const void* logits, int32_t dt, int64_t T, int64_t V, int64_t ld,
                                         const int32_t* actions, const float* behave_logp, const float* prox_logp,
                                         const float* adv, const grpo_segments* seg, const grpo_loss_params* p,
                                         double* loss_out, void* dlogits, grpo_aux* aux, hipStream_t s) {
  const int st = check_logits_call(logits, dt, T, V, ld, actions, behave_logp, adv, seg, p, loss_out, dlogits);
  if (st != GRPO_OK) return st;
  if (loss_ws_layout(T, seg->n_traj).total > (size_t)GRPO_NOALLOC_SCRATCH_BYTES) return GRPO_ERR_WORKSPACE;
  char* ws = nullptr;
  const int sc = scratch_of_stream(s, &ws);
  if (sc != GRPO_OK) return sc;
  return grpo_loss_fwd_bwd(logits, dt, T, V, ld, actions, behave_logp, prox_logp, adv, seg, p, loss_out, dlogits,
                           aux, ws, (size_t)GRPO_NOALLOC_SCRATCH_BYTES, s);
}
