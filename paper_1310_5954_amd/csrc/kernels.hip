// HIP kernels of the local ETKF frame (gfx950).
//
//   k_slopes    a3: Y' = D X'_phi and d = y - D xbar_phi, one thread per
//               (slope row, member), row means by wavefront shuffles.
//   k_rows      a1/a2/a8-merge: weighted merge of the per-domain analysis
//               rows into the ensemble, optionally fused with the AR forecast
//               (Philox4x32-10 + Box-Muller model noise) and the output means.
//   k_analysis_poly  a4-a8: one workgroup per domain: gather, C and b, A^(-1/2)
//               by polynomial stages on the FP64 matrix cores, wbar, T, update.
//   k_analysis  the same with an FP64 one-sided Jacobi eigensolver in LDS, for
//               the instances the stages do not serve (InstDesc::poly).
//
// All kernels walk the entries of one batch class (same padded ensemble size
// and storage precision) so that frames of several instances share a launch.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "desc.hpp"
#include "isqrt_plan.hpp"
#include "launch.hpp"

namespace letkf {

static_assert(kIsqrtEntries == kStageEntries, "stage_guess's range is the table's");

// ----------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11) and one Box-Muller normal per counter.
// ----------------------------------------------------------------------------
__device__ __forceinline__ double philox_normal(uint64_t seed, uint64_t frame, uint32_t act,
                                                uint32_t member) {
  uint32_t c0 = member, c1 = act, c2 = (uint32_t)frame, c3 = (uint32_t)(frame >> 32);
  uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c0), lo0 = 0xD2511F53u * c0;
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c2), lo1 = 0xCD9E8D57u * c2;
    const uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
    c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
  }
  const uint64_t v1 = ((uint64_t)c0 << 21) | (c1 >> 11);
  const uint64_t v2 = ((uint64_t)c2 << 21) | (c3 >> 11);
  const double u1 = ((double)v1 + 0.5) * 0x1.0p-53;
  const double u2 = ((double)v2 + 0.5) * 0x1.0p-53;
  return sqrt(-2.0 * log(u1)) * cospi(2.0 * u2);
}

// Loads through a pointer into device memory taken from a descriptor.  Such a
// pointer is generic, and a generic (flat) load also counts against the LDS
// counter, so every LDS wait (s_waitcnt lgkmcnt) after a prefetch would wait
// for the prefetch too.  Reading through the global address space makes it a
// global load that only the vector-memory counter tracks.
template <typename T>
__device__ __forceinline__ T gload(const T* p) {
  return *(const __attribute__((address_space(1))) T*)p;
}
// The same for stores (a flat store also holds up the next LDS wait).
template <typename T>
__device__ __forceinline__ void gstore(T* p, T v) {
  *(__attribute__((address_space(1))) T*)p = v;
}
// ... and for device-scope atomic adds whose result is not used.
template <typename T>
__device__ __forceinline__ void gatomic_add(T* p, T v) {
  (void)__hip_atomic_fetch_add((__attribute__((address_space(1))) T*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Cross-lane moves of a double with DPP (VALU, no LDS round trip).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  // Every pattern used here reads a valid lane, so no "old" value is needed.
  const long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(x >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Sum over aligned groups of G consecutive lanes (G = 2, 4, 8 or 16); every
// lane of a group ends with the group total.  Stages: swap neighbours, swap
// pairs (quad permutes), then mirror within 8 and within 16 lanes.
template <int G>
__device__ __forceinline__ double group_sum(double v) {
  if constexpr (G >= 2) v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
  if constexpr (G >= 4) v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
  if constexpr (G >= 8) v += dpp_f64<0x141>(v);  // row_half_mirror
  if constexpr (G >= 16) v += dpp_f64<0x140>(v); // row_mirror
  static_assert(G <= 16, "group_sum supports up to 16 lanes");
  return v;
}

// Sum of v over the MP lanes of a member row (MP <= 64: one wavefront segment;
// MP >= 128: wavefronts combined through LDS).  Every thread participates.
// Within 16 lanes by DPP (group_sum), across 16-lane rows by lane shuffles.
template <int MP>
__device__ __forceinline__ double row_sum(double v, double* red) {
  constexpr int W = MP < 64 ? MP : 64;
  v = group_sum<(W < 16 ? W : 16)>(v);
#pragma unroll
  for (int off = 16; off < W; off <<= 1) v += __shfl_xor(v, off, 64);
  if constexpr (MP > 64) {
    const int t = threadIdx.x;
    if ((t & 63) == 0) red[t >> 6] = v;
    __syncthreads();
    const int base = (t / MP) * (MP / 64);
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < MP / 64; ++w) s += red[base + w];
    __syncthreads();
    v = s;
  }
  return v;
}

__device__ __forceinline__ int find_entry(const int32_t* off, int n, int g) {
  int b = 0;
  while (b + 1 < n && off[b + 1] <= g) ++b;
  return b;
}

template <typename T> __device__ __forceinline__ double ld(const T* p) { return (double)*p; }
template <typename T> __device__ __forceinline__ void st(T* p, double v) { *p = (T)v; }

// ----------------------------------------------------------------------------
// a3: slope perturbations and innovation of every slope row of the class,
// Y' = D X'_obs and d = y - D xbar_obs, X_obs the observed instant's rows.
// ----------------------------------------------------------------------------
//
// These row kernels move little (20 MB at 84 x 84, m = 64) and are bound by a
// row's chain of dependent loads (entry, descriptor, index, value), so a row's
// indices and its values are loaded by fours (kRowBatch) rather than one nonzero
// at a time, and the descriptor comes through scalar loads where a workgroup's
// rows share an entry (all but those astride two instances of a batch).
// 84 x 84, m = 64 BF16: k_slopes 15.9 -> 12.5 us, k_rows 19.0 -> 15.5 us;
// 128 x 128, m = 128: 46 -> 33 and 51 -> 40 us.
constexpr int kRowBatch = 4;

// Calls body(b) with the batch entry of row g: a scalar where all rows of the
// workgroup (base .. base + rows - 1, of total) have the same one.
template <typename F>
__device__ __forceinline__ void with_entry(const int32_t* off, int n, int base, int rows, int total, int g, F&& body) {
  const int b0 = __builtin_amdgcn_readfirstlane(find_entry(off, n, base));
  if (off[b0 + 1] >= min(base + rows, total)) body(b0);
  else body(find_entry(off, n, g < total ? g : 0));
}

template <typename T, int MP>
__global__ __launch_bounds__(256) void k_slopes(const InstDesc* __restrict__ tab,
                                                BatchHdr* __restrict__ hdr, int cls, const double* y) {
  constexpr int RPB = 256 / MP > 0 ? 256 / MP : 1;
  __shared__ double red[4];
  ClassBatch& cb = hdr->cls[cls];
  if (blockIdx.x == 0) {
    if ((int)threadIdx.x < cb.n) tab[cb.inst[threadIdx.x]].st->unconverged = 0;
    if (threadIdx.x == 0) cb.next = cb.next_poly = 0;  // the analysis launch that follows claims items from zero
  }
  const int j = threadIdx.x % MP;
  const int total = cb.slope_off[cb.n];
  // grid-stride over row groups (the trip count is uniform within a block)
  for (int base = blockIdx.x * RPB; base < total; base += gridDim.x * RPB) {
    const int g = base + threadIdx.x / MP;
    const bool active = g < total;
    with_entry(cb.slope_off, cb.n, base, RPB, total, g, [&](int b) {
      const InstDesc& I = tab[cb.inst[b]];
      const int m = I.m;
      const int o = g - cb.slope_off[b];
      double v = 0.0, yo = 0.0;
      if (active && j == 0) yo = gload((y ? y : hdr->yptr[cb.ent[b]]) + o);
      if (active && j < m) {
        // the observed instant: phi_k (ring slot cur) or phi_{k-1} (H = [0 D])
        const T* ens = (const T*)I.ens + (size_t)(I.st->cur ^ I.obs_inst) * I.n_act * m;
        const int k1 = gload(I.d_rowptr + o + 1);
        for (int k = gload(I.d_rowptr + o); k < k1; k += kRowBatch) {
          int col[kRowBatch];
          double w[kRowBatch], x[kRowBatch];
#pragma unroll
          for (int u = 0; u < kRowBatch; ++u) {
            const int q = k + u < k1 ? k + u : k;
            col[u] = gload(I.d_col + q);
            w[u] = gload(I.d_val + q);
          }
#pragma unroll
          for (int u = 0; u < kRowBatch; ++u) x[u] = (double)gload(ens + (size_t)col[u] * m + j);
#pragma unroll
          for (int u = 0; u < kRowBatch; ++u)
            if (k + u < k1) v += w[u] * x[u];
        }
      }
      const double ybar = row_sum<MP>(v, red) / (double)m;
      if (active) {
        if (j < m) gstore((T*)I.Yp + (size_t)o * m + j, (T)(v - ybar));
        if (j == 0) {
          gstore(I.d + o, yo - ybar);
          // read elsewhere: kept where a later launch of this frame's slopes (autotune) looks
          if (y) gstore((double*)hdr->yptr[cb.ent[b]] + o, yo);
          if (hdr->check_y && !isfinite(yo)) hdr->bad[cb.ent[b]] = 1;  // every writer stores the same value
        }
      }
    });
  }
}

// ----------------------------------------------------------------------------
// a8 merge and/or a1 forecast, per actuator row (both time instants).
//   MODE 0: merge only         -> ensemble = analysis, amean
//   MODE 1: forecast only      -> phi_{k+1} into the lagged slot, pmean, advance
//   MODE 2: merge + forecast   -> both, amean and pmean, advance
// ----------------------------------------------------------------------------
template <typename T, int MP, int MODE>
__global__ __launch_bounds__(256) void k_rows(const InstDesc* __restrict__ tab,
                                              BatchHdr* __restrict__ hdr, int cls) {
  constexpr int RPB = 256 / MP > 0 ? 256 / MP : 1;
  __shared__ double red[4];
  ClassBatch& cb = hdr->cls[cls];
  const int j = threadIdx.x % MP;
  const int total = cb.act_off[cb.n];
  // grid-stride over row groups (the trip count is uniform within a block)
  for (int base = blockIdx.x * RPB; base < total; base += gridDim.x * RPB) {
    const int g = base + threadIdx.x / MP;
    const bool active = g < total;
    with_entry(cb.act_off, cb.n, base, RPB, total, g, [&](int b) {
      const InstDesc& I = tab[cb.inst[b]];
      const int m = I.m;
      const int a = g - cb.act_off[b];
      const int cur = I.st->cur, ent = cb.ent[b];
      const size_t slot = (size_t)I.n_act * m;
      T* ens = (T*)I.ens;
      T* e_cur = ens + (size_t)cur * slot;
      T* e_prev = ens + (size_t)(cur ^ 1) * slot;
      // an entry whose slopes were not finite keeps its ensemble (group-uniform:
      // the MP lanes of a row share the entry)
      const bool skip = hdr->check_y && hdr->bad[ent];
      const bool live = active && j < m && !skip;
      double vk = 0.0, vkm1 = 0.0;
      if (live) {
        if (MODE == 1) {
          vk = (double)gload(e_cur + (size_t)a * m + j);
          vkm1 = (double)gload(e_prev + (size_t)a * m + j);
        } else {
          const T* Z = (const T*)I.Z;
          const int q1 = gload(I.mptr + a + 1);
          for (int q = gload(I.mptr + a); q < q1; q += kRowBatch) {
            int r0[kRowBatch], r1[kRowBatch];
            double w[kRowBatch], z0[kRowBatch], z1[kRowBatch];
#pragma unroll
            for (int u = 0; u < kRowBatch; ++u) {
              const int x = q + u < q1 ? q + u : q;
              w[u] = gload(I.mw + x);
              r0[u] = gload(I.mrow + 2 * x);
              r1[u] = gload(I.mrow + 2 * x + 1);
            }
#pragma unroll
            for (int u = 0; u < kRowBatch; ++u) {
              z0[u] = (double)gload(Z + (size_t)r0[u] * m + j);
              z1[u] = (double)gload(Z + (size_t)r1[u] * m + j);
            }
            if (I.pist_c) {  // differential pistons of the covering domain (both instants)
#pragma unroll
              for (int u = 0; u < kRowBatch; ++u) {
                const double* c = I.pist_c + (size_t)gload(I.mdom + (q + u < q1 ? q + u : q)) * 2 * m;
                z0[u] += gload(c + j);
                z1[u] += gload(c + m + j);
              }
            }
#pragma unroll
            for (int u = 0; u < kRowBatch; ++u)
              if (q + u < q1) {
                vk += w[u] * z0[u];
                vkm1 += w[u] * z1[u];
              }
          }
          // stored value (rounded to the storage type) is what the forecast uses
          vk = (double)(T)vk;
          vkm1 = (double)(T)vkm1;
          gstore(e_cur + (size_t)a * m + j, (T)vk);
          if (MODE == 0) gstore(e_prev + (size_t)a * m + j, (T)vkm1);
        }
      }
      if (MODE != 1) {
        const double s = row_sum<MP>(live ? vk : 0.0, red);
        if (active && !skip && j == 0) gstore(hdr->amean + hdr->out_off[ent] + a, s / (double)m);
      }
      if (MODE != 0) {
        double nx = 0.0;
        if (live) {
          nx = gload(I.a1 + a) * vk + gload(I.a2 + a) * vkm1;
          if (I.sigma_v != 0.0) nx += I.sigma_v * philox_normal(I.seed, I.st->frame, (uint32_t)a, (uint32_t)j);
          nx = (double)(T)nx;
          gstore(e_prev + (size_t)a * m + j, (T)nx);
        }
        const double s = row_sum<MP>(nx, red);
        if (active && !skip && j == 0) gstore(hdr->pmean + hdr->out_off[ent] + a, s / (double)m);
      }
    });
  }
}

// ---- Differential pistons (Sec. 3.2), between the analysis and the merge ----
// One workgroup per (instance, domain) work item, thread (t, i) for instant t
// and member i.  k_piston_rhs: the overlap mismatch
//   r_l[t, i] = sum over the domain's actuators j of
//               (sum of the covering domains' rows at j) - k_j (own row at j),
// k_piston_solve: c_l = sum_l' G[l, l'] r_l' with the host-formed operator G.
// Instances created without LETKF_FLAG_PISTONS are skipped.
template <typename T>
__global__ __launch_bounds__(256) void k_piston_rhs(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr,
                                                    int cls) {
  const ClassBatch& cb = hdr->cls[cls];
  const int total = cb.dom_off[cb.n], tid = threadIdx.x;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int eb = find_entry(cb.dom_off, cb.n, item);
    const InstDesc& I = tab[cb.inst[eb]];
    const int m = I.m;
    if (!I.pist_op || tid >= 2 * m) continue;
    const int l = item - cb.dom_off[eb], t = tid / m, i = tid % m;
    const T* Z = (const T*)I.Z;
    // terms precomputed at create (row, coefficient): independent loads
    double acc[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc[u] = 0.0;
    const int q0 = I.pist_ptr[l], q1 = I.pist_ptr[l + 1];
    int q = q0;
    for (; q + 8 <= q1; q += 8)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        acc[u] = fma(I.pist_coef[q + u], ld(Z + (size_t)I.pist_row[2 * (q + u) + t] * m + i), acc[u]);
    for (; q < q1; ++q) acc[0] = fma(I.pist_coef[q], ld(Z + (size_t)I.pist_row[2 * q + t] * m + i), acc[0]);
    double rsum = 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) rsum += acc[u];
    I.pist_r[((size_t)l * 2 + t) * m + i] = rsum;
  }
}

__global__ __launch_bounds__(256) void k_piston_solve(const InstDesc* __restrict__ tab,
                                                      const BatchHdr* __restrict__ hdr, int cls) {
  const ClassBatch& cb = hdr->cls[cls];
  const int total = cb.dom_off[cb.n], tid = threadIdx.x;
  for (int item = blockIdx.x; item < total; item += gridDim.x) {
    const int eb = find_entry(cb.dom_off, cb.n, item);
    const InstDesc& I = tab[cb.inst[eb]];
    const int m = I.m;
    if (!I.pist_op || tid >= 2 * m) continue;
    const int l = item - cb.dom_off[eb], t = tid / m, i = tid % m, n = I.n_dom;
    const double* g = I.pist_op + (size_t)l * n;
    // 16 independent partial sums keep that many L2 loads in flight
    double acc[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) acc[u] = 0.0;
    const double* r = I.pist_r + (size_t)t * m + i;
    int k = 0;
    for (; k + 16 <= n; k += 16)
#pragma unroll
      for (int u = 0; u < 16; ++u) acc[u] = fma(g[k + u], r[(size_t)(k + u) * 2 * m], acc[u]);
    for (; k < n; ++k) acc[0] = fma(g[k], r[(size_t)k * 2 * m], acc[0]);
    double c = 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) c += acc[u];
    I.pist_c[((size_t)l * 2 + t) * m + i] = c;
  }
}

__device__ __forceinline__ void advance_class(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr, int cls,
                                              int threads) {
  const ClassBatch& cb = hdr->cls[cls];
  for (int e = threadIdx.x; e < cb.n; e += threads) {
    if (hdr->check_y && hdr->bad[cb.ent[e]]) continue;  // the frame was refused: nothing advanced
    InstState* S = tab[cb.inst[e]].st;
    S->cur ^= 1;
    S->frame += 1;
  }
}

// After a forecast launch: the new instant becomes phi_k (ring swap) and the
// frame counter advances, for every instance of the class.  A launch of its
// own, ordered after k_rows on the stream, instead of a "last block" counter
// in k_rows: a completion counter that every block of k_rows increments
// serialises on one address and cost more than the whole merge.
__global__ __launch_bounds__(64) void k_advance(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr,
                                                int cls) {
  advance_class(tab, hdr, cls, 64);
}

// A frame whose caller waits for its means: they are stored to the caller's
// pinned host buffer by the launch that ends the frame (one workgroup, 16-byte
// stores: the row kernel's single means would cross the bus eight bytes at a
// time), where a copy command of its own is one more dependent packet.
// With the slopes read in place a frame of the 15 x 15 map went from 55.4 to
// 49.3 us, one of the 32 x 32 global domain from 320 to 297 us.
__global__ __launch_bounds__(1024) void k_finish(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr,
                                                 int cls, int advance, const double* __restrict__ mean,
                                                 double* __restrict__ host, int n) {
  typedef double pair __attribute__((ext_vector_type(2)));
  if (advance) advance_class(tab, hdr, cls, 1024);
  for (int i = 2 * threadIdx.x; i + 1 < n; i += 2048) gstore((pair*)(host + i), gload((const pair*)(mean + i)));
  if ((n & 1) && threadIdx.x == 0) gstore(host + n - 1, gload(mean + n - 1));
}

// ----------------------------------------------------------------------------
// a4-a8: per-domain analysis, one workgroup per domain (256 threads; 512 where
// its matrices fill the LDS of a CU, M = 128).
//
// P selects the contraction path: 0 = FP64, 1 = FP32 MFMA
// (v_mfma_f32_16x16x4f32), 2 = BF16 MFMA (v_mfma_f32_16x16x32_bf16) with FP32
// accumulation, 3 = the BF16 path with its Jacobi rotations in FP32 (an
// opt-in variant, LETKF_FLAG_FP32_ROTATIONS).  The eigensolve, wbar and W are
// FP64 on paths 0-2; path 3 rotates in FP32 and keeps the Cholesky, lambda,
// wbar and W in FP64.  On the BF16 paths C uses split operands (hi + lo, three
// products): a single BF16 rounding of sqrt(r) Y' perturbs C by ~1e-3 of its
// largest eigenvalue, which exceeds the smallest ones ((m-1)/rho) that
// dominate W.
// ----------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The thread index as a value the compiler may not move: every phase of the
// analysis derives its index arithmetic from it afresh.  Otherwise, inside the
// persistent item loop, the arithmetic of all phases (invariant across items)
// is hoisted out of the loop and stays live through the whole body, which
// costs registers and so occupancy.
__device__ __forceinline__ int phase_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// What the gathers and updates take from a configuration of M padded members and
// NT_ threads.
template <int M_, int NT_> struct StageCfg {
  static constexpr int M = M_, NT = NT_, NW = NT / 64;
  // the products that form C: the wavefronts as a WR x WC grid, each with
  // TR x TC tiles of 16 x 16 (one wavefront only at M = 16)
  static constexpr int TILES = M / 16;
  static constexpr int WC = TILES >= 2 ? 2 : 1, WR = TILES >= 2 ? NW / 2 : 1;
  static constexpr int TR = TILES / WR, TC = TILES / WC;
  static constexpr int KCD = 16, LDKD = KCD + 1;   // FP64: observations per chunk; an odd row stride puts the 16 rows of an operand load in 16 bank pairs
  static constexpr int KCF = M <= 64 ? 32 : 16;    // FP32: observations per staged chunk
  // row stride (floats) of the transposed chunk: 2 mod 32, so that the 16 rows
  // and 2 k-offsets of a 32-lane operand load fall in 32 different banks
  static constexpr int LDKF = KCF + 2;
  static constexpr int KCB = 32;                   // BF16: observations per chunk (one k-step)
  static constexpr int LDKB = KCB + 8;             // row stride (bf16) of the transposed chunk
  static constexpr int KR = M <= 64 ? 32 : 16;     // update: state rows per chunk (16-row tiles)
  // threads that hold partial sums of b, of norms and of products with a vector
  static constexpr int RT = NT;
};

// k_analysis: 256 threads, 512 at M = 128, where one workgroup fills the LDS of a
// CU and 256 threads are one wavefront per SIMD: nothing overlaps a wavefront's
// LDS traffic, and 32 rows a lane leave no registers to load the next column
// ahead.  RT: sums over threads keep the order of 256 of them.
// 128 x 128 map, m = 128, BF16: the analysis launch 4.70 -> 3.83 ms.
template <int M> struct AnaCfg : StageCfg<M, M <= 64 ? 256 : 512> {
  using B = StageCfg<M, M <= 64 ? 256 : 512>;
  using B::NT;
  using B::KCF;
  using B::LDKF;
  using B::LDKB;
  using B::KR;
  static constexpr int RT = 256;
  static constexpr int KC = 16;                    // FP64 path: rows per staged chunk (keeps m = 64 at 3 workgroups/CU)
  // a thread's outputs where M x M entries are formed on vector FMA: TX x TM, rows
  // row0 + 16 x and columns tid % 16 + 16 y
  static constexpr int TM = M / 16, TX = TM * 256 / NT;
  static constexpr __device__ int row0(int tid) { return NT == 256 ? tid / 16 : tid / 16 % 16 + 16 * TX * (tid / 256); }
  static constexpr int TPP = (2 * NT / M) < M ? (2 * NT / M) : M;  // threads per Jacobi pair
  // Column stride of the M x M matrix in LDS: shifting consecutive columns by
  // one pair-group span (min(TPP, 8) doubles) spreads the pair groups of a
  // wavefront over all banks in every Jacobi step.
  static constexpr int LDB = M + (TPP < 8 ? TPP : 8);
  static constexpr int ACTIVE = (M / 2) * TPP;
  static constexpr int RPT = M / TPP;              // rows per thread in a Jacobi step
  static constexpr int MAX_SWEEPS = 40;
  static constexpr size_t STAGE_BYTES = [] {
    size_t a = (size_t)KC * M * 8, b = (size_t)M * LDKF * 4, c = (size_t)M * LDKB * 2 * 2, d = (size_t)KR * M * 4;
    size_t x = a > b ? a : b;
    x = x > c ? x : c;
    return x > d ? x : d;
  }();
};

// The chunk staging of the gather and the update (phase-dependent type), and the
// vectors of the transform between the two: in one place at M = 128, where LDS
// has no room for both.
template <int M> struct AnaStage {
  alignas(16) unsigned char stage[AnaCfg<M>::STAGE_BYTES];
  double lam[M], zv[M], pcol[2][M];
};
template <> struct AnaStage<128> {
  union {
    alignas(16) unsigned char stage[AnaCfg<128>::STAGE_BYTES];
    struct {
      double lam[128], zv[128], pcol[2][128];
    };
  };
};
// The matrix ahead of them: at LDS address 0 a column's or a partner's offset is
// its address (behind the staging the Jacobi steps spent an add on every other
// one: m = 32 FP32 launches of 8 instances 85.8 -> 88.2 us).
template <int M> struct AnaMatrix {
  double Bm[M * AnaCfg<M>::LDB];                      // A, then U, then T (row-major)
};
template <int M> struct AnaSmem : AnaMatrix<M>, AnaStage<M> {
  using C = AnaCfg<M>;
  using AnaMatrix<M>::Bm;
  using AnaStage<M>::stage;
  static constexpr int LDA = C::LDB;                  // the gathers' stride of A
  static __device__ double pad(double) { return 1.0; }  // diagonal of A past m
  double rc[32], dc[32];
  double bvec[M], nrm[M], wbar[M];
  int perm[M <= 64 ? M : 1];                          // FP64, M <= 64: A's symmetric permutation
  int s_rot;
  __device__ double* red() { return (double*)stage; }  // NT partial sums, aliases the staging area
};

// k_analysis_poly: a wavefront per 16 columns of the M x M matrices, at least four.
template <int M> struct PolyCfg : StageCfg<M, M <= 64 ? 256 : 512> {
  using B = StageCfg<M, M <= 64 ? 256 : 512>;
  static constexpr int LDB = M + (M <= 64 ? 8 : 4);  // column stride of Z and T in LDS
  static constexpr int LDA = M + 2;                  // of A and the stages' left factors
  // tiles of Z, of T, that stay in registers (isqrt_stages)
  static constexpr int keep(int T) { return T <= 3 ? T : T == 4 ? 2 : T == 5 ? 4 : T == 6 ? 3 : T == 7 ? 0 : 1; }
  static constexpr size_t STAGE_BYTES = [] {
    size_t x = 0;
    for (size_t v : {(size_t)M * B::LDKD * 8, (size_t)16 * (M + 1) * 8,
                     (size_t)B::NT * 8, M == 64 ? (size_t)B::NT * 8 * 4 * 2 - (size_t)M * (LDB - LDA) * 8 : 0})  // parked Z, behind A
      x = v > x ? v : x;
    return (x + 15) & ~size_t(15);
  }();
};
template <int M> struct PolySmem {
  using C = PolyCfg<M>;
  static constexpr int LDA = C::LDA;
  // diagonal of A past m (the stages put the mean eigenvalue there)
  static __device__ double pad(double a_diag) { return a_diag; }
  alignas(16) double Bm[M * C::LDB];                  // A, the stages' left factors, Z, then T (row-major)
  alignas(16) unsigned char stage[C::STAGE_BYTES];    // chunk staging (phase-dependent type)
  double rc[32];
  double bvec[M], zv[M], wbar[M], pcol[M];
  __device__ double* red() { return (double*)stage; }  // NT partial sums, aliases the staging area
};

// The entry (i, j) of A = (m-1)/rho I + C into LDS at (i, j) only: for the FP64
// gather, whose 16 tiles cover both halves and compute C_ij and C_ji with the
// same products summed in the same order (bitwise equal), so every entry is
// written once and along rows (the mirrored write went down a column, an 8-way
// bank conflict).
template <typename SM>
__device__ __forceinline__ void put_A_own(SM& sm, int i, int j, int m, double c, double a_diag, double* dbg) {
  double v = c;
  if (i >= m || j >= m) v = (i == j) ? SM::pad(a_diag) : 0.0;
  else {
    if (dbg) dbg[i * m + j] = c;
    if (i == j) v += a_diag;
  }
  sm.Bm[i * SM::LDA + j] = v;
}

// Writes the entry (i, j) of A = (m-1)/rho I + C into LDS (symmetrically: only
// the producer of i <= j writes, to both halves), padded members -> SM::pad on
// the diagonal.
template <typename SM>
__device__ __forceinline__ void put_A(SM& sm, int i, int j, int m, double c, double a_diag, double* dbg) {
  if (i > j) return;
  double v = c;
  if (i >= m || j >= m) v = (i == j) ? SM::pad(a_diag) : 0.0;
  else {
    if (dbg) { dbg[i * m + j] = c; dbg[j * m + i] = c; }
    if (i == j) v += a_diag;
  }
  sm.Bm[j * SM::LDA + i] = v;
  sm.Bm[i * SM::LDA + j] = v;
}

// ---- a4/a5 on the FP64 path: C = Y'^T diag(r) Y', b = Y'^T diag(r) d --------
// As on the MFMA paths below, a chunk of KCH observations is staged transposed
// as At[j][k] = sqrt(r_k) Y'[k][j] (FP64), and wave w owns a TR x TC block of
// 16 x 16 tiles of C, accumulated by v_mfma_f64_16x16x4f64 in FP64 registers.
// A single wavefront per SIMD issues a VALU instruction only every ~8.5
// cycles, so the matrix core reaches the FP64 rate that the FMA loop cannot.
// Lane layout of v_mfma_f64_16x16x4f64 (measured on gfx950): A[i][k] in lane
// i + 16 k, B[k][j] in lane j + 16 k, and result register v of lane l holds
// D[l / 16 + 4 v][l % 16] (rows interleaved, unlike the FP32 16x16x4 form).

template <typename SM>
__device__ __forceinline__ void gather_C_fp64_mfma(SM& sm, const InstDesc& I, int obs_off, int s, double* dbg) {
  using C = typename SM::C;
  constexpr int M = C::M;
  constexpr int NT = C::NT, KCH = C::KCD, LDK = C::LDKD;
  constexpr int TILES = C::TILES, TR = C::TR, TC = C::TC;
  double* At = (double*)sm.stage;
  const int m = I.m, tid = phase_tid(), w = tid / 64, lane = tid % 64;
  const bool wave_on = TILES >= 2 || w == 0;
  const int tr0 = TILES >= 2 ? (w / 2) * TR : 0;
  const int tc0 = TILES >= 2 ? (w % 2) * TC : 0;
  f64x4 acc[TR][TC];
#pragma unroll
  for (int a = 0; a < TR; ++a)
#pragma unroll
    for (int b = 0; b < TC; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  double bpart = 0.0;
  const double* Yp = (const double*)I.Yp;
  const int nobs = 2 * s;
  // The domain's observation table (row of Y', sqrt(r), sqrt(r) d) is staged
  // in LDS, in the space A takes only once the products are done, by segments
  // of SEG observations (one segment on the ELT maps).  The chunk loop then
  // issues only the loads of Y' rows, three chunks of them in flight: with the
  // index, r and d loads in the loop, each chunk's loads waited on the
  // previous chunk's and a chunk spent ~5k cycles for ~1k of products.
  constexpr int SEG = (M * SM::LDA * 8 / 20) / KCH * KCH;
  static_assert(SEG >= KCH && SEG % 2 == 0 && (size_t)SEG * (4 + 8 + 8) <= sizeof(sm.Bm), "observation table");
  int* rowT = reinterpret_cast<int*>(sm.Bm);
  double* sT = sm.Bm + SEG / 2;
  double* sdT = sT + SEG;
  const int32_t* obs_row = I.obs_row + 2 * obs_off;
  const double* obs_sr = I.obs_sr + 2 * obs_off;
  const double* dvec = I.d;
  // Thread (kk0 = tid / M, j = tid % M) stages observations kk0 + e NT / M of
  // every chunk for member j.
  constexpr int EPT = KCH * M / NT;
  static_assert(KCH * M % NT == 0, "whole chunks per thread");
  // M >= 64: a wavefront's lanes share kk0, so their table reads are broadcasts
  const int kk0 = M >= 64 ? __builtin_amdgcn_readfirstlane(tid / M) : tid / M, j = tid % M;
  for (int g0 = 0; g0 < nobs; g0 += SEG) {
    const int gn = nobs - g0 < SEG ? nobs - g0 : SEG;
    const int gr = (gn + KCH - 1) / KCH * KCH;
    // (the previous segment's last chunk ended with a barrier)
    for (int q = tid; q < gr; q += NT) {
      int rw = 0;
      double sr = 0.0, sd = 0.0;
      if (q < gn) {
        rw = gload(obs_row + g0 + q);
        sr = gload(obs_sr + g0 + q);
        sd = sr * gload(dvec + rw);
      }
      rowT[q] = rw;
      sT[q] = sr;
      sdT[q] = sd;
    }
    __syncthreads();
    auto fetch = [&](double (&y)[EPT], int q0) {  // Y' of chunk q0 (segment-relative)
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int q = q0 + kk0 + e * (NT / M);
        y[e] = 0.0;
        if (q < gn && j < m) y[e] = gload(Yp + (size_t)rowT[q] * m + j);
      }
    };
    auto chunk = [&](const double (&y)[EPT], double (&next)[EPT], int q0) {
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int q = q0 + kk0 + e * (NT / M);  // < gr: the table's tail is zero
        const double sy = sT[q] * y[e];
        bpart = fma(sdT[q], sy, bpart);  // r d y with r = sqrt(r)^2
        At[j * LDK + kk0 + e * (NT / M)] = sy;
      }
      __syncthreads();
      if (q0 + 2 * KCH < gn) fetch(next, q0 + 2 * KCH);
      if (wave_on) {
#pragma unroll
        for (int ks = 0; ks < KCH / 4; ++ks) {
          double av[TR], bv[TC];
#pragma unroll
          for (int a = 0; a < TR; ++a) av[a] = At[((tr0 + a) * 16 + lane % 16) * LDK + ks * 4 + lane / 16];
#pragma unroll
          for (int b = 0; b < TC; ++b) bv[b] = At[((tc0 + b) * 16 + lane % 16) * LDK + ks * 4 + lane / 16];
#pragma unroll
          for (int a = 0; a < TR; ++a)
#pragma unroll
            for (int b = 0; b < TC; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
        }
      }
      __syncthreads();
    };
    double ya[EPT], yb[EPT], yc[EPT];
    fetch(ya, 0);
    if (KCH < gn) fetch(yb, KCH);
    for (int q0 = 0; q0 < gn; q0 += 3 * KCH) {
      chunk(ya, yc, q0);
      if (q0 + KCH < gn) chunk(yb, ya, q0 + KCH);
      if (q0 + 2 * KCH < gn) chunk(yc, yb, q0 + 2 * KCH);
    }
  }
  if (wave_on) {
#pragma unroll
    for (int a = 0; a < TR; ++a)
#pragma unroll
      for (int b = 0; b < TC; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          put_A_own(sm, (tr0 + a) * 16 + lane / 16 + 4 * v, (tc0 + b) * 16 + lane % 16, m, acc[a][b][v], I.a_diag, dbg);
  }
  // b: threads sharing j = tid % M hold partial sums
  sm.red()[tid] = bpart;
  __syncthreads();
  if (tid < M) {
    double t = 0.0;
    for (int q = tid; q < NT; q += M) t += sm.red()[q];
    sm.bvec[tid] = tid < m ? t : 0.0;
  }
  __syncthreads();
}

// ---- a4/a5 on the FP32 path -------------------------------------------------
// The chunk of observations is staged transposed, At[j][k] = sqrt(r_k) Y'[k][j],
// so that C = At At^T is one MFMA product per 16 x 16 tile.  Wave w owns a
// TR x TC block of tiles.  b is accumulated in FP64 from the FP32 slopes.
template <typename SM>
__device__ __forceinline__ void gather_C_fp32(SM& sm, const InstDesc& I, int obs_off, int s, double* dbg) {
  using C = typename SM::C;
  constexpr int M = C::M;
  constexpr int NT = C::NT, ST = C::RT;
  const bool staging = ST == NT || phase_tid() < ST;
  constexpr int KCH = C::KCF;
  constexpr int TILES = C::TILES, TR = C::TR, TC = C::TC;
  const int m = I.m, tid = phase_tid(), w = tid / 64, lane = tid % 64;
  const bool wave_on = TILES >= 2 || w == 0;
  const int tr0 = TILES >= 2 ? (w / 2) * TR : 0;
  const int tc0 = TILES >= 2 ? (w % 2) * TC : 0;
  double bpart = 0.0;
  const float* Yp = (const float*)I.Yp;
  const int nobs = 2 * s;
  // Every k-step's product (4 observations) comes out of the MFMA
  // on its own and is added into an FP64 accumulator in LDS (Bm, row-major,
  // each entry owned by one lane).  A single FP32 accumulator over all p_l
  // observations carries ~sqrt(p_l / 4) 2^-24 of |C|, which the inverse square
  // root amplifies by up to kappa(A) / 2 (~1e4 on the ELT workloads).
  for (int idx = tid; idx < M * SM::LDA; idx += NT) sm.Bm[idx] = 0.0;
  // Thread (kk0 = tid / M, j = tid % M), of the first ST, stages observations
  // kk0 + e ST / M of every chunk for member j; the next chunk's rows are loaded into registers
  // before the current chunk's MFMAs, so their latency overlaps the products.
  constexpr int EPT = KCH * M / ST;
  static_assert(KCH * M % ST == 0, "whole chunks per thread");
  const int kk0 = M >= 64 ? __builtin_amdgcn_readfirstlane(tid / M) : tid / M, j = tid % M;
  float yv[EPT];
  double sv[EPT], dv[EPT];  // sqrt(r) (host-computed) and d; fetch() only issues loads
  const int32_t* obs_row = I.obs_row + 2 * obs_off;
  const double* obs_sr = I.obs_sr + 2 * obs_off;
  const double* dvec = I.d;
  auto fetch = [&](int q0) {
    // global loads (see gload), the row indices first, then what depends on them
    int row[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int q = q0 + kk0 + e * (ST / M);
      row[e] = (q < nobs && j < m) ? gload(obs_row + q) : -1;
      sv[e] = q < nobs ? gload(obs_sr + q) : 0.0;
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      yv[e] = 0.f;
      dv[e] = 0.0;
      if (row[e] >= 0) {
        dv[e] = gload(dvec + row[e]);
        yv[e] = gload(Yp + (size_t)row[e] * m + j);
      }
    }
  };
  if (staging) fetch(0);
  for (int q0 = 0; q0 < nobs; q0 += KCH) {
    if (staging)
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int kk = kk0 + e * (ST / M);
      const double y = (double)yv[e];
      const double sy = sv[e] * y;
      bpart += (sv[e] * dv[e]) * sy;  // r d y with r = sqrt(r)^2
      ((float*)sm.stage)[j * C::LDKF + kk] = (float)sy;
    }
    __syncthreads();
    if (staging && q0 + KCH < nobs) fetch(q0 + KCH);
    if (wave_on) {
      const float* At = (const float*)sm.stage;
#pragma unroll
      for (int ks = 0; ks < KCH / 4; ++ks) {
        float av[TR], bv[TC];
#pragma unroll
        for (int a = 0; a < TR; ++a) av[a] = At[((tr0 + a) * 16 + lane % 16) * C::LDKF + ks * 4 + lane / 16];
#pragma unroll
        for (int b = 0; b < TC; ++b) bv[b] = At[((tc0 + b) * 16 + lane % 16) * C::LDKF + ks * 4 + lane / 16];
#pragma unroll
        for (int a = 0; a < TR; ++a)
#pragma unroll
          for (int b = 0; b < TC; ++b) {
            const f32x4 part = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            double* cr = sm.Bm + ((tr0 + a) * 16 + 4 * (lane / 16)) * SM::LDA + (tc0 + b) * 16 + lane % 16;
#pragma unroll
            for (int v = 0; v < 4; ++v) cr[v * SM::LDA] += (double)part[v];
          }
      }
    }
    __syncthreads();
  }
  if (wave_on) {
#pragma unroll
    for (int a = 0; a < TR; ++a)
#pragma unroll
      for (int b = 0; b < TC; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = (tr0 + a) * 16 + 4 * (lane / 16) + v, j = (tc0 + b) * 16 + lane % 16;
          // put_A of (i <= j) overwrites only (i, j), which this lane
          // owns, and (j, i), whose owner does not use its value; so every value
          // that is used is read before anything overwrites it.
          const double c = sm.Bm[i * SM::LDA + j];
          put_A(sm, i, j, m, c, I.a_diag, dbg);
        }
  }
  // b: threads sharing j = tid % M hold partial sums
  if (staging) sm.red()[tid] = bpart;
  __syncthreads();
  if (tid < M) {
    double t = 0.0;
    for (int q = tid; q < ST; q += M) t += sm.red()[q];
    sm.bvec[tid] = tid < m ? t : 0.0;
  }
  __syncthreads();
}

// ---- a4/a5 on the BF16 paths -------------------------------------------------
// Split operands (hi + lo, three products) on v_mfma_f32_16x16x32_bf16, with the
// observation table staged in LDS first (as in the FP64 gather: row of Y',
// sqrt(r), sqrt(r) d, in the space A takes afterwards), so that the chunk
// loop issues only the FP32 loads of Y' rows, three chunks in flight.  With
// the index, r and d loads in the loop a chunk of 32 observations spent
// ~6.6k cycles for a few hundred cycles of products.
template <typename SM>
__device__ __forceinline__ void gather_C_bf16(SM& sm, const InstDesc& I, int obs_off, int s, double* dbg) {
  using C = typename SM::C;
  constexpr int M = C::M;
  constexpr int NT = C::NT, ST = C::RT, KCH = C::KCB, LDKB = C::LDKB;
  const bool staging = ST == NT || phase_tid() < ST;
  constexpr int TILES = C::TILES, TR = C::TR, TC = C::TC;
  const int m = I.m, tid = phase_tid(), w = tid / 64, lane = tid % 64;
  const bool wave_on = TILES >= 2 || w == 0;
  const int tr0 = TILES >= 2 ? (w / 2) * TR : 0;
  const int tc0 = TILES >= 2 ? (w % 2) * TC : 0;
  f32x4 acc[TR][TC];
#pragma unroll
  for (int a = 0; a < TR; ++a)
#pragma unroll
    for (int b = 0; b < TC; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  double bpart = 0.0;
  const float* Yp = (const float*)I.Yp;
  const int nobs = 2 * s;
  constexpr int SEG = (M * SM::LDA * 8 / 20) / KCH * KCH;
  static_assert(SEG >= KCH && SEG % 2 == 0 && (size_t)SEG * (4 + 8 + 8) <= sizeof(sm.Bm), "observation table");
  int* rowT = reinterpret_cast<int*>(sm.Bm);
  double* sT = sm.Bm + SEG / 2;
  double* sdT = sT + SEG;
  const int32_t* obs_row = I.obs_row + 2 * obs_off;
  const double* obs_sr = I.obs_sr + 2 * obs_off;
  const double* dvec = I.d;
  // Thread (kk0 = tid / M, j = tid % M), of the first ST, stages observations
  // kk0 + e ST / M of every chunk for member j.
  constexpr int EPT = KCH * M / ST;
  static_assert(KCH * M % ST == 0, "whole chunks per thread");
  const int kk0 = M >= 64 ? __builtin_amdgcn_readfirstlane(tid / M) : tid / M, j = tid % M;
  __bf16* Ah = (__bf16*)sm.stage;
  __bf16* Al = Ah + M * LDKB;
  for (int g0 = 0; g0 < nobs; g0 += SEG) {
    const int gn = nobs - g0 < SEG ? nobs - g0 : SEG;
    const int gr = (gn + KCH - 1) / KCH * KCH;
    // (the previous segment's last chunk ended with a barrier)
    for (int q = tid; q < gr; q += NT) {
      int rw = 0;
      double sr = 0.0, sd = 0.0;
      if (q < gn) {
        rw = gload(obs_row + g0 + q);
        sr = gload(obs_sr + g0 + q);
        sd = sr * gload(dvec + rw);
      }
      rowT[q] = rw;
      sT[q] = sr;
      sdT[q] = sd;
    }
    __syncthreads();
    auto fetch = [&](float (&y)[EPT], int q0) {  // Y' of chunk q0 (segment-relative)
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int q = q0 + kk0 + e * (ST / M);
        y[e] = 0.f;
        if (q < gn && j < m) y[e] = gload(Yp + (size_t)rowT[q] * m + j);
      }
    };
    auto chunk = [&](const float (&y)[EPT], float (&next)[EPT], int q0) {
      if (staging)
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int q = q0 + kk0 + e * (ST / M);  // < gr: the table's tail is zero
        const int kk = kk0 + e * (ST / M);
        const double sy = sT[q] * (double)y[e];
        bpart += sdT[q] * sy;  // r d y with r = sqrt(r)^2
        // split BF16: x = hi + lo with hi = bf16(x), lo = bf16(x - hi)
        const float xf = (float)sy;
        const __bf16 hi = (__bf16)xf;
        Ah[j * LDKB + kk] = hi;
        Al[j * LDKB + kk] = (__bf16)(xf - (float)hi);
      }
      __syncthreads();
      if (staging && q0 + 2 * KCH < gn) fetch(next, q0 + 2 * KCH);
      if (wave_on) {
        // C += hi hi^T + hi lo^T + lo hi^T (the lo lo^T term is below FP32 rounding)
        bf16x8 ah[TR], al[TR], bh[TC], bl[TC];
#pragma unroll
        for (int a = 0; a < TR; ++a) {
          const int ra = ((tr0 + a) * 16 + lane % 16) * LDKB + 8 * (lane / 16);
          ah[a] = *(const bf16x8*)(Ah + ra);
          al[a] = *(const bf16x8*)(Al + ra);
        }
#pragma unroll
        for (int b = 0; b < TC; ++b) {
          const int rb = ((tc0 + b) * 16 + lane % 16) * LDKB + 8 * (lane / 16);
          bh[b] = *(const bf16x8*)(Ah + rb);
          bl[b] = *(const bf16x8*)(Al + rb);
        }
#pragma unroll
        for (int a = 0; a < TR; ++a)
#pragma unroll
          for (int b = 0; b < TC; ++b) {
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[a], bh[b], acc[a][b], 0, 0, 0);
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[a], bl[b], acc[a][b], 0, 0, 0);
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[a], bh[b], acc[a][b], 0, 0, 0);
          }
      }
      __syncthreads();
    };
    float ya[EPT], yb[EPT], yc[EPT];
    if (staging) fetch(ya, 0);
    if (staging && KCH < gn) fetch(yb, KCH);
    for (int q0 = 0; q0 < gn; q0 += 3 * KCH) {
      chunk(ya, yc, q0);
      if (q0 + KCH < gn) chunk(yb, ya, q0 + KCH);
      if (q0 + 2 * KCH < gn) chunk(yc, yb, q0 + 2 * KCH);
    }
  }
  if (wave_on) {
#pragma unroll
    for (int a = 0; a < TR; ++a)
#pragma unroll
      for (int b = 0; b < TC; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int i = (tr0 + a) * 16 + 4 * (lane / 16) + v, jj = (tc0 + b) * 16 + lane % 16;
          put_A(sm, i, jj, m, (double)acc[a][b][v], I.a_diag, dbg);
        }
  }
  // b: threads sharing j = tid % M hold partial sums
  if (staging) sm.red()[tid] = bpart;
  __syncthreads();
  if (tid < M) {
    double t = 0.0;
    for (int q = tid; q < ST; q += M) t += sm.red()[q];
    sm.bvec[tid] = tid < m ? t : 0.0;
  }
  __syncthreads();
}

// ---- the FP64 gather on vector FMA, k_analysis at M = 128 --------------------
template <int M>
__device__ __forceinline__ void gather_C_fp64(AnaSmem<M>& sm, const InstDesc& I, int obs_off, int s, double* dbg) {
  using C = AnaCfg<M>;
  constexpr int NT = C::NT, KC = C::KC, TM = C::TM, TX = C::TX;
  double* Xc = (double*)sm.stage;
  const int m = I.m, tid = phase_tid(), ti = C::row0(tid), tj = tid % 16;
  double acc[TX][TM];
#pragma unroll
  for (int x = 0; x < TX; ++x)
#pragma unroll
    for (int y = 0; y < TM; ++y) acc[x][y] = 0.0;
  double bacc = 0.0;
  const double* Yp = (const double*)I.Yp;
  const int nobs = 2 * s;
  for (int q0 = 0; q0 < nobs; q0 += KC) {
    const int kc = min(KC, nobs - q0);
    for (int idx = tid; idx < KC * M; idx += NT) {
      const int qq = idx / M, j = idx % M;
      double v = 0.0;
      if (qq < kc && j < m) v = Yp[(size_t)I.obs_row[2 * obs_off + q0 + qq] * m + j];
      Xc[idx] = v;
    }
    if (tid < KC) {
      double r = 0.0, dd = 0.0;
      if (tid < kc) {
        r = I.obs_r[2 * obs_off + q0 + tid];
        dd = I.d[I.obs_row[2 * obs_off + q0 + tid]];
      }
      sm.rc[tid] = r;
      sm.dc[tid] = dd;
    }
    __syncthreads();
    for (int qq = 0; qq < kc; ++qq) {
      const double r = sm.rc[qq];
      double yi[TX], yj[TM];
#pragma unroll
      for (int x = 0; x < TX; ++x) yi[x] = r * Xc[qq * M + ti + 16 * x];
#pragma unroll
      for (int y = 0; y < TM; ++y) yj[y] = Xc[qq * M + tj + 16 * y];
#pragma unroll
      for (int x = 0; x < TX; ++x)
#pragma unroll
        for (int y = 0; y < TM; ++y) acc[x][y] += yi[x] * yj[y];
    }
    if (tid < M)
      for (int qq = 0; qq < kc; ++qq) bacc += sm.rc[qq] * sm.dc[qq] * Xc[qq * M + tid];
    __syncthreads();
  }
#pragma unroll
  for (int x = 0; x < TX; ++x)
#pragma unroll
    for (int y = 0; y < TM; ++y) put_A(sm, ti + 16 * x, tj + 16 * y, m, acc[x][y], I.a_diag, dbg);
  if (tid < M) sm.bvec[tid] = tid < m ? bacc : 0.0;
  __syncthreads();
}

// ---- a6 (first half): Cholesky factor A = L L^T (FP64) ----------------------
// Right-looking, by panels of 16 columns.  Wavefront 0 factors a panel on its
// own: lane l holds rows c0 + l (and c0 + 64 + l at M = 128) of the panel's
// 16 columns, the pivot of column j is read from lane j (readlane), column j is scaled by
// 1/sqrt(a_jj) (one rsqrt) and the later panel columns take its outer product
// with the entries L[c0+jj][c0+j] read from the lanes that hold them - no
// workgroup barrier inside the panel.  Then every wavefront subtracts the
// panel's rank-16 product from the lower triangle of the trailing matrix, in
// 16 x 16 tiles on v_mfma_f64_16x16x4f64 (accumulating onto the tile, with
// the right operand negated).  Two barriers per panel, against one per
// column for a column-at-a-time form.  L is left column-major in Bm (column c
// at Bm[c LDB ..]) with its upper triangle zeroed for the Jacobi phase.  A is
// SPD (all eigenvalues >= (m-1)/rho), so every pivot is positive.
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const long long x = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)x, lane);
  const int hi = __builtin_amdgcn_readlane((int)(x >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <int M>
__device__ __forceinline__ void cholesky(AnaSmem<M>& sm) {
  using C = AnaCfg<M>;
  constexpr int LDB = C::LDB, NT = C::NT, NP = M / 16;
  constexpr int RS = (M + 63) / 64;  // rows per lane: c0 + lane + 64 s, s < RS
  static_assert(M % 16 == 0 && M <= 128, "panels of 16 columns, at most two rows per lane");
  const int tid = phase_tid(), w = tid / 64, lane = tid % 64;
#pragma unroll 1
  for (int p = 0; p < NP; ++p) {
    const int c0 = 16 * p;
    if (w == 0) {
      double a[RS][16];
#pragma unroll
      for (int s = 0; s < RS; ++s) {
        const int r = c0 + lane + 64 * s;
        const bool on = r < M;
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) a[s][jj] = on ? sm.Bm[(c0 + jj) * LDB + r] : 0.0;
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double d = readlane_f64(a[0][j], j);  // a_jj after the earlier columns
        const double rs = rsqrt(d);
        double lj[RS];
        lj[0] = lane > j ? a[0][j] * rs : (lane == j ? d * rs : 0.0);
#pragma unroll
        for (int s = 1; s < RS; ++s) lj[s] = a[s][j] * rs;  // rows past the panel's diagonal block
#pragma unroll
        for (int s = 0; s < RS; ++s) a[s][j] = lj[s];
#pragma unroll
        for (int jj = j + 1; jj < 16; ++jj) {
          const double l = readlane_f64(lj[0], jj);
#pragma unroll
          for (int s = 0; s < RS; ++s) a[s][jj] = fma(-lj[s], l, a[s][jj]);
        }
      }
#pragma unroll
      for (int s = 0; s < RS; ++s) {
        const int r = c0 + lane + 64 * s;
        if (r < M)
#pragma unroll
          for (int jj = 0; jj < 16; ++jj) sm.Bm[(c0 + jj) * LDB + r] = a[s][jj];
      }
    }
    __syncthreads();
    // trailing lower triangle: tile (R, Cc), R >= Cc, of the blocks past the panel
    const int nt = NP - p - 1;
    int t = 0;
    for (int R = 0; R < nt; ++R)
      for (int Cc = 0; Cc <= R; ++Cc, ++t) {
        if (t % (NT / 64) != w) continue;
        const int rb = c0 + 16 * (R + 1), cb = c0 + 16 * (Cc + 1);
        // the tile transposed, D[i][j] = B(rb + j, cb + i): a lane's accumulators
        // then lie along one column of the column-major B, consecutive across
        // the 16 lanes (along a row they would be LDB apart, an 8-way bank
        // conflict on every load and store)
        f64x4 acc;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = sm.Bm[(cb + lane / 16 + 4 * v) * LDB + rb + lane % 16];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const int k = c0 + 4 * ks + lane / 16;
          const double av = -sm.Bm[k * LDB + cb + lane % 16];
          const double bv = sm.Bm[k * LDB + rb + lane % 16];
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) sm.Bm[(cb + lane / 16 + 4 * v) * LDB + rb + lane % 16] = acc[v];
      }
    __syncthreads();
  }
  for (int idx = tid; idx < M * M; idx += NT) {
    const int c = idx / M, r = idx % M;
    if (r < c) sm.Bm[c * LDB + r] = 0.0;
  }
  __syncthreads();
}

// 1/sqrt(x) for x in [1, 2] (or any x but zero, infinity and denormals): the
// hardware estimate e0 (relative error ~2^-23) refined by one third-order step
// c = c0 (1 + e/2 + 3e^2/8), e = 1 - x c0^2, which leaves a relative error of
// order e^3, below the rounding of the result.
__device__ __forceinline__ double rsqrt_1_2(double x) {
  const double c0 = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * c0, c0, 1.0);
  return fma(c0 * e, fma(e, 0.375, 0.5), c0);
}

// Rotation arithmetic in either precision.  approx_*: the hardware estimates
// (FP64: relative error ~2^-23; FP32: about 1 ulp); rsqrt_acc: 1/sqrt(x) for x
// in [1, 2] to the rounding of the type (FP32: the estimate already is).
__device__ __forceinline__ double approx_rsq(double x) { return __builtin_amdgcn_rsq(x); }
__device__ __forceinline__ float approx_rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double approx_rcp(double x) { return __builtin_amdgcn_rcp(x); }
__device__ __forceinline__ float approx_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rsqrt_acc(double x) { return rsqrt_1_2(x); }
// Issue priority of the calling wavefront (0..3; wavefront-uniform argument).
__device__ __forceinline__ void set_issue_prio(int p) {
  if (p >= 3) __builtin_amdgcn_s_setprio(3);
  else if (p == 2) __builtin_amdgcn_s_setprio(2);
  else if (p == 1) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}
// the word holding the sign: non-negative exactly when x >= +0
__device__ __forceinline__ int sign_word(double x) { return (int)(__double_as_longlong(x) >> 32); }
__device__ __forceinline__ int sign_word(float x) { return __float_as_int(x); }
__device__ __forceinline__ float rsqrt_acc(float x) { return __builtin_amdgcn_rsqf(x); }

// Group sum of a float (same lane patterns as the double form).
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
// lanes l and l ^ 8 exchange v (row_ror:8 within each row of 16 lanes)
__device__ __forceinline__ double swap_lanes8(double v) { return dpp_f64<0x128>(v); }
__device__ __forceinline__ float swap_lanes8(float v) { return dpp_f32<0x128>(v); }
template <int G>
__device__ __forceinline__ float group_sum(float v) {
  if constexpr (G >= 2) v += dpp_f32<0xB1>(v);
  if constexpr (G >= 4) v += dpp_f32<0x4E>(v);
  if constexpr (G >= 8) v += dpp_f32<0x141>(v);
  if constexpr (G >= 16) v += dpp_f32<0x140>(v);
  static_assert(G <= 16, "group_sum supports up to 16 lanes");
  return v;
}

// True when every pair of columns of the current B satisfies
// (b_i.b_j)^2 <= tol2 |b_i|^2 |b_j|^2, i.e. when a further sweep would not
// rotate.  Each thread forms a TX x TM block of B^T B from LDS (the norms are
// the ones the sweep kept current).  Block-uniform result; ends with a barrier.
// B: column c at B[c * LD], element type R.
template <typename R, int M, int LD>
__device__ __forceinline__ bool gram_converged(const R* B, const R* nrm, R tol2) {
  constexpr int TM = AnaCfg<M>::TM, TX = AnaCfg<M>::TX;
  const int tid = phase_tid(), ti = AnaCfg<M>::row0(tid), tj = tid % 16;
  R g[TX][TM];
#pragma unroll
  for (int x = 0; x < TX; ++x)
#pragma unroll
    for (int y = 0; y < TM; ++y) g[x][y] = 0;
  // lane tj visits the rows from tj on (mod M): the 16 columns tj + 16 x that
  // a pass of lanes reads then fall in 16 bank pairs (all at one row they sat
  // in two, a column being LD doubles apart)
#pragma unroll 2
  for (int r0 = 0; r0 < M; ++r0) {
    const int r = (r0 + tj) & (M - 1);
    R u[TX], v[TM];
#pragma unroll
    for (int x = 0; x < TX; ++x) u[x] = B[(ti + 16 * x) * LD + r];
#pragma unroll
    for (int y = 0; y < TM; ++y) v[y] = B[(tj + 16 * y) * LD + r];
#pragma unroll
    for (int x = 0; x < TX; ++x)
#pragma unroll
      for (int y = 0; y < TM; ++y) g[x][y] = fma(u[x], v[y], g[x][y]);
  }
  bool bad = false;
#pragma unroll
  for (int x = 0; x < TX; ++x)
#pragma unroll
    for (int y = 0; y < TM; ++y) {
      const int i = ti + 16 * x, j = tj + 16 * y;
      bad |= i < j && g[x][y] * g[x][y] > tol2 * (nrm[i] * nrm[j]);
    }
  return !__syncthreads_or(bad);
}

// The same test for FP64 columns at M = 64 with the products on the matrix
// cores: wavefront w forms the 2 x 2 tiles (16 x 16 each) of B^T B at tile rows
// 2 (w / 2), 2 (w / 2) + 1 and tile columns 2 (w % 2), 2 (w % 2) + 1.  Each lane
// reads two consecutive rows of its column with one 16-byte load, the A / B
// operands of two k-steps (rows r0 + 2 k and r0 + 2 k + 1 for the operand's
// k = lane / 16).  The VALU form spent ~25k cycles per test on 512 LDS loads
// and 1024 FMAs per thread; this one 64 MFMAs and 32 loads per wavefront.
template <int LD>
__device__ __forceinline__ bool gram_converged_mfma64(const double* B, const double* nrm, double tol2) {
  const int tid = phase_tid(), w = tid / 64, lane = tid % 64;
  const int tr0 = (w >> 1) * 2, tc0 = (w & 1) * 2;
  const int kq = lane / 16, cl = lane % 16;
  f64x4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int r0 = 0; r0 < 64; r0 += 8) {
    const int r = r0 + 2 * kq;
    double2 av[2], bv[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      av[a] = *(const double2*)&B[((tr0 + a) * 16 + cl) * LD + r];
      bv[a] = *(const double2*)&B[((tc0 + a) * 16 + cl) * LD + r];
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].x, bv[b].x, acc[a][b], 0, 0, 0);
        acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a].y, bv[b].y, acc[a][b], 0, 0, 0);
      }
  }
  bool bad = false;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = (tr0 + a) * 16 + kq + 4 * v, j = (tc0 + b) * 16 + cl;
        const double g = acc[a][b][v];
        bad |= i < j && g * g > tol2 * (nrm[i] * nrm[j]);
      }
  return !__syncthreads_or(bad);
}

// One sweep at M = 128 (see jacobi_core): 64 pair slots of 8 lanes, 16 rows a
// lane.  The same steps as below with the loops over groups and steps kept as
// loops (unrolled, the 127 steps are four times the instruction cache), two
// steps to a pass: after the even one the slots q and q ^ 1 exchange partners by
// a lane swap, the odd one writes its partner back and loads the next pass's.  A
// branch is taken by whole wavefronts, a lane whose pair does not rotate with
// c = 1, sn = 0.
// Lane e of a slot holds rows (e >> 1) + 4 (e & 1) + 8 u, so that a dot
// product is summed as by four lanes of two partial sums each, and products are
// fused where they are written so: the rotations, and with them the FP32 and
// BF16 trajectories (which round X' every frame), do not depend on how many
// threads share a column.
template <typename R, int LD>
__device__ __forceinline__ void sweep_128(__attribute__((address_space(3))) R* LB, __attribute__((address_space(3))) R* LN,
                                          int* s_rot, R tol4, R trig4, int& big) {
#pragma clang fp contract(off)
  using LR = __attribute__((address_space(3))) R;
  constexpr int RPT = 16;
  const int tid = phase_tid(), q = tid / 8, e = tid % 8;
  LR* const L0 = LB + (e >> 1) + 4 * (e & 1);
  R xi[RPT], xa[RPT], xb[RPT], al = 0, ba = 0, bb = 0;
  // A step of the pair (xi, xc), norms al and bc: put(u, v) takes the partner's
  // values and end(n) its norm, on both sides of the branch, so that neither is
  // a value the two sides have to agree on a register for.
  auto step = [&](const R (&xc)[RPT], const R bc, auto&& put, auto&& end) {
    R g = 0;
#pragma unroll
    for (int u = 0; u < RPT; ++u) g = fma(xi[u], xc[u], g);
    const R gsum = group_sum<8>(g);
    const R ab = al * bc, g2 = gsum + gsum, g4 = g2 * g2;
    const bool rot = g4 > tol4 * ab;
    if (__builtin_amdgcn_ballot_w64(rot) != 0) {
      big = max(big, sign_word(fma(-trig4, ab, g4)));  // negative where no rotation
      const R dd = bc - al;
      const R q2 = fma(dd, dd, g4);
      const R den = fma(q2, approx_rsq(q2), fabs(dd));
      const R t = rot ? copysign((R)1, dd) * g2 * approx_rcp(den) : (R)0;
      const R c = rot ? rsqrt_acc(fma(t, t, (R)1)) : (R)1;
      const R sn = c * t;
#pragma unroll
      for (int u = 0; u < RPT; ++u) {
        const R a = xi[u], b = xc[u];
        const R sa = sn * a, sb = sn * b;
        xi[u] = fma(c, a, -sb);
        put(u, fma(c, b, sa));
      }
      al = fma(-t, gsum, al);
      end(bc + t * gsum);
      *s_rot = 1;
    } else {
#pragma unroll
      for (int u = 0; u < RPT; ++u) put(u, xc[u]);
      end(bc);
    }
  };
  auto load = [&](int i, int j) {  // the pair slot's column and its first partner
    const LR* bi = L0 + i * LD;
    const LR* bj = L0 + j * LD;
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      xi[u] = bi[8 * u];
      xa[u] = bj[8 * u];
    }
    al = LN[i];
    ba = LN[j];
  };
  auto finish = [&](int i) {
    LR* bi = L0 + i * LD;
#pragma unroll
    for (int u = 0; u < RPT; ++u) bi[8 * u] = xi[u];
    if (e == 0) LN[i] = al;
    __syncthreads();
  };
  {  // the first group's only step
    LR* bj = L0 + (2 * q + 1) * LD;
    load(2 * q, 2 * q + 1);
    step(xa, ba, [&](int u, R v) { bj[8 * u] = v; }, [&](R n) { LN[2 * q + 1] = n; });
    finish(2 * q);
  }
#pragma unroll 1
  for (int h = 1; h < 7; ++h) {
    const int low = 1 << h, i = ((q >> h) << (h + 1)) | (q & (low - 1)), kend = 2 << h;
    load(i, i ^ low);
#pragma unroll 1
    for (int k = low; k < kend; k += 2) {
      step(xa, ba, [&](int u, R v) { xb[u] = swap_lanes8(v); }, [&](R n) { bb = swap_lanes8(n); });
      LR* bj = L0 + (i ^ (k + 1)) * LD;
      step(xb, bb, [&](int u, R v) { bj[8 * u] = v; }, [&](R n) { LN[i ^ (k + 1)] = n; });
      if (k + 2 < kend) {
        // the next partner was written by a slot of this wavefront, except after
        // every eighth step
        if ((k + 2) % 8 == 0) __syncthreads();
        else __asm__ volatile("" ::: "memory");
        const LR* bn = L0 + (i ^ (k + 2)) * LD;
#pragma unroll
        for (int u = 0; u < RPT; ++u) xa[u] = bn[8 * u];
        ba = LN[i ^ (k + 2)];
      }
    }
    finish(i);
  }
}

// ---- a6 (second half): one-sided (Hestenes) Jacobi on the columns of L ------
// L J = U Sigma with U the eigenvectors of A = L L^T and lambda = sigma^2, so
// no rotation accumulator is needed; rounding scales with sqrt(lambda), and
// the Cholesky factor's columns start closer to orthogonal than those of A.
// A sweep visits the pairs (i, i^k), k = 1..M-1 (M-1 perfect matchings that
// cover every pair once).  Steps are grouped by the highest set bit h of k:
// within a group every pair joins a column with bit h clear (the "lower"
// column) to one with bit h set, and each lower column meets all its
// partners in that group, so its pair slot keeps it in registers for the
// whole group and only the partner column goes through LDS each step.
// The columns are B[c * LD ..] (element type R: FP64, or FP32 for the BF16
// path), their squared norms nrm[c]; tol is the rotation threshold.  Returns
// the sweeps done; `converged` is set when a sweep rotated nothing or the
// Gram test passed, and stays false when the sweep cap ended the loop.
template <typename R, int M, int LD>
__device__ __forceinline__ int jacobi_core(AnaSmem<M>& sm, int m, R* B, R* nrm, R tol, bool& converged, bool fair) {
  using C = AnaCfg<M>;
  constexpr int NT = C::NT, TPP = C::TPP;
  constexpr int PSW = 64 / TPP;  // pair slots per wavefront
  static_assert(TPP <= 64 && 64 % TPP == 0, "pair slots tile the wavefront");
  const int tid = phase_tid();
  const bool active = C::ACTIVE >= NT || tid < C::ACTIVE;
  const int q = tid / TPP, sub = tid % TPP;
  const R tol2 = tol * tol;
  // Once no rotation of a sweep had a relative off-diagonal above trig, the
  // next sweep is likely to find nothing to do, and the Gram test (a fraction
  // of a sweep's cost) is tried instead.  trig = tol^(1/3) / 5: on a CPU
  // replay of the 375 domains of the 84 x 84 map this is where fewer wasted
  // final sweeps stop paying for more failed Gram tests (FP64, tol 4.5e-13:
  // 7.63 -> 7.08 sweeps and 0.44 -> 1.03 Gram tests per domain against the
  // former 1e-7; tol 1e-6: 6.96 -> 6.3 sweeps; tol 1e-4 stays at 6.0).
  const R trig = (R)0.2 * cbrt(tol);
  const R trig2 = trig * trig;
  const R tol4 = (R)4 * tol2, trig4 = (R)4 * trig2;
  // partners exchanged between slots q and q ^ 1 by a lane swap within 16-lane rows
  constexpr bool SWAP = TPP == 8;
  // the step's column and norm accesses through LDS-typed pointers, so that
  // their addresses are 32-bit offsets (a generic pointer makes every partner
  // address a 64-bit multiply-add)
  using LR = __attribute__((address_space(3))) R;
  LR* const LB = (LR*)B;
  LR* const LN = (LR*)nrm;
  int sweeps = 0;
  converged = false;
  for (; sweeps < C::MAX_SWEEPS;) {
    // progress-ordered issue (see k_analysis): the priority falls as the sweeps go by
    if (fair) set_issue_prio(sweeps < 3 ? 3 : sweeps < 5 ? 2 : sweeps < 6 ? 1 : 0);
    {
      constexpr int TPC = C::RT / M;  // threads per column for the norms
      const bool on = C::RT == NT || tid < C::RT;
      const int c = tid / TPC, part = tid % TPC;
      // de Rijk's ordering: every sweep starts with the m columns sorted by
      // decreasing norm (the padded unit columns stay at m..M-1), which saves
      // about one sweep in twelve on the ELT domains (CPU replay).  A column's
      // rank is counted by its TPC threads over interleaved norms; the columns
      // move, in passes of at most 16 values per thread, only when the order
      // changed (late sweeps mostly keep it).
      constexpr int PER = M / TPC, CH = PER < 16 ? PER : 16;
      R ss = 0;
      // column c's threads start at a row that shifts with c, so that the four
      // columns a pass of lanes reads fall in different banks
      // (M = 128: the addresses of its 64 loads formed anew, eight at a time; they
      // would stay live over all sweeps)
      int cn = c;
      if constexpr (M == 128) __asm__ volatile("" : "+v"(cn));
      auto term = [&](int j0) {
        const R v = B[cn * LD + part + TPC * ((j0 + cn) & (PER - 1))];
        ss = fma(v, v, ss);
      };
      if constexpr (M < 128) {
        for (int j0 = 0; j0 < PER; ++j0) term(j0);
      } else if (on) {
#pragma unroll 8
        for (int j0 = 0; j0 < PER; ++j0) term(j0);
      }
      ss = group_sum<TPC>(ss);
      if (on && part == 0) nrm[c] = ss;
      if (tid == 0) sm.s_rot = 0;  // last read before the previous sweep's closing barrier
      __syncthreads();
      R ahead = 0;  // columns ahead of c among this thread's share (exact small integers)
      if (on && c < m)
        for (int c2 = part; c2 < m; c2 += TPC) {
          const R n2 = nrm[c2];
          ahead += (n2 > ss || (n2 == ss && c2 < c)) ? (R)1 : (R)0;
        }
      ahead = group_sum<TPC>(ahead);
      const int rank = c < m ? (int)ahead : c;
      if (__syncthreads_or(on && rank != c)) {
        for (int k0 = 0; k0 < PER; k0 += CH) {
          // rows rotated by c within the pass, as in the norms: the reads then
          // avoid bank conflicts, and the writes (to the rank's column, same
          // rows) mostly do
          R v[CH];
          if (on)
#pragma unroll
            for (int k = 0; k < CH; ++k) v[k] = B[cn * LD + part + TPC * (k0 + ((k + cn) & (CH - 1)))];
          // every read of this pass's rows (rows TPC k0 .. TPC (k0 + CH) - 1, which no
          // other pass touches) is done before any column moves; the sweep reads
          // the moved columns after the barrier that follows
          __syncthreads();
          // the write addresses recomputed from a copy of c the compiler cannot
          // see through: kept from the reads, the CH addresses stayed live
          // across the barrier and raised the kernel's register count
          int cw = c;
          __asm__ volatile("" : "+v"(cw));
          if (on)
#pragma unroll
            for (int k = 0; k < CH; ++k) B[rank * LD + part + TPC * (k0 + ((k + cw) & (CH - 1)))] = v[k];
        }
        if (on && part == 0) nrm[rank] = ss;
        __syncthreads();  // the moved columns and norms before the sweep reads them
      }
    }
    int big = INT_MIN;
    if constexpr (M == 128) {
      sweep_128<R, LD>(LB, LN, &sm.s_rot, tol4, trig4, big);
    } else
#pragma unroll
    for (int h = 0; (1 << h) < M; ++h) {
      const int i = ((q >> h) << (h + 1)) | (q & ((1 << h) - 1));
      const int kend = 2 << h;
      R xi[C::RPT];
      R al = 0;
      // One step k: pair (i, i ^ k) with the partner column in xc (norm bc).
      // The next step's partner arrives in xn (norm bn) before
      // this step rotates the lower column (registers only), so that its
      // latency overlaps that arithmetic instead of stalling the next dot
      // product; two register sets alternate between consecutive steps.
      // Between an even step k and k + 1 the slots exchange partners in pairs
      // (slot q takes the column slot q ^ 1 just rotated), so with SWAP the
      // rotated partner goes to its next slot by a lane swap and not through
      // LDS; the odd step after it writes that column back, rotated or not,
      // since its LDS copy is then out of date.
      auto step = [&](const int k, R (&xc)[C::RPT], R& bc, R (&xn)[C::RPT], R& bn) {
        // the lower column index as a value the compiler may not carry across
        // steps: unrolled, it would otherwise keep every step's partner
        // address live from the start of the group (registers, occupancy)
        int iv = i;
        __asm__ volatile("" : "+v"(iv));
        iv &= M - 1;  // a known range: 24-bit multiply-adds for the addresses
        const int jj = iv ^ k;
        const bool swp = SWAP && (k & 1) == 0 && k + 1 < kend;
        const bool stale = SWAP && (k & 1) == 1 && k > (1 << h);
        R c = 1, sn = 0;
        bool rot = false;
        if (active) {
          R g0 = 0, g1 = 0;
#pragma unroll
          for (int t = 0; t < C::RPT; ++t) {
            if (t & 1) g1 = fma(xi[t], xc[t], g1);
            else g0 = fma(xi[t], xc[t], g0);
          }
          const R gsum = group_sum<TPP>(g0 + g1);
          // (2 gsum)^2 serves both the test, against 4 tol^2 al bc, and the angle
          const R ab = al * bc, g2 = gsum + gsum, g4 = g2 * g2;
          if (swp) {
            // A step whose partner leaves by the lane exchange: when any pair of
            // the wavefront rotates, every lane takes the step, a lane whose pair
            // does not with t = 0, c = 1, sn = 0 (an exact identity).  The branch
            // is wavefront-uniform, so the rotated columns need no merge with
            // the unrotated ones of masked lanes (that merge cost a register move
            // per value).
            rot = g4 > tol4 * ab;
            if (__builtin_amdgcn_ballot_w64(rot) != 0) {
              big = max(big, sign_word(fma(-trig4, ab, g4)));  // negative where no rotation
              const R dd = bc - al;
              const R q2 = fma(dd, dd, g4);
              const R den = fma(q2, approx_rsq(q2), fabs(dd));
              const R t = rot ? copysign((R)1, dd) * g2 * approx_rcp(den) : (R)0;
              c = rot ? rsqrt_acc(fma(t, t, (R)1)) : (R)1;
              sn = c * t;
#pragma unroll
              for (int u = 0; u < C::RPT; ++u) {
                const R a = xi[u], b = xc[u];
                xi[u] = c * a - sn * b;
                xc[u] = sn * a + c * b;
              }
              al -= t * gsum;
              bc += t * gsum;
              sm.s_rot = 1;
              // the exchange on both sides of the branch, so that the rotated
              // partner goes from the registers it was computed in
#pragma unroll
              for (int u = 0; u < C::RPT; ++u) xn[u] = swap_lanes8(xc[u]);
              bn = swap_lanes8(bc);
            } else {
#pragma unroll
              for (int u = 0; u < C::RPT; ++u) xn[u] = swap_lanes8(xc[u]);
              bn = swap_lanes8(bc);
            }
          } else if (g4 > tol4 * ab) {
            rot = true;
            // the largest sign word of g4 - 4 trig^2 al bc: non-negative once a
            // rotation of this sweep had a cosine above trig (an integer
            // maximum: no exec-mask update, no NaN handling)
            big = max(big, sign_word(fma(-trig4, ab, g4)));
            // t = tan(theta), the smaller root of t^2 + 2 zeta t - 1 = 0 with
            // zeta = (be - al) / (2 gsum), written without the quotient zeta.
            // c = (1 + t^2)^(-1/2) to the rounding of R keeps c^2 + s^2 = 1 to
            // rounding for whatever t is used, so t itself comes from the
            // hardware's approximate rsq / rcp: its error only changes how far
            // this rotation reduces gsum, never orthogonality.
            const R dd = bc - al;
            const R q2 = fma(dd, dd, g4);
            const R den = fma(q2, approx_rsq(q2), fabs(dd));
            const R t = copysign((R)1, dd) * g2 * approx_rcp(den);
            c = rsqrt_acc(fma(t, t, (R)1));
            sn = c * t;
            // the partner first: the slot that pairs it next reads it from LDS
            LR* bj = LB + jj * LD;
#pragma unroll
            for (int u = 0; u < C::RPT; ++u) bj[sub + u * TPP] = sn * xi[u] + c * xc[u];
            al -= t * gsum;
            bc += t * gsum;
            // one lane of the slot stores the norm and the flag (all eight storing
            // the same value saved an exec-mask region but cost ~1 % of the sweep)
            if (sub == 0) {
              LN[jj] = bc;
              sm.s_rot = 1;
            }
          }
          if (stale && !rot) {
            LR* bj = LB + jj * LD;
#pragma unroll
            for (int u = 0; u < C::RPT; ++u) bj[sub + u * TPP] = xc[u];
            LN[jj] = bc;
          }
        }
        // Step k + 1 reads a partner column (and its norm) that step k wrote:
        // the writer's lower column differs from this slot's in the low bits
        // where k and k + 1 differ, so it is a pair slot of the same wavefront
        // unless k + 1 is a multiple of PSW, and the LDS operations of one
        // wavefront take effect in order.  Only those steps need the
        // workgroup barrier (the group's last step is followed by one anyway);
        // the others only keep the compiler from moving LDS accesses across.
        if ((k + 1) % PSW == 0 && k + 1 < kend) __syncthreads();
        else __asm__ volatile("" ::: "memory");
        if (active && !swp && k + 1 < kend) {
          const LR* bk = LB + (iv ^ (k + 1)) * LD;
#pragma unroll
          for (int t = 0; t < C::RPT; ++t) xn[t] = bk[sub + t * TPP];
          bn = LN[iv ^ (k + 1)];
        }
        if (rot && !swp) {
#pragma unroll
          for (int u = 0; u < C::RPT; ++u) xi[u] = c * xi[u] - sn * xc[u];
        }
      };
      R xa[C::RPT], xb[C::RPT];
      R ba = 0, bb = 0;
      if (active) {
        const R* b0 = B + (i ^ (1 << h)) * LD;  // the group's first partner
#pragma unroll
        for (int t = 0; t < C::RPT; ++t) {
          xi[t] = B[i * LD + sub + t * TPP];
          xa[t] = b0[sub + t * TPP];
        }
        al = nrm[i];
        ba = nrm[i ^ (1 << h)];
      }
#pragma unroll
      for (int k = 1 << h; k < kend; k += 2) {
        step(k, xa, ba, xb, bb);
        if (k + 1 < kend) step(k + 1, xb, bb, xa, ba);
      }
      if (active) {
#pragma unroll
        for (int t = 0; t < C::RPT; ++t) B[i * LD + sub + t * TPP] = xi[t];
        if (sub == 0) nrm[i] = al;
      }
      __syncthreads();
    }
    ++sweeps;
    const int any = sm.s_rot;
    const int any_big = __syncthreads_or(big >= 0);
    bool gram = false;
    if (any && !any_big) {
      if constexpr (sizeof(R) == 8 && M == 64 && LD % 2 == 0) gram = gram_converged_mfma64<LD>((const double*)B, (const double*)nrm, (double)tol2);
      else gram = gram_converged<R, M, LD>(B, nrm, tol2);
    }
    if (!any || gram) {
      converged = true;
      break;
    }
  }
  return sweeps;
}

// Rotations are skipped once |b_i.b_j| <= tol |b_i| |b_j|; the W and T this
// leaves behind are off by about 4 tol (relative).  FP64 path: tol = 32 M eps
// (2.3e-13 at M = 64).  The rounding of the eigenvectors (eps |L| per column,
// amplified by the conditioning) leaves W about 2e-12 off whatever the
// tolerance, so this one adds nothing measurable: over the 375 domains of the
// 84x84 map, W stays within 2.05e-12 of the exact one against 2.00e-12 at
// tol = M eps, in at most 8 sweeps instead of 11 (CPU replay).  The FP32 and
// BF16 paths form C with relative errors ~5e-8 and ~4e-6, which put their T
// about 6e-5 and 4e-3 from the FP64 result whatever the eigensolver does;
// their tolerances, 1e-6 and 1e-4, keep the eigensolver's share an order of
// magnitude below that.  At 1e-4 the rotations themselves can run in FP32
// (rounding ~6e-8 per rotation, a converged off-diagonal of a few 1e-6), which
// the opt-in BF16 variant (P = 3) does: L is rounded to FP32 in place (float
// columns at stride M + TPP inside the double storage), rotated, and widened
// back.  The other paths rotate in FP64.
template <int P, int M>
__device__ __forceinline__ int jacobi(AnaSmem<M>& sm, int m, bool& converged, bool fair) {
  using C = AnaCfg<M>;
  if constexpr (P == 3) {
    // In-place width change by chunks of CC columns (at most 16 values per
    // thread in flight).  A float column c ends at or below the start of
    // double column c + 1 (LDF <= 2 LDB and M <= 2 LDB), so narrowing in
    // increasing column order, and widening in decreasing order, never
    // overwrites a value that a later chunk still has to read; each chunk
    // reads everything before its barrier and writes after it.
    constexpr int NT = C::NT, LDB = C::LDB, LDF = M + C::TPP;
    constexpr int CC = M * M / NT <= 16 ? M : 16 * NT / M, PER = CC * M / NT;
    static_assert(LDF <= 2 * LDB && M <= 2 * LDB && M % CC == 0 && (CC * M) % NT == 0,
                  "float columns fit in the double storage");
    float* Bf = reinterpret_cast<float*>(sm.Bm);
    float* nf = reinterpret_cast<float*>(sm.nrm);
    const int tid = phase_tid();
    for (int c0 = 0; c0 < M; c0 += CC) {
      float v[PER];
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int idx = tid + NT * k, c = c0 + idx / M, r = idx % M;
        v[k] = (float)sm.Bm[c * LDB + r];
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int idx = tid + NT * k, c = c0 + idx / M, r = idx % M;
        Bf[c * LDF + r] = v[k];
      }
    }
    __syncthreads();
    const int sweeps = jacobi_core<float, M, LDF>(sm, m, Bf, nf, 1e-4f, converged, fair);
    for (int c0 = M - CC; c0 >= 0; c0 -= CC) {
      float v[PER];
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int idx = tid + NT * k, c = c0 + idx / M, r = idx % M;
        v[k] = Bf[c * LDF + r];
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int idx = tid + NT * k, c = c0 + idx / M, r = idx % M;
        sm.Bm[c * LDB + r] = (double)v[k];
      }
    }
    __syncthreads();
    return sweeps;
  } else {
    const double tol = P == 0 ? 32.0 * (double)M * 1.1102230246251565e-16 : (P == 1 ? 1e-6 : 1e-4);
    return jacobi_core<double, M, C::LDB>(sm, m, sm.Bm, sm.nrm, tol, converged, fair);
  }
}

// Product of the transposed M x M matrix in LDS (column c at Bm[c * LDB ..]) with a
// vector, by TPC = RT / M lanes per output reduced by DPP: lane group o = tid / TPC,
// lane part = tid % TPC takes every TPC-th term (two accumulators), and every
// lane of the group gets the sum.  With the column stride LDB the lanes of a
// wavefront read distinct banks in both forms.
// sum over r of Bm[o LDB + r] v[r]
template <typename SM>
__device__ __forceinline__ double colsum(const SM& sm, const double* v, int o, int part) {
  using C = typename SM::C;
  constexpr int M = C::M;
  constexpr int TPC = C::RT / M, PER = M / TPC, LDB = C::LDB;
  double t0 = 0.0, t1 = 0.0;
#pragma unroll 8
  for (int k = 0; k < PER; k += 2) {
    t0 = fma(sm.Bm[o * LDB + part + TPC * k], v[part + TPC * k], t0);
    if (k + 1 < PER) t1 = fma(sm.Bm[o * LDB + part + TPC * (k + 1)], v[part + TPC * (k + 1)], t1);
  }
  return group_sum<TPC>(t0 + t1);
}
// rowsum: sum over c of Bm[c LDB + o] z[c]   (U z)
template <int M>
__device__ __forceinline__ double rowsum(const AnaSmem<M>& sm, const double* z, int o, int part) {
  using C = AnaCfg<M>;
  constexpr int TPC = C::RT / M, PER = M / TPC, LDB = C::LDB;
  double t0 = 0.0, t1 = 0.0;
#pragma unroll 8
  for (int k = 0; k < PER; k += 2) {
    t0 = fma(sm.Bm[(part + TPC * k) * LDB + o], z[part + TPC * k], t0);
    if (k + 1 < PER) t1 = fma(sm.Bm[(part + TPC * (k + 1)) * LDB + o], z[part + TPC * (k + 1)], t1);
  }
  return group_sum<TPC>(t0 + t1);
}

// One step of iterative refinement of wbar = A^-1 b (FP64 path).  U from the
// one-sided Jacobi carries rounding of order eps |L| in every column, which the
// weights 1/lambda of U Lambda^-1 U^T b amplify for the small eigenvalues
// (wbar relative errors ~1e-10 at m = 100 against ~1e-12 for W).  The
// residual res = b - A wbar is therefore formed with A itself, as the gather
// built it (Ag: the domain's copy of A = (m-1)/rho I + C taken before the
// Cholesky, its lower triangle packed by rows), not through the eigenvectors,
// and wbar += U Lambda^-1 U^T res.  Uses pcol[0] (residual) and pcol[1].
template <int M>
__device__ __forceinline__ void refine_wbar(AnaSmem<M>& sm, const double* __restrict__ Ag, int m) {
  constexpr int TPC = AnaCfg<M>::RT / M, PER = M / TPC;
  const int tid = phase_tid(), o = tid / TPC, part = tid % TPC;
  const bool on = AnaCfg<M>::RT == AnaCfg<M>::NT || tid < AnaCfg<M>::RT;
  double* res = sm.pcol[0];
  double* z = sm.pcol[1];
  __syncthreads();  // wbar complete
  if (on) {
    // (A wbar)_o: row o of the symmetric A; entry (o, c) is packed at row
    // max(o, c), column min(o, c).  Padded rows and columns read entry 0 and
    // are masked by arithmetic (res is zero past m anyway).
    double a[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int c = part + TPC * k;
      const bool in = c < m && o < m;
      const int hi = c > o ? c : o, lo = c > o ? o : c;
      a[k] = (in ? 1.0 : 0.0) * gload(Ag + (in ? tri_size(hi) + lo : 0));
    }
    double t0 = 0.0, t1 = 0.0;
#pragma unroll
    for (int k = 0; k < PER; k += 2) {
      t0 = fma(a[k], sm.wbar[part + TPC * k], t0);
      if (k + 1 < PER) t1 = fma(a[k + 1], sm.wbar[part + TPC * (k + 1)], t1);
    }
    const double t = group_sum<TPC>(t0 + t1);
    if (part == 0) res[o] = o < m ? sm.bvec[o] - t : 0.0;
  }
  __syncthreads();
  if (on) {
    const double t = colsum(sm, res, o, part);
    if (part == 0) z[o] = o < m ? t / sm.lam[o] : 0.0;
  }
  __syncthreads();
  if (on) {
    const double w = rowsum<M>(sm, z, o, part);
    if (part == 0 && o < m) sm.wbar[o] += w;
  }
  __syncthreads();
}

// One step of iterative refinement of wbar on the FP32 / BF16 paths, whose
// Jacobi stops at a looser tolerance: there U^T is a poorer inverse of U, and
// the 1/lambda weights make wbar = U Lambda^-1 U^T b some 1e3 - 1e4 tol off,
// while W stays within 4 tol.  The normalised columns of L J still satisfy
// U Lambda U^T = (L J)(L J)^T = L L^T = A to rounding whether or not the
// sweeps converged, so res = b - U (Lambda (U^T wbar)) is an accurate residual
// from LDS alone, and each wbar += U Lambda^-1 U^T res shrinks the error by a
// factor of order tol kappa(A): two steps at tol 1e-6 and three at 1e-4 leave
// wbar below 1e-8 and 2e-5 on the 15x15 (m = 100) and 84x84 workloads.
template <int M>
__device__ __forceinline__ void refine_wbar_lj(AnaSmem<M>& sm, int m) {
  constexpr int TPC = AnaCfg<M>::RT / M;
  const int tid = phase_tid(), o = tid / TPC, part = tid % TPC;
  const bool on = AnaCfg<M>::RT == AnaCfg<M>::NT || tid < AnaCfg<M>::RT;
  double* z = sm.pcol[0];
  double* res = sm.pcol[1];
  __syncthreads();  // wbar complete
  if (on) {
    const double t = colsum(sm, sm.wbar, o, part);
    if (part == 0) z[o] = o < m ? sm.lam[o] * t : 0.0;
  }
  __syncthreads();
  if (on) {
    const double t = rowsum<M>(sm, z, o, part);
    if (part == 0) res[o] = o < m ? sm.bvec[o] - t : 0.0;
  }
  __syncthreads();
  if (on) {
    const double t = colsum(sm, res, o, part);
    if (part == 0) z[o] = o < m ? t / sm.lam[o] : 0.0;
  }
  __syncthreads();
  if (on) {
    const double w = rowsum<M>(sm, z, o, part);
    if (part == 0 && o < m) sm.wbar[o] += w;
  }
  __syncthreads();
}

// ---- a7: lambda, U, wbar = U Lambda^-1 U^T b, T = U sqrt((m-1)/Lambda) U^T + wbar 1^T
// (from the converged columns sigma_i u_i of L J)
// Leaves T row-major in Bm (T[k][j] at Bm[k*LDB + j], zero outside m x m).
template <int P, int M>
__device__ __forceinline__ void transform(AnaSmem<M>& sm, const InstDesc& I, int l, double* dbg) {
  const int m = I.m;
  using C = AnaCfg<M>;
  constexpr int NT = C::NT, LDB = C::LDB, TM = C::TM, TX = C::TX;
  const int tid = phase_tid(), ti = C::row0(tid), tj = tid % 16;
  const bool on = C::RT == NT || tid < C::RT;
  // debug: shader-clock stamps inside this phase (after U, after wbar, after its refinement)
  auto substamp = [&](int k) {
    if (dbg && threadIdx.x == 0) dbg[2 * m * m + m + 10 + k] = (double)clock64();
  };
  if (on) {
    constexpr int TPC = C::RT / M;
    const int c = tid / TPC, part = tid % TPC;
    double ss = 0.0;
    for (int r = part; r < M; r += TPC) { const double v = sm.Bm[c * LDB + r]; ss += v * v; }
    ss = group_sum<TPC>(ss);
    if (part == 0) {
      sm.lam[c] = ss;          // columns of L J are sigma_i u_i and lambda_i = sigma_i^2
      sm.nrm[c] = 1.0 / sqrt(ss);
    }
  }
  __syncthreads();
  for (int idx = tid; idx < M * M; idx += NT) {
    const int c = idx / M, r = idx % M;
    sm.Bm[c * LDB + r] *= sm.nrm[c];
  }
  __syncthreads();
  substamp(0);
  {
    // wbar = U Lambda^-1 U^T b
    constexpr int TPC = C::RT / M;
    const int o = tid / TPC, part = tid % TPC;
    const double t = on ? colsum(sm, sm.bvec, o, part) : 0.0;
    if (on && part == 0) {
      sm.zv[o] = o < m ? t / sm.lam[o] : 0.0;
      sm.nrm[o] = o < m ? sqrt((double)(m - 1) / sm.lam[o]) : 0.0;
    }
    __syncthreads();
    const double w = on ? rowsum<M>(sm, sm.zv, o, part) : 0.0;
    if (on && part == 0) sm.wbar[o] = o < m ? w : 0.0;
  }
  __syncthreads();
  substamp(1);
  if constexpr (P == 0) {
    refine_wbar<M>(sm, I.Ascr + (size_t)l * tri_size(m), m);
  } else {
#pragma unroll 1
    for (int k = 0; k < (P == 1 ? 2 : 3); ++k) refine_wbar_lj<M>(sm, m);
  }
  substamp(2);
  if constexpr (M <= 64) {
    // T = (U S) U^T on v_mfma_f64_16x16x4f64 (S = diag sqrt((m-1)/lambda), zero
    // past m): k-steps over 4 columns c of U; wave w owns the same WT x WT block
    // of 16 x 16 tiles as in the FP64 gather.  Column c of U is Bm[c LDB ..],
    // so A[i][k] = U[i][c] s_c and B[k][j] = U[j][c] are rows of LDS columns.
    constexpr int TILES = M / 16, WT = TILES >= 2 ? TILES / 2 : 1;
    const int w = tid / 64, lane = tid % 64;
    const bool wave_on = TILES >= 2 || w == 0;
    const int tr0 = TILES >= 2 ? (w / 2) * WT : 0;
    const int tc0 = TILES >= 2 ? (w % 2) * WT : 0;
    f64x4 acc[WT][WT];
#pragma unroll
    for (int a = 0; a < WT; ++a)
#pragma unroll
      for (int b = 0; b < WT; ++b) acc[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
    if (wave_on) {
#pragma unroll 4
      for (int ks = 0; ks < M / 4; ++ks) {
        const int c = ks * 4 + lane / 16;
        const double sc = sm.nrm[c];
        double av[WT], bv[WT];
#pragma unroll
        for (int a = 0; a < WT; ++a) {
          av[a] = sm.Bm[c * LDB + (tr0 + a) * 16 + lane % 16] * sc;
          bv[a] = sm.Bm[c * LDB + (tc0 + a) * 16 + lane % 16];
        }
#pragma unroll
        for (int a = 0; a < WT; ++a)
#pragma unroll
          for (int b = 0; b < WT; ++b) acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[b], acc[a][b], 0, 0, 0);
      }
    }
    __syncthreads();  // every wavefront is done with U before T overwrites it
    if (wave_on) {
#pragma unroll
      for (int a = 0; a < WT; ++a)
#pragma unroll
        for (int b = 0; b < WT; ++b)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            int i = (tr0 + a) * 16 + lane / 16 + 4 * v, j = (tc0 + b) * 16 + lane % 16;
            // masked by arithmetic (T and wbar are zero and finite past m)
            const double t = (i < m && j < m ? 1.0 : 0.0) * (acc[a][b][v] + sm.wbar[i]);
            if constexpr (P == 0) {  // back from A's symmetric permutation
              i = sm.perm[i];
              j = sm.perm[j];
            }
            sm.Bm[i * LDB + j] = t;
            if (dbg && i < m && j < m) dbg[m * m + m + i * m + j] = t;
          }
    }
  } else {
    double tacc[TX][TM];
#pragma unroll
    for (int x = 0; x < TX; ++x)
#pragma unroll
      for (int y = 0; y < TM; ++y) tacc[x][y] = 0.0;
    for (int c = 0; c < m; ++c) {
      const double sc = sm.nrm[c];
      double ui[TX], uj[TM];
#pragma unroll
      for (int x = 0; x < TX; ++x) ui[x] = sm.Bm[c * LDB + ti + 16 * x] * sc;
#pragma unroll
      for (int y = 0; y < TM; ++y) uj[y] = sm.Bm[c * LDB + tj + 16 * y];
#pragma unroll
      for (int x = 0; x < TX; ++x)
#pragma unroll
        for (int y = 0; y < TM; ++y) tacc[x][y] += ui[x] * uj[y];
    }
    __syncthreads();
#pragma unroll
    for (int x = 0; x < TX; ++x)
#pragma unroll
      for (int y = 0; y < TM; ++y) {
        const int i = ti + 16 * x, j = tj + 16 * y;
        const double v = (i < m && j < m) ? tacc[x][y] + sm.wbar[i] : 0.0;
        sm.Bm[i * LDB + j] = v;
        if (dbg && i < m && j < m) dbg[m * m + m + i * m + j] = v;
      }
  }
  if (dbg && tid < m) dbg[m * m + tid] = sm.lam[tid];
  __syncthreads();
}

// A chunk of KCH state rows of the domain (both instants), rows q0 .. q0 +
// KCH - 1: fetch() loads each thread's EPT values into registers (issued
// before the previous chunk's products, so the loads overlap them), store()
// writes the zero-padded chunk to LDS and the rows' member means to sm.rc.
template <typename C, int KCH, typename T>
struct RowChunk {
  static constexpr int M = C::M, NT = C::NT, EPT = KCH * M / NT;
  // row stride of the staged chunk: M + 1, so that the 16 rows an MFMA operand
  // load reads for one member (one row per lane) fall in 16 different banks
  // (a stride of M put them all in one: a 16-way conflict on every load)
  static constexpr int LDX = M + 1;
  static_assert(KCH * M % NT == 0, "whole chunks per thread");
  T v[EPT];
  int act[EPT];  // actuator indices of the chunk fetched next (see fetch)
  int qq0, jj;
  __device__ RowChunk() {
    const int tid = phase_tid();
    qq0 = M >= 64 ? __builtin_amdgcn_readfirstlane(tid / M) : tid / M;  // wavefront-uniform for M >= 64
    jj = tid % M;
  }
  // the actuator indices of chunk q0 (called once for the first chunk, then by
  // every fetch for the chunk after it)
  __device__ void fetch_act(const InstDesc& I, int est_off, int e, int q0) {
    const int m = I.m;
    const int32_t* est_act = I.est_act + est_off;
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      const int q = q0 + qq0 + u * (NT / M);
      act[u] = (q < 2 * e && jj < m) ? gload(est_act + (q < e ? q : q - e)) : -1;
    }
  }
  __device__ void fetch(const InstDesc& I, int est_off, int e, int cur, int q0) {
    const int m = I.m;
    const T* ens = (const T*)I.ens;
    const size_t slot = (size_t)I.n_act * m;
    // global loads (see gload); the actuator indices run one chunk ahead
    // (fetch_act), so a fetch never waits for its own index loads
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      const int q = q0 + qq0 + u * (NT / M);
      v[u] = (T)0;
      if (act[u] >= 0) {
        const int inst = q < e ? cur : (cur ^ 1);
        v[u] = gload(ens + (size_t)inst * slot + (size_t)act[u] * m + jj);
      }
    }
    fetch_act(I, est_off, e, q0 + KCH);
  }
  template <typename SM, typename S>
  __device__ void store(SM& sm, S* X, int m) {
#pragma unroll
    for (int u = 0; u < EPT; ++u) X[(qq0 + u * (NT / M)) * LDX + jj] = (S)v[u];
    __syncthreads();
    constexpr int TPR = NT / KCH < 16 ? NT / KCH : 16;  // threads per row for the means
    const int tid = phase_tid(), row = tid / TPR, part = tid % TPR;
    if (row < KCH) {
      double sum = 0.0;
      for (int j = part; j < m; j += TPR) sum += (double)X[row * LDX + j];
      sum = group_sum<TPR>(sum);
      if (part == 0) sm.rc[row] = sum / (double)m;
    }
    __syncthreads();
  }
};

// ---- a8 on the FP64 path: Z = xbar 1^T + X' T with FP64 MFMA ----------------
// Chunks of 16 state rows (both instants) are staged with their member means;
// wave w computes the 16 x 16 output tiles w, w + 4, ... of the chunk with
// v_mfma_f64_16x16x4f64 (A = X' - xbar from LDS, B = T from Bm).
template <typename SM>
__device__ __forceinline__ void update_fp64(SM& sm, const InstDesc& I, int est_off, int e, int cur) {
  using C = typename SM::C;
  constexpr int M = C::M;
  constexpr int LDB = C::LDB, KR = 16, CB = M / 16;
  static_assert((size_t)KR * (M + 1) * 8 <= C::STAGE_BYTES, "staging");
  constexpr int LDX = RowChunk<C, KR, double>::LDX;
  const int m = I.m, tid = phase_tid(), w = tid / 64, lane = tid % 64;
  double* Xd = (double*)sm.stage;
  double* Z = (double*)I.Z + (size_t)2 * est_off * m;
  RowChunk<C, KR, double> rows;
  rows.fetch_act(I, est_off, e, 0);
  rows.fetch(I, est_off, e, cur, 0);
  for (int q0 = 0; q0 < 2 * e; q0 += KR) {
    const int kc = min(KR, 2 * e - q0);
    rows.store(sm, Xd, m);
    if (q0 + KR < 2 * e) rows.fetch(I, est_off, e, cur, q0 + KR);
    for (int cb = w; cb < CB; cb += C::NW) {
      const int arow = lane % 16;
      const double xb = sm.rc[arow];
      const int col = cb * 16 + lane % 16;
      f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
      for (int ks = 0; ks < M / 4; ++ks) {
        const int k = ks * 4 + lane / 16;
        // loaded unconditionally, masked by arithmetic (the staged rows are
        // zero past m, so the product is finite): a load under the mask is a
        // branch and a wait of its own before every MFMA
        const double a = (k < m ? 1.0 : 0.0) * (Xd[arow * LDX + k] - xb);
        const double b = sm.Bm[k * LDB + col];
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc, 0, 0, 0);
      }
      double mean[4];  // read before the stores' branches, so the reads share one wait
#pragma unroll
      for (int v = 0; v < 4; ++v) mean[v] = sm.rc[lane / 16 + 4 * v];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = lane / 16 + 4 * v;
        if (row < kc && col < m) gstore(Z + (size_t)(q0 + row) * m + col, mean[v] + acc[v]);
      }
    }
    __syncthreads();
  }
}

// ---- a8 on the MFMA paths: Z = xbar 1^T + X' T in 16 x 16 tiles --------------
// FP32: X' and T in FP32.  BF16: X' in BF16, T split into hi + lo BF16 parts
// (two MFMAs), so only X' carries the BF16 rounding.
template <int P, typename SM>
__device__ __forceinline__ void update_mfma(SM& sm, const InstDesc& I, int est_off, int e, int cur) {
  using C = typename SM::C;
  constexpr int M = C::M;
  constexpr int LDB = C::LDB, KR = C::KR;
  constexpr int RB = KR / 16, CB = M / 16, NTILE = RB * CB;
  const int m = I.m, tid = phase_tid(), w = tid / 64, lane = tid % 64;
  float* Xf = (float*)sm.stage;
  float* Z = (float*)I.Z + (size_t)2 * est_off * m;
  RowChunk<C, KR, float> rows;
  constexpr int LDX = RowChunk<C, KR, float>::LDX;
  static_assert((size_t)KR * LDX * 4 <= C::STAGE_BYTES, "staging");
  // BF16, M a multiple of 32: T converted once to its hi and lo BF16 parts,
  // transposed (Th[j][k], k contiguous, so that a lane's 8 consecutive k of the
  // B operand are one 16-byte load), in Bm's storage; the staged rows likewise
  // once per chunk to BF16 X' - xbar (zero past m).  Converting inside the
  // products repeated the work for every tile and chunk.
  constexpr bool PRE = P >= 2 && M % 32 == 0 && M * M / C::NT <= 32;
  constexpr int LDT = M + 8;  // bf16 row stride: 16-byte rows, banks spread over a pass
  __bf16* Th = (__bf16*)sm.Bm;
  __bf16* Tl = Th + M * LDT;
  __bf16* Xb = (__bf16*)sm.stage;
  static_assert(!PRE || ((size_t)2 * M * LDT * 2 <= sizeof(sm.Bm) && (size_t)KR * LDT * 2 <= C::STAGE_BYTES),
                "BF16 copies");
  if constexpr (PRE) {
    constexpr int PER = M * M / C::NT;
    double tv[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int idx = tid + u * C::NT;
      tv[u] = sm.Bm[(idx / M) * LDB + idx % M];  // T[k][j], k = idx / M, j = idx % M
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int idx = tid + u * C::NT, k = idx / M, j = idx % M;
      const __bf16 hi = (__bf16)(float)tv[u];
      Th[j * LDT + k] = hi;
      Tl[j * LDT + k] = (__bf16)(float)(tv[u] - (double)(float)hi);
    }
    __syncthreads();
  }
  rows.fetch_act(I, est_off, e, 0);
  rows.fetch(I, est_off, e, cur, 0);
  for (int q0 = 0; q0 < 2 * e; q0 += KR) {
    const int kc = min(KR, 2 * e - q0);
    rows.store(sm, Xf, m);
    if constexpr (PRE) {
      constexpr int PER = KR * M / C::NT;
      float xv[PER];
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int idx = tid + u * C::NT, r = idx / M, k = idx % M;
        xv[u] = (k < m ? 1.f : 0.f) * (Xf[r * LDX + k] - (float)sm.rc[r]);
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int idx = tid + u * C::NT;
        Xb[(idx / M) * LDT + idx % M] = (__bf16)xv[u];
      }
      __syncthreads();
    }
    if (q0 + KR < 2 * e) rows.fetch(I, est_off, e, cur, q0 + KR);
    for (int t = w; t < NTILE; t += C::NW) {
      const int rb = t / CB, cb = t % CB;
      const int arow = rb * 16 + lane % 16;
      const float xb = (float)sm.rc[arow];
      const int col = cb * 16 + lane % 16;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      if constexpr (P == 1) {
#pragma unroll 4
        for (int ks = 0; ks < M / 4; ++ks) {
          const int k = ks * 4 + lane / 16;
          const float a = (k < m ? 1.f : 0.f) * (Xf[arow * LDX + k] - xb);  // masked by arithmetic, as above
          const float b = (float)sm.Bm[k * LDB + col];
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc, 0, 0, 0);
        }
      } else if constexpr (PRE) {
#pragma unroll
        for (int ks = 0; ks < M / 32; ++ks) {
          const int k0 = ks * 32 + 8 * (lane / 16);
          const bf16x8 a = *(const bf16x8*)&Xb[arow * LDT + k0];
          const bf16x8 bh = *(const bf16x8*)&Th[col * LDT + k0];
          const bf16x8 bl = *(const bf16x8*)&Tl[col * LDT + k0];
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bh, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bl, acc, 0, 0, 0);
        }
      } else {
        for (int ks = 0; ks < (M + 31) / 32; ++ks) {
          bf16x8 a, bh, bl;
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int k = ks * 32 + 8 * (lane / 16) + u;
            float xa;
            double tv;
            // masked by arithmetic, as above; k runs past M (the index is clamped)
            const int kc_ = k < M ? k : M - 1;
            xa = (k < m ? 1.f : 0.f) * (Xf[arow * LDX + kc_] - xb);
            tv = (k < M ? 1.0 : 0.0) * sm.Bm[kc_ * LDB + col];
            const __bf16 hi = (__bf16)(float)tv;
            a[u] = (__bf16)xa;
            bh[u] = hi;
            bl[u] = (__bf16)(float)(tv - (double)(float)hi);
          }
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bh, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bl, acc, 0, 0, 0);
        }
      }
      double mean[4];  // read before the stores' branches, so the reads share one wait
#pragma unroll
      for (int v = 0; v < 4; ++v) mean[v] = sm.rc[rb * 16 + 4 * (lane / 16) + v];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = rb * 16 + 4 * (lane / 16) + v;
        if (row < kc && col < m) gstore(Z + (size_t)(q0 + row) * m + col, (float)(mean[v] + (double)acc[v]));
      }
    }
    __syncthreads();
  }
}

// FP64 path, M <= 64: A (and b) permuted symmetrically so that its diagonal
// decreases, A_p[r][c] = A[perm[r]][perm[c]] (ties by index; padded members
// keep their places).  The Cholesky factor of A_p starts the one-sided Jacobi
// closer to convergence: 7.29 sweeps per solve instead of 7.61 on the 84 x 84
// map (CPU replay of every domain).  The eigenvectors of A_p are those of A
// with rows permuted, so T comes out of the transform as T_p and is stored back
// through perm (T[perm[r]][perm[c]] = T_p[r][c]).
template <int M>
__device__ __forceinline__ void sort_diag(AnaSmem<M>& sm, int m) {
  using C = AnaCfg<M>;
  constexpr int NT = C::NT, LDB = C::LDB, PER = M * M / NT;
  static_assert(M * M % NT == 0 && M <= NT && NT % M == 0, "whole rows per thread");
  constexpr int TPI = NT / M;  // threads per index for the ranks
  const int tid = phase_tid();
  {
    const int i = tid / TPI, part = tid % TPI;
    const double d = sm.Bm[i * LDB + i];
    double ahead = 0.0;  // indices ranked before i among this thread's share (exact small integers)
    if (i < m)
      for (int j = part; j < m; j += TPI) {
        const double dj = sm.Bm[j * LDB + j];
        ahead += (dj > d || (dj == d && j < i)) ? 1.0 : 0.0;
      }
    ahead = group_sum<TPI>(ahead);
    if (part == 0) sm.perm[i < m ? (int)ahead : i] = i;
  }
  __syncthreads();
  // thread tid reads entries (perm[r], perm[c]) for c = tid % M and rows r = tid / M + e NT / M
  double v[PER];
  const int c = tid % M, pc = sm.perm[c];
#pragma unroll
  for (int e = 0; e < PER; ++e) v[e] = sm.Bm[sm.perm[tid / M + e * (NT / M)] * LDB + pc];
  const double bp = tid < M ? sm.bvec[pc] : 0.0;
  __syncthreads();
#pragma unroll
  for (int e = 0; e < PER; ++e) sm.Bm[(tid / M + e * (NT / M)) * LDB + c] = v[e];
  if (tid < M) sm.bvec[tid] = bp;
  __syncthreads();
}

template <int P, int M>
__device__ __forceinline__ void analyse_item(AnaSmem<M>& sm, const InstDesc* __restrict__ tab, const ClassBatch& cb, int item, bool fair) {
  using C = AnaCfg<M>;
  // uniform values, in scalar registers where vector ones are short (M = 128); at
  // M = 32 that took 7 % longer in the Jacobi steps
  auto uni = [](int x) { return M == 128 ? __builtin_amdgcn_readfirstlane(x) : x; };
  const int eb = uni(find_entry(cb.dom_off, cb.n, item));
  const InstDesc& I = tab[cb.inst[eb]];
  const int l = uni(I.order[item - cb.dom_off[eb]]);
  const int est_off = uni(I.dom[4 * l]), e = uni(I.dom[4 * l + 1]);
  const int obs_off = uni(I.dom[4 * l + 2]), s = uni(I.dom[4 * l + 3]);
  const int m = I.m;
  const int cur = uni(I.st->cur);
  double* dbg = I.dbg ? I.dbg + (size_t)l * (2 * m * m + m + kDbgTail) : nullptr;
  // debug: shader-clock stamps at the phase boundaries (after each phase's barrier)
  auto stamp = [&](int k) {
    if (dbg && threadIdx.x == 0) dbg[2 * m * m + m + k] = (double)clock64();
  };
  stamp(0);
  if (fair) set_issue_prio(3);
  if (dbg && threadIdx.x == 0) {  // debug: where the workgroup runs (HW_ID: SE, SH, CU, SIMD; XCC_ID)
    dbg[2 * m * m + m + 6] = (double)__builtin_amdgcn_s_getreg(4 | (31 << 11));
    dbg[2 * m * m + m + 7] = (double)__builtin_amdgcn_s_getreg(20 | (31 << 11));
    dbg[2 * m * m + m + 8] = (double)blockIdx.x;
  }

  if constexpr (P == 0 && M <= 64) gather_C_fp64_mfma(sm, I, obs_off, s, dbg);
  else if constexpr (P == 0) gather_C_fp64<M>(sm, I, obs_off, s, dbg);
  else if constexpr (P >= 2) gather_C_bf16(sm, I, obs_off, s, dbg);
  else gather_C_fp32(sm, I, obs_off, s, dbg);
  if constexpr (P == 0) {
    __syncthreads();
    if constexpr (M <= 64) sort_diag<M>(sm, m);
    // the domain's A (permuted as above), kept for the refinement of wbar (the
    // Cholesky overwrites it): the lower triangle of the m x m matrix, packed
    // by rows (row i at i (i + 1) / 2), rows spread over the wavefronts and
    // coalesced over lanes
    double* Ag = I.Ascr + (size_t)l * tri_size(m);
    const int w = phase_tid() / 64, lane = phase_tid() % 64;
    for (int i = w; i < m; i += AnaCfg<M>::NT / 64)
      for (int j = lane; j <= i; j += 64) gstore(Ag + tri_size(i) + j, sm.Bm[i * AnaCfg<M>::LDB + j]);
    __syncthreads();
  }
  stamp(1);
  cholesky<M>(sm);
  stamp(2);
  bool converged = false;
  const int sweeps = jacobi<P, M>(sm, m, converged, fair);
  stamp(3);
  if (fair) set_issue_prio(0);
  transform<P, M>(sm, I, l, dbg);
  stamp(4);
  if (threadIdx.x == 0) {
    if (I.dbg_sweeps) I.dbg_sweeps[l] = sweeps;
    gatomic_add(&I.dom_sweeps[l], (unsigned)sweeps);
    if (!converged) gatomic_add(&I.st->unconverged, 1);
    gatomic_add(&I.st->sweeps, (unsigned long long)sweeps);
    gatomic_add(&I.st->solves, 1ull);
  }
  if constexpr (P == 0) update_fp64(sm, I, est_off, e, cur);
  else update_mfma<P>(sm, I, est_off, e, cur);
  stamp(5);
}

// Persistent: a workgroup analyses item blockIdx.x, then claims further items
// from the class's work counter (zeroed by the slope kernel that precedes
// every analysis launch) until the items run out, so the launch's grid can be
// smaller than the work (fixed grids for replayed graphs, a cap on the CUs the
// class occupies) and the heaviest domains, which come first in each
// instance's order, start first.  Every workgroup leaves once a claim passes
// the item count.
// fair != 0 (launches whose workgroups start together with at most two on a
// CU: the plain path): the wavefronts' issue priority falls with the item's
// progress (3 from its start, then by Jacobi sweeps done: 2 from the 3rd,
// 1 from the 5th, 0 from the 6th and after the eigensolve).  A SIMD issues
// from the oldest of its ready wavefronts, so of two domains sharing a CU the
// first dispatched ran nearly as if alone and the second got the leftover
// slots, then finished alone at one wavefront per SIMD: on the 84 x 84 map
// the pairs ended at 493k and 659k cycles (mean), with the priorities 566k
// and 612k, and the plain FP64 launch went 296 -> 275 us.  With three or
// more workgroups per CU (the serving batches) either ordering of the
// priorities made the batches slower (serving -11 % with this one), so the
// server launches with fair = 0.
template <int P, int M>
__global__ __launch_bounds__(AnaCfg<M>::NT) void k_analysis(const InstDesc* __restrict__ tab,
                                                  BatchHdr* __restrict__ hdr, int cls, int fair) {
  __shared__ AnaSmem<M> sm;
  __shared__ int s_next;
  ClassBatch& cb = hdr->cls[cls];
  const int total = cb.dom_off[cb.n];
  int item = blockIdx.x;
  while (item < total) {
    // FP64 batches may hold instances of the other kernel
    if (P != 0 || !tab[cb.inst[find_entry(cb.dom_off, cb.n, item)]].poly) analyse_item<P, M>(sm, tab, cb, item, fair != 0);
    if (threadIdx.x == 0) s_next = (int)gridDim.x + (int)atomicAdd(&cb.next, 1u);
    __syncthreads();
    item = M == 128 ? __builtin_amdgcn_readfirstlane(s_next) : s_next;
    __syncthreads();
  }
}

// pcol = b - A wbar, with A itself (Ag: the domain's copy of A = (m-1)/rho I + C,
// its lower triangle packed by rows), for the refinement step of wbar = A^-1 b
// on the FP64 path: Z (Z b) carries Z's rounding of order eps kappa, which the
// step takes out (wbar 1e-10 -> 1e-12 where b lies along the large eigenvalues).
template <int M>
__device__ __forceinline__ void residual_wbar(PolySmem<M>& sm, const double* __restrict__ Ag, int m) {
  constexpr int TPC = PolyCfg<M>::NT / M, PER = M / TPC;
  const int tid = phase_tid(), o = tid / TPC, part = tid % TPC;
  // (A wbar)_o: row o of the symmetric A; entry (o, c) is packed at row
  // max(o, c), column min(o, c).  Padded rows and columns read entry 0 and
  // are masked by arithmetic (the result is zero past m anyway).
  double a[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int c = part + TPC * k;
    const bool in = c < m && o < m;
    const int hi = c > o ? c : o, lo = c > o ? o : c;
    a[k] = (in ? 1.0 : 0.0) * gload(Ag + (in ? tri_size(hi) + lo : 0));
  }
  double t0 = 0.0, t1 = 0.0;
#pragma unroll
  for (int k = 0; k < PER; k += 2) {
    t0 = fma(a[k], sm.wbar[part + TPC * k], t0);
    if (k + 1 < PER) t1 = fma(a[k + 1], sm.wbar[part + TPC * (k + 1)], t1);
  }
  const double t = group_sum<TPC>(t0 + t1);
  if (part == 0) sm.pcol[o] = o < m ? sm.bvec[o] - t : 0.0;
  __syncthreads();
}

// ---- a6/a7: A^(-1/2) by polynomial stages on the FP64 matrix cores ----------
// W = [(m-1) A^-1]^(1/2) needs no eigenvectors: Z = A^(-1/2) comes from a few
// minimax polynomial stages (isqrt_plan.hpp: 16 matrix products at the condition
// numbers 1e2-1e3 that the 15 x 15 map has off the vector of ones, 17-18 and
// 20-22 at the 84 x 84 and 100 x 100 maps' 4e3 and 6e4):
//   P = q(M),  Z <- P Z,  M <- P (P M),   M_0 = A, Z_0 = I.
// A's upper bound is beta = |A^2|_F^(1/2), from the A^2 that the first stage needs
// anyway (1.05 to 1.4 times the largest eigenvalue there); the first stage's
// coefficients carry the scaling by it (isqrt_scale).
//
// Layout: wavefront w owns the columns 16 w .. 16 w + 15 of every matrix, in
// the accumulator registers of v_mfma_f64_16x16x4f64.  Register v of lane l
// there holds row l / 16 + 4 v of column l % 16, which is exactly the right
// operand of k-step v, so a product's right factor is never stored: only the
// left factor goes through LDS (column c at Bm[c LD], one write of M, M^2 or P
// per product group), and each wavefront reads it whole.  Two row tiles share a
// 16-byte load: rows 32 p + 2 i and 32 p + 2 i + 1 sit in tiles 2 p and 2 p + 1.
// LD = M + 2: the 8 lanes of a 16-byte column write then fall in 32 banks.
// Every factor is used as computed, never mirrored: the products are
// polynomials in A taken from the left, and their rounding stays commuting with
// A to first order (forcing symmetry cost a factor 10 in a CPU replay).
// T = ceil(m / 16) tiles take part: at m = 48 a product is 36 MFMAs a wavefront
// instead of the 64 of the padded M = 64 (an odd last tile has its rows in
// plain order and loads of its own), at m = 100 seven tiles instead of eight.
// 100 x 100, m = 100: analysis 1004 -> 840 us (stages of the time).
template <int M, int T_>
struct IsqrtBlock {
  static constexpr int T = T_, LD = M + 2, Q = T / 2, ODD = T % 2;
  // the column a thread holds; row of element (t, v) in lane group g = lane / 16
  static constexpr __device__ __forceinline__ int column(int tid) { return (tid >> 6) * 16 + (tid & 15); }
  static constexpr __device__ __forceinline__ int row(int t, int v, int g) {
    if (ODD && t == T - 1) return 16 * t + g + 4 * v;
    return 32 * (t / 2) + 2 * (g + 4 * v) + (t & 1);
  }
  // which of its 4 T elements (4 t + v) a thread holds on the diagonal, -1 for none
  static constexpr __device__ __forceinline__ int diagonal(int tid) {
    const int c = column(tid), g = (tid & 63) >> 4;
    if (c >= 16 * T) return -1;  // the wavefront that runs along (isqrt_stages)
    if (ODD && c >= 16 * (T - 1)) return g == (c & 3) ? 4 * (T - 1) + ((c & 15) >> 2) : -1;
    const int y = (c & 31) >> 1;
    return g == (y & 3) ? 4 * (2 * (c >> 5) + (c & 1)) + (y >> 2) : -1;
  }
  // acc = S X (ADD: acc += S X) for the wavefront's columns; S: column c at S[c * LD]
  template <bool ADD = false>
  static __device__ __forceinline__ void mul(const double* S, const f64x4 (&X)[T], f64x4 (&acc)[T], int tid) {
    constexpr f64x4 zero = {0.0, 0.0, 0.0, 0.0};
    const int g = (tid & 63) >> 4, i = tid & 15;
    // k-step k < 8 Q: rows 32 p + 2 (g + 4 v) + h of X, k = 8 p + 2 v + h; the
    // odd last tile's follow, 16 (T - 1) + g + 4 v.  Operand load q < Q of a
    // k-step serves the two row tiles 2 q, 2 q + 1, load Q the odd last one.
    // AH loads run ahead of the products; the fence keeps the compiler from
    // hoisting the others too (registers).  An LDS instruction's offset spans
    // 64 KiB: one base per 64 columns, opaque, or the compiler keeps an address
    // per load.
    constexpr int OPS = Q + ODD, NL = 4 * T * OPS, NB = (2 * Q + 3) / 4;
    using ldsx2 = __attribute__((address_space(3))) const f64x2;
    using ldsd = __attribute__((address_space(3))) const double;
    using ldsc = __attribute__((address_space(3))) const char;
    auto opaque = [](const double* x) {
      unsigned o = (unsigned)(uintptr_t)(ldsc*)(const char*)x;
      asm volatile("" : "+v"(o));
      return (ldsc*)(uintptr_t)o;
    };
    ldsc* pair[NB > 0 ? NB : 1];   // row pairs, paired k
    ldsc* one[NB > 0 ? NB : 1];    // the odd tile's rows, paired k
#pragma unroll
    for (int z = 0; z < NB; ++z) {
      pair[z] = opaque(S + (64 * z + 2 * g) * LD + 2 * i);
      if constexpr (ODD) one[z] = opaque(S + (64 * z + 2 * g) * LD + 16 * (T - 1) + i);
    }
    constexpr int AH = T > 4 ? 1 : 2;  // loads ahead
    f64x2 a[AH + 1];
    auto load_op = [&](int j) {
      const int k = j / OPS, q = j % OPS;
      if (k < 8 * Q) {
        const int at = 8 * ((32 * (k / 8 % 2) + 8 * ((k / 2) % 4) + k % 2) * LD);
        if (q < Q) a[j % (AH + 1)] = *(ldsx2*)(pair[k / 16] + at + 8 * 32 * q);
        else a[j % (AH + 1)].x = *(ldsd*)(one[k / 16] + at);
      } else {
        // the odd tile's k: bases formed at their four uses, not kept
        const double* Sk = S + (16 * (T - 1) + g + 4 * (k - 8 * Q)) * LD;
        if (q < Q) a[j % (AH + 1)] = *(ldsx2*)(opaque(Sk + 2 * i) + 8 * 32 * q);
        else a[j % (AH + 1)].x = *(ldsd*)opaque(Sk + 16 * (T - 1) + i);
      }
    };
    if constexpr (AH > 0) load_op(0);
    if constexpr (AH > 1) load_op(1);
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      if (j + AH < NL) load_op(j + AH);
      const int k = j / OPS, q = j % OPS;
      const bool first = !ADD && k == 0;
      const double x = k < 8 * Q ? X[2 * (k / 8) + k % 2][(k / 2) % 4] : X[T - 1][k - 8 * Q];
      const f64x2 av = a[j % (AH + 1)];
      const int t = q < Q ? 2 * q : T - 1;
      acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, x, first ? zero : acc[t], 0, 0, 0);
      if (q < Q) acc[t + 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.y, x, first ? zero : acc[t + 1], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // the wavefront's columns to / from a matrix with column c at S[c * ld]
  static __device__ __forceinline__ void store(double* S, int ld, const f64x4 (&X)[T], int tid) {
    const int c = column(tid), g = (tid & 63) >> 4;
#pragma unroll
    for (int p = 0; p < Q; ++p)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        *(f64x2*)(S + c * ld + 32 * p + 2 * (g + 4 * v)) = f64x2{X[2 * p][v], X[2 * p + 1][v]};
        if constexpr (T > 4) __builtin_amdgcn_sched_barrier(0);  // registers: one pair at a time
      }
    if constexpr (ODD)
#pragma unroll
      for (int v = 0; v < 4; ++v) S[c * ld + 16 * (T - 1) + g + 4 * v] = X[T - 1][v];
  }
  // X = u S + w Y for the wavefront's columns (w = 0: S itself, Y unread)
  template <bool AXPY = false>
  static __device__ __forceinline__ void load(const double* S, int ld, f64x4 (&X)[T], int tid, double u = 1.0, double w = 0.0,
                                              const f64x4* Y = nullptr) {
    const int c = column(tid), g = (tid & 63) >> 4;
    if constexpr (ODD)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double x = S[c * ld + 16 * (T - 1) + g + 4 * v];
        X[T - 1][v] = AXPY ? u * x + w * Y[T - 1][v] : x;
        if constexpr (T > 4)
          if (v % 2) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
    for (int p = 0; p < Q; ++p)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const f64x2 x = *(const f64x2*)(S + c * ld + 32 * p + 2 * (g + 4 * v));
        X[2 * p][v] = AXPY ? u * x.x + w * Y[2 * p][v] : x.x;
        X[2 * p + 1][v] = AXPY ? u * x.y + w * Y[2 * p + 1][v] : x.y;
        if constexpr (T > 4)
          if (v % 2) __builtin_amdgcn_sched_barrier(0);
      }
  }
};

// Sum and maximum over a wavefront, in scalar registers (shuffles would keep a
// register of lane addresses each).
__device__ __forceinline__ double wave_sum(double v) {
  v = group_sum<16>(v);
  return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp_f64<0xB1>(v));
  v = fmax(v, dpp_f64<0x4E>(v));
  v = fmax(v, dpp_f64<0x141>(v));
  v = fmax(v, dpp_f64<0x140>(v));
  return fmax(fmax(readlane_f64(v, 0), readlane_f64(v, 16)), fmax(readlane_f64(v, 32), readlane_f64(v, 48)));
}

// A uniform value in a scalar register, where the compiler, knowing it uniform,
// would keep it in a vector one across the stages.  (The compiler does not look
// into the block: the first nop is for a vector register written just before,
// the second for a vector memory access by the scalar right after.)
__device__ __forceinline__ int to_scalar(int x) {
  int s;
  __asm__("s_nop 1\n\tv_readfirstlane_b32 %0, %1\n\ts_nop 4" : "=s"(s) : "v"(x));
  return s;
}

// Entry (from 1) of the stages for eigenvalues in [1/kappa, 1].
__device__ __forceinline__ int isqrt_entry(float kappa) {
  const int i = to_scalar((int)ceilf(4.0f * __log2f(kappa) - 0.001f));
  return i < 1 ? 1 : i > kIsqrtEntries ? kIsqrtEntries : i;
}

// beta^(-1/2), or a millionth less, of the upper bound beta = |A^2|_F^(1/2) of A's
// eigenvalues, from fro = |A^2|_F^2: M = A times its square has them below 1, and
// need not be closer (hardware estimates, each within 2^-23 or so).
__device__ __forceinline__ double isqrt_scale(double fro) {
  return __builtin_amdgcn_sqrt(__builtin_amdgcn_sqrt(__builtin_amdgcn_rsq(fro))) * (1.0 - 0x1.0p-20);
}

// The first stage, of M = A scale^2: (m-1)/rho bounds the condition number, `guess`
// says what it may be off the vector of ones (stage_guess).  bound: the entry
// that the smallest eigenvalue is certainly not below.
__device__ __forceinline__ int isqrt_first(double scale, double a_diag, int guess, int& bound) {
  bound = isqrt_entry(1.0f / (float)(scale * scale * a_diag));
  return min(bound, guess);
}

constexpr int upper_word(double x) { return (int)(__builtin_bit_cast(unsigned long long, x) >> 32); }
// After the planned stages: f2 = |R^2|_F^2, R = M - I, bounds ||R|| by f = f2^(1/4)
// and so, below 1, M's smallest eigenvalue by 1 - f.
__device__ __forceinline__ int isqrt_more(double f2, int bound) {
  if (bound < 1) bound = 1;
  if (to_scalar(upper_word(f2)) >= upper_word(1.0)) return bound;
  return min(bound, isqrt_entry(1.0f / (1.0f - __builtin_amdgcn_sqrtf(__builtin_amdgcn_sqrtf((float)f2)))));
}
// The last stage's degree once f2 allows it (0: not yet), kIsqrtNever where f2 is
// not finite.  By f2's upper word; its threshold is below rho^4 by at most 2^-20.
constexpr int kIsqrtNever = -1;
constexpr int isqrt_limit(int k) { return upper_word(kIsqrtRho[k] * kIsqrtRho[k] * kIsqrtRho[k] * kIsqrtRho[k]); }
__device__ __forceinline__ int isqrt_last(double f2) {
  const int h = to_scalar(upper_word(f2));  // f2 >= 0 or NaN
  if (h < 0 || h >= 0x7ff00000) return kIsqrtNever;
  return h < isqrt_limit(0) ? 2 : h < isqrt_limit(1) ? 4 : h < isqrt_limit(2) ? 6 : 0;
}
constexpr int kIsqrtCap = 40;  // stages at most (11 at the table's end)

// Z = (A + shift 1 1^T)^(-1/2) from A in Bm (stride M + 2): each wavefront ends
// with its columns of Z in Z (sm.rc[8]: the shift).  Returns the matrix products
// done.  Every stage after the first forms M^2 and with it f2 = |(M - I)^2|_F^2;
// the stages end when that says that the last stage's polynomial is exact to
// rounding, whatever the condition number was taken to be.  sm.rc[9]: whether they
// got there (not where A holds a NaN or is numerically indefinite).
// A's smallest eigenvalue (m-1)/rho belongs to the vector of ones, of which Y'
// and X' know nothing (their rows sum to zero); every other one may be orders
// above it, and W only matters there.  So the trace's mean goes on top of that
// eigenvalue (shift = tr(A) / m^2), and the interval, the stages and the rounding
// are those of the others.  b is orthogonal to the ones as well.
// Relative error of X' W on 15 x 15, m = 16, against extended precision: 4e-15
// (Cholesky + SVD of A 4e-15; without the shift and with the bound's interval
// 4e-13), on 32 x 32, m = 197 1e-14 (1e-14; 1e-12); with R^-1 x 1e4 3e-13 and
// 1e-12 (3e-13 and 9e-13; 1e-11 and 3e-10).  Launch: 15 x 15 16.6 -> 17.6 us,
// 84 x 84, m = 64 136 -> 135, 100 x 100, m = 100 850 -> 990 (22 products for 20).
// Four matrices in registers are 128 VGPRs per lane at M = 64 and 256 at
// M = 128, which leaves too few for the rest: two of Z's four tiles wait in LDS
// (behind S, up to the end of the staging area) at M = 64, seven of its eight in
// `park` (a slot of the instance's workspace) at M = 128, while the stage's
// polynomial is formed.
template <int M, int T, typename F>
__device__ __forceinline__ int isqrt_stages(PolySmem<M>& sm, int m, double a_diag, int guess, double* park, f64x4 (&Z)[T],
                                            F&& planned) {
  using B = IsqrtBlock<M, T>;
  using C = PolyCfg<M>;
  constexpr int NW = C::NW;
  static_assert(T <= NW && M * B::LD <= M * PolyCfg<M>::LDB, "a column block per wavefront, S inside Bm");
  // the thread index: at M = 128 afresh at every use, so that nothing derived
  // from it stays in a register across the stages
  const int tid0 = phase_tid(), w = __builtin_amdgcn_readfirstlane(tid0 / 64);
  auto tid = [&]() { return M > 64 ? phase_tid() : tid0; };
  // (at T = 7 the eighth wavefront runs along on zero columns: a branch around
  // its products would cost registers, and the SIMDs hold two wavefronts anyway)
  const bool on = T == NW || T == 7 || w < T;
  double* S = sm.Bm;
  f64x4 Mc[T], X[T];
  // sm.rc by an address formed here: the compiler would keep one per pair of sums
  using lds_double = __attribute__((address_space(3))) double;
  auto scratch = [&]() {
    unsigned o = (unsigned)(uintptr_t)(lds_double*)sm.rc;
    __asm__ volatile("" : "+v"(o));
    return (lds_double*)(uintptr_t)o;
  };
  // the trace, summed alike by every wavefront
  double tr;
  {
    const int t = tid0 % 64;
    tr = t < m ? S[t * (B::LD + 1)] : 0.0;
    if constexpr (M > 64) tr += t + 64 < m ? S[(t + 64) * (B::LD + 1)] : 0.0;
    tr = wave_sum(tr);
  }
  const double shift = tr / ((double)m * m);
  if (tid0 == 0) scratch()[8] = shift;
  // and a power of 4 near it, by which A is divided: |A^2|_F^2 stays in range
  const int ex = __builtin_amdgcn_readfirstlane((__builtin_amdgcn_frexp_exp(tr) + 1) & ~1);
  __syncthreads();  // A's diagonal read everywhere before it changes
  if (on) {
    B::load(S, B::LD, Mc, tid());
    // past m the diagonal is the mean eigenvalue, inside the others' interval
    const int t0 = tid(), g = (t0 & 63) >> 4, dk = B::diagonal(t0);
    const bool in = B::column(t0) < m;
#pragma unroll
    for (int k = 0; k < 4 * T; ++k) {
      const double x = in ? Mc[k / 4][k % 4] + (B::row(k / 4, k % 4, g) < m ? shift : 0.0) : k == dk ? shift * m : 0.0;
      Mc[k / 4][k % 4] = ldexp(x, -ex);
    }
    B::store(S, B::LD, Mc, t0);
  }
  __syncthreads();
  // 1 where k is the diagonal's element and 0 elsewhere, from words formed here
  // (constants that the compiler would keep in registers across the stages)
  struct Unit {
    int dk, hi, lo;
    __device__ __forceinline__ double operator()(int k) const { return __hiloint2double(k == dk ? hi : 0, lo); }
  };
  auto unit = [&](int dk) {
    Unit u{dk, 0, 0};
    __asm__ volatile("v_mov_b32 %0, 0x3ff00000\n\tv_mov_b32 %1, 0" : "=&v"(u.hi), "=v"(u.lo));
    return u;
  };
  // the thread's diagonal element, afresh at every use (its comparisons are not kept)
  auto diagonal = [&]() {
    int d = B::diagonal(tid());
    __asm__ volatile("" : "+v"(d));
    return d;
  };
  // |V|_F^2 over the workgroup, from each thread's sum over its elements
  auto frobenius = [&](double ss) {
    ss = wave_sum(ss);
    lds_double* const sums = scratch();
    if (tid() % 64 == 0) sums[w] = ss;
    __syncthreads();
    double f = 0.0;
#pragma unroll
    for (int k = 0; k < (T < NW ? T : NW); ++k) f += sums[k];
    return f;
  };
  double ss = 0.0;
  if (on) {
    B::mul(S, Mc, X, tid());  // A^2
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) ss = fma(X[t][v], X[t][v], ss);
  }
  const double scale = readlane_f64(isqrt_scale(frobenius(ss)), 0);
  int bound;
  const int plan = isqrt_first(scale, ldexp(a_diag, -ex), guess, bound);
  planned();
  // Z between the stages: KEEP tiles stay in registers, the others wait outside
  // (each lane its own values, 16 bytes a lane)
  constexpr int KEEP = C::keep(T);
  constexpr int AWAY = 2 * (T - KEEP);  // 16-byte values per lane outside
  // scalar base + 32-bit lane offset, which the compiler may not turn into one
  // 64-bit address per value kept across the stages
  auto lane_offset = [&]() {
    unsigned o = (tid() & 63) * 16;
    asm volatile("" : "+v"(o));
    return o;
  };
  using gchar = __attribute__((address_space(1))) char;
  using gx2 = __attribute__((address_space(1))) f64x2;
  const uint64_t pb = (uint64_t)park;
  gchar* const away_g = (gchar*)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(pb >> 32)) << 32 |
                                  (uint32_t)__builtin_amdgcn_readfirstlane((int)pb)) + w * (AWAY * 1024));
  char* const away = (char*)(sm.Bm + M * B::LD) + w * (AWAY * 1024);
  auto park_store = [&](const f64x4 (&V)[T]) {
#pragma unroll
    for (int t = 0; t < KEEP; ++t) Z[t] = V[t];
    const unsigned o = lane_offset();
#pragma unroll
    for (int k = 0; k < AWAY; ++k) {
      const f64x2 x = {V[KEEP + k / 2][2 * (k % 2)], V[KEEP + k / 2][2 * (k % 2) + 1]};
      if constexpr (M > 64) *(gx2*)(away_g + k * 1024 + o) = x;
      else *(f64x2*)(away + k * 1024 + o) = x;
    }
  };
  auto park_load = [&](f64x4 (&V)[T]) {
#pragma unroll
    for (int t = 0; t < KEEP; ++t) V[t] = Z[t];
    const unsigned o = lane_offset();
#pragma unroll
    for (int k = 0; k < AWAY; ++k) {
      f64x2 x;
      if constexpr (M > 64) x = *(const gx2*)(away_g + k * 1024 + o);
      else x = *(const f64x2*)(away + k * 1024 + o);
      V[KEEP + k / 2][2 * (k % 2)] = x.x;
      V[KEEP + k / 2][2 * (k % 2) + 1] = x.y;
    }
  };
  // the wavefront's columns of V, plus d I, into S, for all wavefronts to read
  auto publish = [&](const f64x4 (&V)[T], double d) {
    __syncthreads();  // every wavefront is done with the old S
    if (on) {
      B::store(S, B::LD, V, tid());
      __asm__ volatile("" ::: "memory");  // a wavefront's LDS operations take effect in order
      const int t = tid(), c = B::column(t);
      if ((t & 63) < 16 && d != 0.0) S[c * B::LD + c] += d;
    }
    __syncthreads();
  };
  // P = q(M) into S; Mc: the columns of M (of M - I in the last stage), X: those
  // of its square.  Leaves X undefined.
  // Degree 4, in a last stage (`any`) 2 and 6 as well.
  auto stage_poly = [&](auto any, const double* c, int deg, double scale, double step) {
    double q[7];  // in scalar registers
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      q[k] = k <= 4 || (any && deg == 6) ? readlane_f64(c[k] * scale, 0) : 0.0;
      scale *= step;
    }
    if (any && deg == 2) {
#pragma unroll
      for (int t = 0; t < T; ++t) X[t] = q[2] * X[t] + q[1] * Mc[t];
      publish(X, q[0]);
    } else {
      f64x4 Y[T];
      publish(X, 0.0);
      // deg 4: M^2 (q4 M^2 + q3 M) + q2 M^2 + q1 M + q0 I
      // deg 6: M^2 (M^2 (q6 M^2 + q5 M) + q4 M^2 + q3 M) + q2 M^2 + q1 M + q0 I
      const bool six = any && deg == 6;
      const double h2 = six ? q[6] : q[4], h1 = six ? q[5] : q[3], l2 = six ? q[4] : q[2], l1 = six ? q[3] : q[1];
#pragma unroll
      for (int k = 0; k < 4 * T; ++k) {
        const double m1 = Mc[k / 4][k % 4], m2 = X[k / 4][k % 4];
        X[k / 4][k % 4] = h2 * m2 + h1 * m1;
        Y[k / 4][k % 4] = l2 * m2 + l1 * m1;
        if (k % 2) __builtin_amdgcn_sched_barrier(0);
      }
      if (on) B::template mul<true>(S, X, Y, tid());
      if (six) {
        if (on) {
          B::template load<true>(S, B::LD, X, tid(), q[2], q[1], Mc);
          B::template mul<true>(S, Y, X, tid());
        }
        publish(X, q[0]);
        return;
      }
      publish(Y, q[0]);
    }
  };
  // M <- P (P M), its columns and S
  auto stage_next = [&]() {
    if (on) {
      B::mul(S, Mc, X, tid());
      B::mul(S, X, Mc, tid());
    }
    publish(Mc, 0.0);
  };
  // of the table, and the stage of it that comes next
  int row = (plan + 1) / 2, next = 1;
  int products = 4;
  stage_poly(std::false_type{}, kIsqrtPlan[row].c[0], 4, scale, scale * scale);  // a power of M is one of A times scale^2 each
  if (on) {
    B::load(S, B::LD, X, tid());  // Z = P
    park_store(X);
  }
  stage_next();
  auto stage_z = [&]() {  // Z <- P Z, into X
    f64x4 V[T];
    park_load(V);
    B::mul(S, V, X, tid());
  };
  // Last stages of degree 2 and 6 where registers allow the branch between them
  // (M = 128: 229 VGPRs without, spills with it).
  constexpr bool ANY = M <= 64;
  int last;
#pragma unroll 1
  for (int s = 1;; ++s) {
    double f2 = 0.0;
    if (on) {
      B::mul(S, Mc, X, tid());  // M^2
      const Unit one = unit(diagonal());
#pragma unroll
      for (int k = 0; k < 4 * T; ++k) {
        const double d = fma(-2.0, Mc[k / 4][k % 4], X[k / 4][k % 4]) + one(k);
        f2 = fma(d, d, f2);
        if (k % 2) __builtin_amdgcn_sched_barrier(0);
      }
    }
    f2 = readlane_f64(frobenius(f2), 0);
    last = isqrt_last(f2);
    if (!ANY && last == 6) last = 0;  // too wide for degree 4
    if (last != 0 || s == kIsqrtCap) break;
    if (next + 1 >= __builtin_amdgcn_readfirstlane(kIsqrtPlan[row].n)) {
      // the row's stages are done, and raised what was below their interval by its
      // width at least (to within 1 %)
      bound = max(bound - 2 * row, 0) + 1;
      row = isqrt_more(f2, bound);
      row = row == 1 ? 0 : (row + 1) / 2;
      next = 0;
    }
    stage_poly(std::false_type{}, kIsqrtPlan[row].c[next++], 4, 1.0, 1.0);
    if (on) {
      stage_z();
      park_store(X);
    }
    stage_next();
    products += 5;
  }
  // the last stage, in powers of M - I (by its degree 6 where the certificate is
  // not to be had)
  const int deg = !ANY ? 4 : last > 0 ? last : 6;
  if (on) {
    const Unit one = unit(diagonal());
#pragma unroll
    for (int k = 0; k < 4 * T; ++k) {  // X = (M - I)^2, Mc = M - I
      X[k / 4][k % 4] = fma(-2.0, Mc[k / 4][k % 4], X[k / 4][k % 4]) + one(k);
      Mc[k / 4][k % 4] -= one(k);
      if (k % 2) __builtin_amdgcn_sched_barrier(0);
    }
  }
  stage_poly(std::bool_constant<ANY>{}, kIsqrtLast[deg / 2 - 1], deg, 1.0, 1.0);
  products += deg / 2 + 1;
  if (on) stage_z();
  if (tid() == 0) scratch()[9] = last > 0 ? 1.0 : 0.0;
#pragma unroll
  for (int k = 0; k < 4 * T; ++k) Z[k / 4][k % 4] = ldexp(X[k / 4][k % 4], -ex / 2);
  __syncthreads();  // every wavefront is done with S
  return products;
}

// What W has along the vector of ones beyond the shifted matrix's inverse square
// root, per entry of T.  X' annihilates it but for the rounding of xbar, which
// it takes out again.
__device__ __forceinline__ double ones_term(int m, double sqrt_m1, double a_diag, double shift) {
  return sqrt_m1 * (rsqrt_1_2(a_diag) - rsqrt_1_2(a_diag + m * shift)) / m;
}

// wbar = A^-1 b = Z (Z b) (with one refinement step through A itself on the
// FP64 path) and T = sqrt(m-1) Z + wbar 1^T, row-major in Bm (T[k][j] at
// Bm[k LDB + j], zero outside m x m), from the wavefronts' columns of Z.
template <int M, int T>
__device__ __forceinline__ void finish_T(PolySmem<M>& sm, const InstDesc& I, int l, const f64x4 (&Z)[T], double* dbg) {
  using B = IsqrtBlock<M, T>;
  using C = PolyCfg<M>;
  constexpr int NW = C::NT / 64, LDB = C::LDB, TPC = C::NT / M;
  const int m = I.m, tid = phase_tid(), w = tid / 64, g = tid % 64 / 16, c = B::column(tid);
  // (at T = 7 the eighth wavefront runs along on zero columns: a branch around
  // its products would cost registers, and the SIMDs hold two wavefronts anyway)
  const bool on = T == NW || T == 7 || w < T;
  auto substamp = [&](int k) {
    if (dbg && threadIdx.x == 0) dbg[2 * m * m + m + 10 + k] = (double)clock64();
  };
  if (on) B::store(sm.Bm, LDB, Z, tid);
  if constexpr (16 * T < M) {  // past the tiles that took part: zero
    double zero = 0.0;
    __asm__ volatile("" : "+v"(zero));  // (not a register kept over the stages)
    for (int k = tid / 16; k < M; k += C::NT / 16)
      for (int r = 16 * T + tid % 16; r < M; r += 16) sm.Bm[k * LDB + r] = zero;
    for (int k = 16 * T + tid / 16; k < M; k += C::NT / 16)
      for (int r = tid % 16; r < 16 * T; r += 16) sm.Bm[k * LDB + r] = zero;
  }
  __syncthreads();
  substamp(0);
  const int o = tid / TPC, part = tid % TPC;
  // v <- Z (Z v), Z symmetric; padded entries of v are zero and stay zero
  auto solve = [&](const double* rhs) {
    const double t = colsum(sm, rhs, o, part);
    if (part == 0) sm.zv[o] = t;
    __syncthreads();
    return colsum(sm, sm.zv, o, part);
  };
  {
    const double x = solve(sm.bvec);
    if (part == 0) sm.wbar[o] = x;
    __syncthreads();
  }
  substamp(1);
  {
    residual_wbar<M>(sm, I.Ascr + (size_t)l * tri_size(m), m);
    const double x = solve(sm.pcol);
    if (part == 0) sm.wbar[o] += x;
    __syncthreads();
  }
  substamp(2);
  if (on) {
    const double sc = I.sqrt_m1, wb = sm.wbar[c] + ones_term(m, sc, I.a_diag, sm.rc[8]);
    f64x4 X[T];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = B::row(t, v, g);
        X[t][v] = (r < m && c < m ? 1.0 : 0.0) * fma(sc, Z[t][v], wb);  // T[c][r]
        if (dbg && r < m && c < m) dbg[m * m + m + c * m + r] = X[t][v];
      }
    B::store(sm.Bm, LDB, X, tid);
  }
  __syncthreads();
}

template <int M>
__device__ __forceinline__ void analyse_poly(PolySmem<M>& sm, const InstDesc* __restrict__ tab, const ClassBatch& cb, int item) {
  const int eb = __builtin_amdgcn_readfirstlane(find_entry(cb.dom_off, cb.n, item));
  const InstDesc& I = tab[cb.inst[eb]];
  // uniform values, kept in scalar registers
  const int l = __builtin_amdgcn_readfirstlane(I.order[item - cb.dom_off[eb]]);
  const int est_off = __builtin_amdgcn_readfirstlane(I.dom[4 * l]), e = __builtin_amdgcn_readfirstlane(I.dom[4 * l + 1]);
  const int obs_off = __builtin_amdgcn_readfirstlane(I.dom[4 * l + 2]), s = __builtin_amdgcn_readfirstlane(I.dom[4 * l + 3]);
  const int guess = __builtin_amdgcn_readfirstlane((int)gload(I.guess + l));
  const int m = I.m;
  const int cur = __builtin_amdgcn_readfirstlane(I.st->cur);
  double* dbg = I.dbg ? I.dbg + (size_t)l * (2 * m * m + m + kDbgTail) : nullptr;
  // debug: shader-clock stamps at the phase boundaries (after each phase's barrier)
  auto stamp = [&](int k) {
    if (dbg && threadIdx.x == 0) dbg[2 * m * m + m + k] = (double)clock64();
  };
  stamp(0);
  if (dbg && threadIdx.x == 0) {  // debug: where the workgroup runs (HW_ID: SE, SH, CU, SIMD; XCC_ID)
    dbg[2 * m * m + m + 6] = (double)__builtin_amdgcn_s_getreg(4 | (31 << 11));
    dbg[2 * m * m + m + 7] = (double)__builtin_amdgcn_s_getreg(20 | (31 << 11));
    int wg = blockIdx.x;
    __asm__ volatile("" : "+s"(wg));  // (its conversion is not kept over the items)
    dbg[2 * m * m + m + 8] = (double)wg;
  }

  constexpr int ld = PolySmem<M>::LDA;
  gather_C_fp64_mfma(sm, I, obs_off, s, dbg);
  {
    // the domain's A, kept for the refinement of wbar (the stages overwrite
    // it): the lower triangle of the m x m matrix, packed by rows (row i at
    // i (i + 1) / 2), rows spread over the wavefronts and coalesced over lanes
    double* Ag = I.Ascr + (size_t)l * tri_size(m);
    const int w = phase_tid() / 64, lane = phase_tid() % 64;
    for (int i = w; i < m; i += PolyCfg<M>::NT / 64)
      for (int j = lane; j <= i; j += 64) gstore(Ag + tri_size(i) + j, sm.Bm[i * ld + j]);
  }
  stamp(1);
  {
    double* park = I.park;  // M > 64: this workgroup's slot (concurrent workgroups never share a slot)
    static_assert(M <= 64 || (kParkDoubles >= M * 16 * (8 - PolyCfg<M>::keep(8)) && kParkDoubles >= M * 16 * (7 - PolyCfg<M>::keep(7))), "parking slots");
    if (M > 64) park += (size_t)(I.n_dom <= kParkSlots ? l : (int)blockIdx.x) * kParkDoubles;
    auto solve = [&](auto tiles) {
      constexpr int T = decltype(tiles)::value;
      f64x4 Z[T];
      const int products = isqrt_stages<M, T>(sm, m, I.a_diag, guess, park, Z, [&]() { stamp(2); });
      stamp(3);
      if (threadIdx.x == 0) {
        if (I.dbg_sweeps) I.dbg_sweeps[l] = products;
        gatomic_add(&I.dom_sweeps[l], (unsigned)products);
        if (sm.rc[9] == 0.0) gatomic_add(&I.st->unconverged, 1);
        gatomic_add(&I.st->sweeps, (unsigned long long)products);
        gatomic_add(&I.st->solves, 1ull);
      }
      finish_T<M, T>(sm, I, l, Z, dbg);
    };
    const int t = (m + 15) / 16;
    if constexpr (M == 64) {
      if (t <= 3) solve(std::integral_constant<int, 3>{});
      else solve(std::integral_constant<int, 4>{});
    } else if constexpr (M == 128) {
      if (t <= 5) solve(std::integral_constant<int, 5>{});
      else if (t == 6) solve(std::integral_constant<int, 6>{});
      else if (t == 7) solve(std::integral_constant<int, 7>{});
      else solve(std::integral_constant<int, 8>{});
    } else {
      solve(std::integral_constant<int, M / 16>{});
    }
  }
  stamp(4);
  update_fp64(sm, I, est_off, e, cur);
  stamp(5);
}

// Persistent like k_analysis, with a work counter of its own (a batch may hold
// instances of both kernels).
template <int M>
__global__ __launch_bounds__(PolyCfg<M>::NT, M <= 32 ? 4 : M <= 64 ? 3 : 2) void k_analysis_poly(const InstDesc* __restrict__ tab,
                                                  BatchHdr* __restrict__ hdr, int cls) {
  __shared__ PolySmem<M> sm;
  __shared__ int s_next;
  ClassBatch& cb = hdr->cls[cls];
  const int total = cb.dom_off[cb.n];
  int item = blockIdx.x;
  while (item < total) {
    if (tab[cb.inst[find_entry(cb.dom_off, cb.n, item)]].poly) analyse_poly<M>(sm, tab, cb, item);
    if (threadIdx.x == 0) s_next = (int)gridDim.x + (int)atomicAdd(&cb.next_poly, 1u);
    __syncthreads();
    item = __builtin_amdgcn_readfirstlane(s_next);
    __syncthreads();
  }
}

// ----------------------------------------------------------------------------
// Debug instances (LETKF_FLAG_DEBUG) of k_analysis_poly: the eigenvalues of a domain's
// A = (m-1)/rho I + C, from the C that the analysis left in the debug record,
// by Cholesky and a one-sided Jacobi in LDS, when the record is read
// (letkf_debug_domain).  No frame runs it.
// ----------------------------------------------------------------------------
template <int M>
__global__ __launch_bounds__(AnaCfg<M>::NT) void k_lambda(const InstDesc* __restrict__ inst, int l) {
  using C = AnaCfg<M>;
  __shared__ AnaSmem<M> sm;
  const InstDesc& I = *inst;
  const int m = I.m, tid = phase_tid();
  double* dbg = I.dbg + (size_t)l * (2 * m * m + m + kDbgTail);
  for (int idx = tid; idx < M * M; idx += C::NT) {
    const int c = idx / M, r = idx % M;
    const double v = c < m && r < m ? gload(dbg + c * m + r) : 0.0;
    sm.Bm[c * C::LDB + r] = v + (r == c ? I.a_diag : 0.0);
  }
  __syncthreads();
  cholesky<M>(sm);
  bool converged = false;
  jacobi<0, M>(sm, m, converged, false);
  for (int c = tid; c < m; c += C::NT) {
    double ss = 0.0;
    for (int r = 0; r < M; ++r) ss = fma(sm.Bm[c * C::LDB + r], sm.Bm[c * C::LDB + r], ss);
    gstore(dbg + m * m + c, ss);  // columns of L J are sigma_i u_i and lambda_i = sigma_i^2
  }
}

// ----------------------------------------------------------------------------
// a4-a8 for ensembles of 129..256 members (padded to a multiple of 16, leading
// dimension 256, FP64).  A domain's matrices (512 KB each) do not fit in LDS, so
// its analysis is a sequence of launches over scratch in the instance workspace
// (which stays in L2 between launches), one wavefront group per 16 x 16 tile:
//   k_big_gram    A = (m-1)/rho I + Y'^T diag(r) Y' by tiles, b = Y'^T diag(r) d
//   k_big_mul     the matrix products of the polynomial stages of A^(-1/2)
//                 (isqrt_stages says how they are chosen and ended), one launch
//                 per product
//   k_big_slow    the stages past the launched ones, for condition numbers that
//                 need more than kBigStages of them (an empty launch otherwise)
//   k_big_wbar    wbar = Z (Z b), refined once with A
//   k_big_update  Z_l = xbar 1^T + X' (sqrt(m-1) Z + wbar 1^T)
// Every stage has degree 4, so that the launch sequence is the same for every
// condition number; the launches of stages a domain does not need return at
// once.  On the 32 x 32 pupil (m = 197, one domain) the blocked Jacobi this
// replaced took 3.42 of the analysis's 3.98 ms, in 312 dependent launches.
// ----------------------------------------------------------------------------
constexpr int kBigM = 256;
constexpr int kBigLd = kBigM + 8;     // LDS column stride in k_big_round
constexpr int kBigMaxSweeps = 24;
constexpr int kBigStages = 8;

struct BigDom {
  const InstDesc* I;
  int l, est_off, e, obs_off, s;
  double* A;
  double* W;   // 5 matrices: M, M^2 (then P M), P, Z of even and of odd stages
  double* v;
  int32_t* f;  // f[3]: the stages done, 0 until the last one is chosen
  __device__ double* mat(int k) const { return W + (size_t)k * kBigM * kBigM; }
  // of A + shift 1 1^T, divided by 2^ex ahead of the stages
  __device__ double& shift() const { return v[2 * kBigM]; }
  __device__ double& ex() const { return v[2 * kBigM + 1]; }
  // partial sums of |(M - I)^2|_F^2 (first stage: of |A^2|_F^2), by tile
  __device__ double* part() const { return v + 3 * kBigM; }
  // of stage s: the table entry planned for it (0: none), and the bound's
  __device__ double* plan(int s) const { return v + 4 * kBigM + 2 * s; }
  __device__ const double* Z() const { return mat(3 + (f[3] - 1) % 2); }
};
static_assert(2 * (kIsqrtCap + 2) <= kBigM, "plans of every stage");

__device__ __forceinline__ BigDom big_dom(const InstDesc* __restrict__ tab, const ClassBatch& cb, int item) {
  BigDom d;
  const int eb = find_entry(cb.dom_off, cb.n, item);
  d.I = &tab[cb.inst[eb]];
  d.l = item - cb.dom_off[eb];
  d.est_off = d.I->dom[4 * d.l];
  d.e = d.I->dom[4 * d.l + 1];
  d.obs_off = d.I->dom[4 * d.l + 2];
  d.s = d.I->dom[4 * d.l + 3];
  d.A = d.I->bigA + (size_t)d.l * kBigM * kBigM;
  d.W = d.I->bigW + (size_t)d.l * 5 * kBigM * kBigM;
  d.v = d.I->bigv + (size_t)d.l * 5 * kBigM;
  d.f = d.I->bigf + 4 * d.l;
  return d;
}

__device__ __forceinline__ double* big_dbg(const BigDom& D) {
  const int m = D.I->m;
  return D.I->dbg ? D.I->dbg + (size_t)D.l * (2 * m * m + m + kDbgTail) : nullptr;
}

// The sum of v over a 256-thread workgroup, on every thread.
__device__ __forceinline__ double block_sum256(double v, double* red) {
  v = wave_sum(v);
  if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = v;
  __syncthreads();
  const double t = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return t;
}

// grid (upper tiles ti <= tj, items), 16 wavefronts: one 16 x 16 tile of C per
// workgroup, the observations in blocks of 16 dealt over the wavefronts (block
// b to wavefront b mod 16), four k-steps of v_mfma_f64_16x16x4f64 each, and
// their partial tiles summed in LDS.  91 workgroups at m = 197, against the ten
// 64 x 64 tiles of the former split, whose 51 chunks in sequence were a latency
// chain (306 us on the global 32 x 32 domain; 8 wavefronts: 28.3 us, 16: 18.2).  A diagonal tile also forms its
// 16 entries of b.
constexpr int kGramWaves = 16, kGramObs = 2048;
__global__ __launch_bounds__(64 * kGramWaves) void k_big_gram(const InstDesc* __restrict__ tab,
                                                              const BatchHdr* __restrict__ hdr, int cls) {
  __shared__ int rowT[kGramObs];
  __shared__ double rT[kGramObs], rdT[kGramObs];
  __shared__ double red[kGramWaves][16 * 17], bred[kGramWaves][16];
  const ClassBatch& cb = hdr->cls[cls];
  if ((int)blockIdx.y >= cb.dom_off[cb.n]) return;
  const BigDom D = big_dom(tab, cb, blockIdx.y);
  const InstDesc& I = *D.I;
  const int m = I.m, nt = (m + 15) / 16;
  int t = blockIdx.x, ti = 0;
  while (ti < nt && t >= nt - ti) { t -= nt - ti; ++ti; }
  if (ti >= nt) return;
  const int tj = ti + t, i0 = 16 * ti, j0 = 16 * tj;
  const bool diag = ti == tj;
  const int tid = threadIdx.x, w = tid / 64, lane = tid % 64, g = lane / 16, i = lane % 16, nobs = 2 * D.s;
  const double* Yp = (const double*)I.Yp;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  double bpart = 0.0;
  const bool ia = i0 + i < m, ja = j0 + i < m;
  for (int g0 = 0; g0 < nobs; g0 += kGramObs) {
    const int gn = min(kGramObs, nobs - g0), gr = (gn + 15) & ~15;
    if (g0) __syncthreads();
    for (int q = tid; q < gr; q += 64 * kGramWaves) {
      int row = 0;
      double r = 0.0, rd = 0.0;
      if (q < gn) {
        row = gload(I.obs_row + 2 * D.obs_off + g0 + q);
        r = gload(I.obs_r + 2 * D.obs_off + g0 + q);
        rd = r * gload(I.d + row);
      }
      rowT[q] = row;
      rT[q] = r;
      rdT[q] = rd;
    }
    __syncthreads();
    // observation 16 b + 4 g + h in k-step h; a block past the table has weight zero
#pragma unroll 4
    for (int b = w; b < gr / 16; b += kGramWaves) {
      double ya[4], yb[4];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const double* y = Yp + (size_t)rowT[16 * b + 4 * g + h] * m;
        ya[h] = ia ? gload(y + i0 + i) : 0.0;
        yb[h] = diag ? ya[h] : ja ? gload(y + j0 + i) : 0.0;
      }
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        if (diag) bpart = fma(rdT[16 * b + 4 * g + h], ya[h], bpart);
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ya[h], rT[16 * b + 4 * g + h] * yb[h], acc, 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) red[w][i * 17 + g + 4 * v] = acc[v];
  bpart += __shfl_xor(bpart, 16, 64);
  bpart += __shfl_xor(bpart, 32, 64);
  if (lane < 16) bred[w][i] = bpart;
  __syncthreads();
  double* dbg = big_dbg(D);
  if (tid < 256) {
    const int r = tid % 16, c = tid / 16;
    double x = 0.0;
#pragma unroll
    for (int k = 0; k < kGramWaves; ++k) x += red[k][c * 17 + r];
    const int gi = i0 + r, gj = j0 + c;
    if (!diag || r <= c) {  // one writer per symmetric pair
      double a;
      if (gi < m && gj < m) {
        a = x + (gi == gj ? I.a_diag : 0.0);
        if (dbg) {
          dbg[(size_t)gi * m + gj] = x;
          dbg[(size_t)gj * m + gi] = x;
        }
      } else {
        a = gi == gj ? I.a_diag : 0.0;  // (the stages put the mean eigenvalue there)
      }
      D.A[(size_t)gj * kBigM + gi] = a;
      D.A[(size_t)gi * kBigM + gj] = a;
    }
  }
  if (blockIdx.x == 0 && tid == 0) D.f[3] = 0;
  if (diag && tid < 16) {
    double x = 0.0;
#pragma unroll
    for (int k = 0; k < kGramWaves; ++k) x += bred[k][tid];
    D.v[i0 + tid] = i0 + tid < m ? x : 0.0;
  }
}

// Tile (tr, tc) of L X, column-major matrices of leading dimension 256, by a
// 256-thread workgroup: wavefront w takes the 16-row blocks w, w + 4, ... of the
// contraction, all its operand loads first (the loads' latency, not the 13 to 16
// products of a wavefront, is what a tile takes), and the four partial tiles
// are summed in LDS.  left(r, k) and right(k, c) load the operands (right two
// consecutive k).  Thread t returns element (t % 16, t / 16) of the tile.
template <typename FL, typename FR>
__device__ __forceinline__ double big_tile(FL&& left, FR&& right, int tr, int tc, int nt, double (&red)[4][16 * 17]) {
  const int tid = threadIdx.x, w = tid / 64, lane = tid % 64, g = lane / 16, i = lane % 16;
  double a[16];
  f64x2 x[8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int b = w + 4 * k;
    const bool in = b < nt;
    const int k0 = 16 * (in ? b : 0) + 4 * g;
#pragma unroll
    for (int h = 0; h < 4; ++h) a[4 * k + h] = left(16 * tr + i, k0 + h);
#pragma unroll
    for (int h = 0; h < 2; ++h) x[2 * k + h] = right(k0 + 2 * h, 16 * tc + i);
    if (!in)
#pragma unroll
      for (int h = 0; h < 2; ++h) x[2 * k + h] = f64x2{0.0, 0.0};
  }
  __builtin_amdgcn_sched_barrier(0);  // every load issued before the first product waits
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 16; ++k)
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k], x[k / 2][k % 2], acc, 0, 0, 0);
#pragma unroll
  for (int v = 0; v < 4; ++v) red[w][i * 17 + g + 4 * v] = acc[v];
  __syncthreads();
  const int o = tid / 16 * 17 + tid % 16;
  const double t = (red[0][o] + red[1][o]) + (red[2][o] + red[3][o]);
  __syncthreads();
  return t;
}
__device__ __forceinline__ double big_product_tile(const double* L, const double* X, int tr, int tc, int nt, double (&red)[4][16 * 17]) {
  return big_tile([&](int r, int k) { return gload(L + (size_t)k * kBigM + r); },
                  [&](int k, int c) { return gload((const f64x2*)(X + (size_t)c * kBigM + k)); }, tr, tc, nt, red);
}

// Tile (tr, tc) of M^2 of stage s (of the first: of A^2, A shifted and scaled,
// which it leaves in M).  Returns the square of the thread's element of M^2 - 2 M + I
// (first stage: of A^2).
__device__ __forceinline__ double big_square(const BigDom& D, int s, int tr, int tc, int nt, double (&red)[4][16 * 17], double* bs) {
  const int r = 16 * tr + threadIdx.x % 16, c = 16 * tc + threadIdx.x / 16, m = D.I->m;
  const size_t at = (size_t)c * kBigM + r;
  double* M = D.mat(0);
  double t;
  if (s == 0) {
    const double* A = D.A;
    const double tr_A = block_sum256((int)threadIdx.x < m ? gload(A + (size_t)threadIdx.x * (kBigM + 1)) : 0.0, bs);
    const double shift = tr_A / ((double)m * m);
    const int ex = (__builtin_amdgcn_frexp_exp(tr_A) + 1) & ~1;
    auto get = [&](int r, int c) {  // past m the diagonal is the mean eigenvalue
      return ldexp(r < m && c < m ? gload(A + (size_t)c * kBigM + r) + shift : r == c ? shift * m : 0.0, -ex);
    };
    t = big_tile(get, [&](int k, int c) { return f64x2{get(k, c), get(k + 1, c)}; }, tr, tc, nt, red);
    gstore(M + at, get(r, c));
    if (tr == 0 && tc == 0 && threadIdx.x == 0) {
      D.shift() = shift;
      D.ex() = (double)ex;
    }
  } else {
    t = big_product_tile(M, M, tr, tc, nt, red);
  }
  gstore(D.mat(1) + at, t);
  const double d = s == 0 ? t : fma(-2.0, gload(M + at), t) + (r == c ? 1.0 : 0.0);
  return d * d;
}

// What stage s does, from f2 = |(M - I)^2|_F^2 (first stage: |A^2|_F^2).  The plan of
// a stage is written by the stage before it, so that every workgroup of a launch
// reads the same.
struct BigStage {
  const IsqrtStage* E;  // null: the last stage
  double scale;         // first stage: isqrt_scale
  bool converged;
};
__device__ __forceinline__ BigStage big_stage(const BigDom& D, int s, double f2, bool writer) {
  BigStage g{nullptr, 1.0, true};
  int plan, bound;
  if (s == 0) {
    g.scale = isqrt_scale(f2);
    plan = isqrt_first(g.scale, ldexp(D.I->a_diag, -(int)D.ex()), D.I->guess[D.l], bound);
  } else {
    plan = (int)D.plan(s)[0];
    bound = (int)D.plan(s)[1];
    const int last = isqrt_last(f2);
    g.converged = last == 2 || last == 4;
    if (g.converged || s == kIsqrtCap || last == kIsqrtNever) {
      if (writer) D.f[3] = s + 1;
      return g;
    }
    if (plan == 0) plan = isqrt_more(f2, bound);
  }
  g.E = &kIsqrtStage4[plan - 1];
  if (writer) {
    const int next = g.E->next;
    D.plan(s + 1)[0] = next;
    D.plan(s + 1)[1] = max(bound - (plan - next), next);
  }
  return g;
}

// Tile (tr, tc) of P = M^2 (q4 M^2 + q3 M) + q2 M^2 + q1 M + q0 I of stage s, in
// powers of M - I for the last stage.
__device__ __forceinline__ void big_poly(const BigDom& D, int s, const BigStage& G, int tr, int tc, int nt, double (&red)[4][16 * 17]) {
  const double* M = D.mat(0);
  const double* M2 = D.mat(1);
  const double* coef = G.E ? G.E->c : kIsqrtLast[1];
  double q[5], scale = G.scale;
  const double step = scale * scale;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    q[k] = coef[k] * scale;
    scale *= step;
  }
  const int r = 16 * tr + threadIdx.x % 16, c = 16 * tc + threadIdx.x / 16;
  const size_t at = (size_t)c * kBigM + r;
  double t, e1 = gload(M + at), e2 = gload(M2 + at);
  if (G.E) {
    t = big_tile([&](int r, int k) { return gload(M2 + (size_t)k * kBigM + r); },
                 [&](int k, int c) {
                   const size_t x = (size_t)c * kBigM + k;
                   return q[3] * gload((const f64x2*)(M + x)) + q[4] * gload((const f64x2*)(M2 + x));
                 }, tr, tc, nt, red);
  } else {
    auto one = [](int r, int c) { return r == c ? 1.0 : 0.0; };
    t = big_tile([&](int r, int k) {
                   const size_t x = (size_t)k * kBigM + r;
                   return fma(-2.0, gload(M + x), gload(M2 + x)) + one(r, k);
                 },
                 [&](int k, int c) {
                   const size_t x = (size_t)c * kBigM + k;
                   const f64x2 d = {one(k, c), one(k + 1, c)}, v = gload((const f64x2*)(M + x));
                   return q[3] * (v - d) + q[4] * (gload((const f64x2*)(M2 + x)) - 2.0 * v + d);
                 }, tr, tc, nt, red);
    e2 = fma(-2.0, e1, e2) + one(r, c);
    e1 -= one(r, c);
  }
  t += q[2] * e2 + q[1] * e1 + (r == c ? q[0] : 0.0);
  gstore(D.mat(2) + at, t);
  if (s == 0) gstore(D.mat(3) + at, t);  // Z = P
}

// Tile (tr, tc) of: kind 2: Z <- P Z    3: P M (into M^2's place)    4: M <- P (P M)
__device__ __forceinline__ void big_product(const BigDom& D, int kind, int s, int tr, int tc, int nt, double (&red)[4][16 * 17]) {
  const double* X = kind == 2 ? D.mat(3 + (s + 1) % 2) : kind == 3 ? D.mat(0) : D.mat(1);
  double* out = kind == 2 ? D.mat(3 + s % 2) : kind == 3 ? D.mat(1) : D.mat(0);
  const double t = big_product_tile(D.mat(2), X, tr, tc, nt, red);
  gstore(out + (size_t)(16 * tc + threadIdx.x / 16) * kBigM + 16 * tr + threadIdx.x % 16, t);
}

// grid (16 nt, ...): tile (x / 16, x % 16); KIND 0: M^2 and its partial sums,
// 1: the stage chosen from them and P, 2: products 2 and 3, by blockIdx.z, 4: that
// product.
template <int KIND>
__global__ __launch_bounds__(256) void k_big_mul(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr,
                                                 int cls, int s) {
  __shared__ double red[4][16 * 17];
  __shared__ double bs[4];
  const ClassBatch& cb = hdr->cls[cls];
  if ((int)blockIdx.y >= cb.dom_off[cb.n]) return;
  const BigDom D = big_dom(tab, cb, blockIdx.y);
  const int nt = (D.I->m + 15) / 16, tr = blockIdx.x / 16, tc = blockIdx.x % 16, tid = threadIdx.x;
  if (tr >= nt || tc >= nt) return;
  // done before this stage; at KIND 1 its first workgroup may just be writing
  // f[3] = s + 1, which reads the same here as 0
  const int done = D.f[3];
  if (done != 0 && done <= s) return;
  if (KIND == 0) {
    const double sum = block_sum256(big_square(D, s, tr, tc, nt, red, bs), bs);
    if (tid == 0) D.part()[blockIdx.x] = sum;
  } else if (KIND == 1) {
    // every workgroup sums the same partials in the same order
    const double f2 = block_sum256(tid / 16 < nt && tid % 16 < nt ? D.part()[tid] : 0.0, bs);
    const bool writer = blockIdx.x == 0 && tid == 0;
    const BigStage G = big_stage(D, s, f2, writer);
    if (writer && !G.converged && !G.E) gatomic_add(&D.I->st->unconverged, 1);
    big_poly(D, s, G, tr, tc, nt, red);
  } else {
    const int kind = KIND == 2 ? (s == 0 ? 3 : 2 + (int)blockIdx.z) : KIND;
    if (kind >= 3 && done == s + 1) return;
    big_product(D, kind, s, tr, tc, nt, red);
  }
}

// grid (items): the stages past kBigStages, one workgroup per domain (condition
// numbers above 1e9 or so off the vector of ones).
__global__ __launch_bounds__(256) void k_big_slow(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr,
                                                  int cls) {
  __shared__ double red[4][16 * 17];
  __shared__ double bs[4];
  const ClassBatch& cb = hdr->cls[cls];
  if ((int)blockIdx.x >= cb.dom_off[cb.n]) return;
  const BigDom D = big_dom(tab, cb, blockIdx.x);
  if (D.f[3] != 0) return;
  const int nt = (D.I->m + 15) / 16;
  for (int s = kBigStages; s <= kIsqrtCap; ++s) {
    double f2 = 0.0;
    for (int t = 0; t < nt * nt; ++t) f2 += big_square(D, s, t / nt, t % nt, nt, red, bs);
    f2 = block_sum256(f2, bs);
    const bool writer = threadIdx.x == 0;
    const BigStage G = big_stage(D, s, f2, writer);
    if (writer && !G.converged && !G.E) gatomic_add(&D.I->st->unconverged, 1);
    for (int t = 0; t < nt * nt; ++t) big_poly(D, s, G, t / nt, t % nt, nt, red);
    for (int kind = 2; kind <= (G.E ? 4 : 2); ++kind) {
      __syncthreads();
      for (int t = 0; t < nt * nt; ++t) big_product(D, kind, s, t / nt, t % nt, nt, red);
    }
    if (!G.E) break;
    __syncthreads();
  }
}

// grid (items), 1024 threads: wbar = Z (Z b) and one refinement step with A; the
// columns of Z (and of A) dealt over eight thread groups, a thread two rows of
// each.  One workgroup's reads of the matrix, five times, are what it takes:
// 16 bytes a lane, sixteen columns in flight (eight bytes and eight columns over
// four groups: 33.6 -> 24.1 us at m = 197).  Rows past m read the padded matrix; those past the padding
// read entries that no sum uses.
__global__ __launch_bounds__(1024) void k_big_wbar(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr,
                                                   int cls) {
  __shared__ double x[kBigM];
  __shared__ alignas(16) double part[8][kBigM];
  const ClassBatch& cb = hdr->cls[cls];
  if ((int)blockIdx.x >= cb.dom_off[cb.n]) return;
  const BigDom D = big_dom(tab, cb, blockIdx.x);
  const InstDesc& I = *D.I;
  const int m = I.m, mp = (m + 15) & ~15, tid = threadIdx.x, q = tid / 128, r2 = 2 * (tid % 128);
  const int ex = (int)D.ex();
  const double* Z = D.Z();  // times 2^(ex / 2)
  auto product = [&](const double* B) {  // x <- B x; returns row tid (the first 256 threads)
    f64x2 t0 = {0.0, 0.0}, t1 = {0.0, 0.0};
    if (r2 < mp) {
      const int c0 = q * (mp / 8), c1 = c0 + mp / 8;  // an even number of columns
      for (int c = c0; c < c1; c += 16) {
        f64x2 z[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) z[u] = gload((const f64x2*)(B + (size_t)(c + u < c1 ? c + u : c0) * kBigM + r2));
#pragma unroll
        for (int u = 0; u < 16; u += 2)
          if (c + u < c1) {
            t0 = x[c + u] * z[u] + t0;
            t1 = x[c + u + 1] * z[u + 1] + t1;
          }
      }
    }
    *(f64x2*)&part[q][r2] = t0 + t1;
    __syncthreads();
    double t = 0.0;
    if (tid < kBigM) {
      t = ((part[0][tid] + part[1][tid]) + (part[2][tid] + part[3][tid])) +
          ((part[4][tid] + part[5][tid]) + (part[6][tid] + part[7][tid]));
      x[tid] = t;
    }
    __syncthreads();
    return t;
  };
  if (tid < kBigM) x[tid] = tid < mp ? D.v[tid] : 0.0;
  __syncthreads();
  product(Z);
  const double w0 = ldexp(product(Z), -ex);
  if (tid < kBigM) x[tid] = w0;
  __syncthreads();
  const double aw = product(D.A);
  if (tid < kBigM) x[tid] = tid < m ? D.v[tid] - aw : 0.0;
  __syncthreads();
  product(Z);
  const double w1 = ldexp(product(Z), -ex);
  // wbar and what W lacks along the ones, which enter T in the same way
  const double wbar = w0 + w1 + ones_term(m, I.sqrt_m1, I.a_diag, D.shift());
  if (tid < kBigM) D.v[kBigM + tid] = tid < m ? wbar : 0.0;
  if (double* dbg = big_dbg(D)) {
    if (tid < kBigM) x[tid] = tid < m ? wbar : 0.0;
    __syncthreads();
    const double sc = ldexp(I.sqrt_m1, -ex / 2);
    const int r = tid % kBigM;
    for (int k = tid / kBigM; k < m; k += 4)
      if (r < m) dbg[(size_t)m * m + m + (size_t)k * m + r] = fma(sc, Z[(size_t)r * kBigM + k], x[k]);
  }
  if (tid == 0) {
    const int products = 5 * D.f[3] - 3;  // 4 in the first stage, 3 in the last
    if (I.dbg_sweeps) I.dbg_sweeps[D.l] = products;
    gatomic_add(&I.st->sweeps, (unsigned long long)products);
    gatomic_add(&I.st->solves, 1ull);
  }
}

// grid (16-row tiles of the domain's state rows, groups of four column tiles,
// items): Z_l = xbar + sqrt(m-1) X' Z + X' wbar.  The 16 rows X' are staged
// once in LDS, each wavefront forms one 16 x 16 output tile on FP64 MFMA with
// the columns of Z straight from L2 (32 contiguous bytes a lane).  440 workgroups
// on the global 32 x 32 domain; the VALU form over 64 x 64 tiles took 66 us.
__global__ __launch_bounds__(256) void k_big_update(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr,
                                                    int cls) {
  constexpr int LDX = kBigM + 1;
  __shared__ double Xs[16 * LDX], xb[16], xw[16];
  const ClassBatch& cb = hdr->cls[cls];
  if ((int)blockIdx.z >= cb.dom_off[cb.n]) return;
  const BigDom D = big_dom(tab, cb, blockIdx.z);
  const InstDesc& I = *D.I;
  const int m = I.m, nt = (m + 15) / 16, rows = 2 * D.e, tid = threadIdx.x, w = tid / 64, lane = tid % 64;
  const int q0 = 16 * blockIdx.x, tc = 4 * blockIdx.y + w;
  if (q0 >= rows || 4 * (int)blockIdx.y >= nt) return;
  const int cur = I.st->cur;
  const double* Z = D.Z();
  const double* wbar = D.v + kBigM;
  const double* ens = (const double*)I.ens;
  const size_t slot = (size_t)I.n_act * m;
  {
    // 16 threads a row: its values into registers, their mean, then X' to LDS
    const int rr = tid / 16, part = tid % 16, q = q0 + rr;
    double x[16], sum = 0.0, dot = 0.0;
    const bool on = q < rows;
    const double* row = ens + (size_t)((q < D.e ? cur : cur ^ 1)) * slot +
                        (size_t)(on ? I.est_act[D.est_off + (q < D.e ? q : q - D.e)] : 0) * m;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int j = part + 16 * k;
      x[k] = on && j < m ? gload(row + j) : 0.0;
      sum += x[k];
    }
    const double mean = group_sum<16>(sum) / (double)m;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int j = part + 16 * k;
      const double xp = j < m ? x[k] - mean : 0.0;
      Xs[rr * LDX + j] = xp;
      dot = fma(xp, j < m ? gload(wbar + j) : 0.0, dot);
    }
    dot = group_sum<16>(dot);
    if (part == 0) {
      xb[rr] = mean;
      xw[rr] = dot;
    }
  }
  __syncthreads();
  if (tc >= nt) return;
  const int g = lane / 16, i = lane % 16, col = 16 * tc + i;
  const double* Zc = Z + (size_t)col * kBigM + 4 * g;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int b = 0; b < nt; ++b) {
    const f64x2 z0 = gload((const f64x2*)(Zc + 16 * b)), z1 = gload((const f64x2*)(Zc + 16 * b) + 1);
    const double* xr = Xs + i * LDX + 16 * b + 4 * g;
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[0], z0.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[1], z0.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[2], z1.x, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[3], z1.y, acc, 0, 0, 0);
  }
  const double sc = ldexp(I.sqrt_m1, -(int)D.ex() / 2);
  double* out = (double*)I.Z + (size_t)2 * D.est_off * m;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int rr = g + 4 * v;
    if (q0 + rr < rows && col < m) gstore(out + (size_t)(q0 + rr) * m + col, xb[rr] + (xw[rr] + sc * acc[v]));
  }
}

// ---- debug instances, m > 128: the eigenvalues of one domain's A -------------
// As for m <= 128, when that domain's record is read: Cholesky, then the one-sided
// Jacobi by blocks (L J = U Sigma).  The columns form NB blocks of 16 (NB even;
// columns past m are unit vectors that never rotate).  A sweep is NB - 1 rounds
// of a round-robin tournament between the blocks (circle method, block 0
// fixed); in a round every pair of blocks is one workgroup that holds its 32
// columns in LDS and rotates the 256 pairs between them in 16 steps of 16
// disjoint pairs (the first round also the pairs inside each block), so every
// pair of columns is visited once per sweep.  Launch boundaries order the
// rounds; a converged domain's later launches return at once.
// A = L L^T into B (column-major, leading dimension kBigM; the upper triangle
// zero, padded members the identity), right-looking by panels of 16 columns
// as the m <= 128 kernel: wavefront 0 factors the panel in registers (rows
// c0 + lane + 64 s), which also stages it in LDS, and all eight wavefronts
// subtract its rank-16 product from the trailing lower triangle in 16 x 16
// tiles on FP64 MFMA (the tiles in B, whose loads are the latency that more
// wavefronts hide; the panel's columns from LDS).
constexpr int kBigCholWaves = 8;
__global__ __launch_bounds__(64 * kBigCholWaves) void k_big_chol(const InstDesc* __restrict__ tab,
                                                                 const BatchHdr* __restrict__ hdr, int cls, int item) {
  __shared__ double pnl[16][kBigM];
  const ClassBatch& cb = hdr->cls[cls];
  const BigDom D = big_dom(tab, cb, item);
  const int m = D.I->m, mp = (m + 15) & ~15, tid = threadIdx.x, w = tid / 64, lane = tid % 64;
  for (int idx = tid; idx < kBigM * kBigM; idx += 64 * kBigCholWaves) {
    const int c = idx / kBigM, r = idx % kBigM;
    double v;
    if (c < m) v = (r >= c && r < m) ? D.A[(size_t)c * kBigM + r] : 0.0;  // A symmetric
    else v = r == c ? 1.0 : 0.0;
    D.W[idx] = v;
  }
  if (tid < 3) D.f[tid] = 0;
  __syncthreads();
  for (int c0 = 0; c0 < mp; c0 += 16) {
    if (w == 0) {
      double a[4][16];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = c0 + lane + 64 * s;
        const bool on = r < mp;
#pragma unroll
        for (int jj = 0; jj < 16; ++jj) a[s][jj] = on ? D.W[(size_t)(c0 + jj) * kBigM + r] : 0.0;
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const double d = readlane_f64(a[0][j], j);  // a_jj after the earlier columns
        const double rs = rsqrt(d);
        double lj[4];
        lj[0] = lane > j ? a[0][j] * rs : (lane == j ? d * rs : 0.0);
#pragma unroll
        for (int s = 1; s < 4; ++s) lj[s] = a[s][j] * rs;
#pragma unroll
        for (int s = 0; s < 4; ++s) a[s][j] = lj[s];
#pragma unroll
        for (int jj = j + 1; jj < 16; ++jj) {
          const double l = readlane_f64(lj[0], jj);
#pragma unroll
          for (int s = 0; s < 4; ++s) a[s][jj] = fma(-lj[s], l, a[s][jj]);
        }
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = c0 + lane + 64 * s;
        if (r < mp)
#pragma unroll
          for (int jj = 0; jj < 16; ++jj) {
            D.W[(size_t)(c0 + jj) * kBigM + r] = a[s][jj];
            pnl[jj][r] = a[s][jj];
          }
      }
    }
    __syncthreads();
    const int nt = (mp - c0) / 16 - 1;
    int t = 0;
    for (int R = 0; R < nt; ++R)
      for (int Cc = 0; Cc <= R; ++Cc, ++t) {
        if (t % kBigCholWaves != w) continue;
        const int rb = c0 + 16 * (R + 1), cb = c0 + 16 * (Cc + 1);
        f64x4 acc;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = D.W[(size_t)(cb + lane % 16) * kBigM + rb + lane / 16 + 4 * v];
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const int k = 4 * ks + lane / 16;
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(pnl[k][rb + lane % 16], -pnl[k][cb + lane % 16], acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) D.W[(size_t)(cb + lane % 16) * kBigM + rb + lane / 16 + 4 * v] = acc[v];
      }
    __syncthreads();
  }
}

// grid (nb / 2, items): the workgroup of block pair blockIdx.x in round `round`.
__global__ __launch_bounds__(256) void k_big_round(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr,
                                                   int cls, int item, int nb, int round) {
  __shared__ double col[32 * kBigLd];
  __shared__ double nrm[32];
  const ClassBatch& cb = hdr->cls[cls];
  const BigDom D = big_dom(tab, cb, item);
  if (D.f[0]) return;  // converged: uniform over the workgroup
  const int m = D.I->m, tid = threadIdx.x, w = blockIdx.x, n1 = nb - 1;
  const int a = w == 0 ? 0 : 1 + (round + w) % n1;
  const int b = w == 0 ? 1 + round % n1 : 1 + (round + n1 - w) % n1;
  // LDS column k: block a's column k (k < 16), block b's column k - 16
  for (int idx = tid; idx < 32 * kBigM; idx += 256) {
    const int k = idx / kBigM, r = idx % kBigM;
    const int c = 16 * (k < 16 ? a : b) + (k & 15);
    col[k * kBigLd + r] = D.W[(size_t)c * kBigM + r];
  }
  __syncthreads();
  {
    const int k = tid / 8, part = tid % 8;
    double ss = 0.0;
    for (int r = part; r < kBigM; r += 8) {
      const double v = col[k * kBigLd + r];
      ss = fma(v, v, ss);
    }
    ss = group_sum<8>(ss);
    if (part == 0) nrm[k] = ss;
  }
  __syncthreads();
  const double tol = 32.0 * (double)m * 1.1102230246251565e-16;  // as in the m <= 128 kernel
  const double tol2 = tol * tol;
  const int p = tid / 16, sub = tid % 16;  // pair slot, lane within the pair
  bool rotated = false;
  auto step = [&](int ci, int cj) {
    double xi[16], xj[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      xi[t] = col[ci * kBigLd + sub + 16 * t];
      xj[t] = col[cj * kBigLd + sub + 16 * t];
    }
    double g0 = 0.0, g1 = 0.0;
#pragma unroll
    for (int t = 0; t < 16; t += 2) {
      g0 = fma(xi[t], xj[t], g0);
      g1 = fma(xi[t + 1], xj[t + 1], g1);
    }
    const double gsum = group_sum<16>(g0 + g1);
    const double al = nrm[ci], be = nrm[cj];  // the pairs of a step are disjoint
    if (gsum * gsum > tol2 * (al * be)) {
      const double dd = be - al, g2 = 2.0 * gsum;
      const double q2 = fma(dd, dd, g2 * g2);
      const double den = fma(q2, __builtin_amdgcn_rsq(q2), fabs(dd));
      const double t = copysign(1.0, dd) * g2 * __builtin_amdgcn_rcp(den);
      const double c = rsqrt_1_2(fma(t, t, 1.0));
      const double sn = c * t;
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const double x = xi[u];
        col[ci * kBigLd + sub + 16 * u] = c * x - sn * xj[u];
        col[cj * kBigLd + sub + 16 * u] = sn * x + c * xj[u];
      }
      if (sub == 0) {
        nrm[ci] = al - t * gsum;
        nrm[cj] = be + t * gsum;
      }
      rotated = true;
    }
    __syncthreads();
  };
  if (round == 0) {
    // pairs inside each block, (i, i ^ k): slots 0..7 block a, 8..15 block b
    const int base = p < 8 ? 0 : 16, q = p & 7;
    for (int k = 1; k < 16; ++k) {
      const int hk = 31 - __clz(k);
      const int i = ((q >> hk) << (hk + 1)) | (q & ((1 << hk) - 1));
      step(base + i, base + (i ^ k));
    }
  }
  // the 256 pairs between the blocks: slot p keeps block a's column p (and its
  // norm) in registers and meets block b's columns p, p + 1, ... (mod 16)
  {
    double xi[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) xi[t] = col[p * kBigLd + sub + 16 * t];
    double al = nrm[p];
    bool moved = false;
    for (int st = 0; st < 16; ++st) {
      const int cj = 16 + ((p + st) & 15);
      double xj[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) xj[t] = col[cj * kBigLd + sub + 16 * t];
      double g0 = 0.0, g1 = 0.0;
#pragma unroll
      for (int t = 0; t < 16; t += 2) {
        g0 = fma(xi[t], xj[t], g0);
        g1 = fma(xi[t + 1], xj[t + 1], g1);
      }
      const double gsum = group_sum<16>(g0 + g1);
      const double be = nrm[cj];
      if (gsum * gsum > tol2 * (al * be)) {
        const double dd = be - al, g2 = 2.0 * gsum;
        const double q2 = fma(dd, dd, g2 * g2);
        const double den = fma(q2, __builtin_amdgcn_rsq(q2), fabs(dd));
        const double t = copysign(1.0, dd) * g2 * __builtin_amdgcn_rcp(den);
        const double c = rsqrt_1_2(fma(t, t, 1.0));
        const double sn = c * t;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const double x = xi[u];
          xi[u] = c * x - sn * xj[u];
          col[cj * kBigLd + sub + 16 * u] = sn * x + c * xj[u];
        }
        al -= t * gsum;
        if (sub == 0) nrm[cj] = be + t * gsum;
        moved = true;
      }
      __syncthreads();
    }
    if (moved) {
      rotated = true;
#pragma unroll
      for (int t = 0; t < 16; ++t) col[p * kBigLd + sub + 16 * t] = xi[t];
    }
  }
  if (__syncthreads_or(rotated)) {
    for (int idx = tid; idx < 32 * kBigM; idx += 256) {
      const int k = idx / kBigM, r = idx % kBigM;
      const int c = 16 * (k < 16 ? a : b) + (k & 15);
      D.W[(size_t)c * kBigM + r] = col[k * kBigLd + r];
    }
    if (tid == 0) atomicAdd(&D.f[1], 1);
  }
}

__global__ void k_big_sweep(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr, int cls, int item) {
  const ClassBatch& cb = hdr->cls[cls];
  const BigDom D = big_dom(tab, cb, item);
  if (D.f[0]) return;
  D.f[2] += 1;
  if (D.f[1] == 0) {
    D.f[0] = 1;
  } else if (D.f[2] >= kBigMaxSweeps) {
    D.f[0] = 2;
  }
  D.f[1] = 0;
}

// Thread c: lambda_c, the squared norm of column c of L J.
__global__ __launch_bounds__(256) void k_big_lambda(const InstDesc* __restrict__ tab, const BatchHdr* __restrict__ hdr,
                                                    int cls, int item) {
  const ClassBatch& cb = hdr->cls[cls];
  const BigDom D = big_dom(tab, cb, item);
  const int m = D.I->m, c = threadIdx.x;
  double* dbg = big_dbg(D);
  if (!dbg || c >= m) return;
  double ss = 0.0;
  for (int r = 0; r < m; ++r) ss = fma(D.W[(size_t)c * kBigM + r], D.W[(size_t)c * kBigM + r], ss);
  dbg[(size_t)m * m + c] = ss;
}

// ----------------------------------------------------------------------------
// The allocation-free frame (letkf_step_noalloc): callers that cannot
// allocate device memory run a frame with its per-frame scratch in this
// file-scope array instead of the instance workspace.  Each GPU holds its own
// copy (kScratchBytes) until the process ends, shared by every such call on
// that GPU.  Host code reaches it only through the address hipGetSymbolAddress
// returns for the current device (scratch_address), never through its name.
// ----------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

hipError_t scratch_address(int device, unsigned char** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static unsigned char* addr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!addr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // the current device's copy
    if (e != hipSuccess) return e;
    addr[device] = (unsigned char*)p;
  }
  *out = addr[device];
  return hipSuccess;
}

// One workgroup: word copies of the instance descriptor and of the class's
// batch entry, then the pointers moved into the array.  Everything the frame
// kernels read of the header is written here (the work counter is zeroed by
// the slope kernel); the other classes' entries are never read.
__global__ __launch_bounds__(256) void k_noalloc_setup(const InstDesc* __restrict__ src,
                                                       const BatchHdr* __restrict__ src_hdr, unsigned char* sp,
                                                       NoallocLayout lay, const double* y, double* pred, int cls) {
  InstDesc* d = (InstDesc*)(sp + lay.desc);
  BatchHdr* h = (BatchHdr*)(sp + lay.hdr);
  static_assert(sizeof(InstDesc) % 4 == 0 && sizeof(ClassBatch) % 4 == 0, "word copies");
  for (int i = threadIdx.x; i < (int)(sizeof(InstDesc) / 4); i += blockDim.x)
    ((uint32_t*)d)[i] = ((const uint32_t*)src)[i];
  for (int i = threadIdx.x; i < (int)(sizeof(ClassBatch) / 4); i += blockDim.x)
    ((uint32_t*)&h->cls[cls])[i] = ((const uint32_t*)&src_hdr->cls[cls])[i];
  __syncthreads();
  if (threadIdx.x == 0) {
    d->Yp = sp + lay.Yp;
    d->d = (double*)(sp + lay.d);
    d->Z = sp + lay.Z;
    d->Ascr = lay.Ascr ? (double*)(sp + lay.Ascr) : nullptr;
    h->yptr[0] = y;
    h->amean = (double*)(sp + lay.amean);
    h->pmean = pred;
    h->out_off[0] = 0;
    h->check_y = 0;
    h->bad[0] = 0;
  }
}

void launch_noalloc_setup(const InstDesc* src, const BatchHdr* src_hdr, unsigned char* sp, const NoallocLayout& lay,
                          const double* y, double* pred, int cls, hipStream_t s) {
  hipLaunchKernelGGL(k_noalloc_setup, dim3(1), dim3(256), 0, s, src, src_hdr, sp, lay, y, pred, cls);
}

// ----------------------------------------------------------------------------
// launchers
// ----------------------------------------------------------------------------
// Row and item kernels loop grid-stride, so their grids are capped: a launch
// never needs more than this many workgroups to cover its work.
constexpr int kRowGridCap = 4096;
constexpr int kItemGridCap = 2048;

template <typename T, int MP>
static void launch_rows_t(int mode, int rows, const InstDesc* tab, BatchHdr* hdr, int cls,
                          hipStream_t s, const HostMeans& out) {
  const int grid = min((rows + 256 / MP - 1) / (256 / MP), kRowGridCap);
  if (grid <= 0) return;
  if (mode == 0) hipLaunchKernelGGL((k_rows<T, MP, 0>), dim3(grid), dim3(256), 0, s, tab, hdr, cls);
  if (mode == 1) hipLaunchKernelGGL((k_rows<T, MP, 1>), dim3(grid), dim3(256), 0, s, tab, hdr, cls);
  if (mode == 2) hipLaunchKernelGGL((k_rows<T, MP, 2>), dim3(grid), dim3(256), 0, s, tab, hdr, cls);
  if (out.host) hipLaunchKernelGGL(k_finish, dim3(1), dim3(1024), 0, s, tab, hdr, cls, mode != 0, out.mean, out.host, rows);
  else if (mode != 0) hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, tab, hdr, cls);
}

template <typename T, int MP>
static void launch_slopes_t(int rows, const InstDesc* tab, BatchHdr* hdr, int cls, hipStream_t s, const double* y) {
  const int grid = min((rows + 256 / MP - 1) / (256 / MP), kRowGridCap);
  if (grid > 0) hipLaunchKernelGGL((k_slopes<T, MP>), dim3(grid), dim3(256), 0, s, tab, hdr, cls, y);
}

#define LETKF_DISPATCH(FN, cls, ...)                                          \
  do {                                                                        \
    const int prec_ = (cls) / 4, sz_ = (cls) % 4;                             \
    if ((cls) == kBigClass) {                                                 \
      FN<double, 256>(__VA_ARGS__);                                           \
    } else if (prec_ == 0) {                                                  \
      if (sz_ == 0) FN<double, 16>(__VA_ARGS__);                              \
      else if (sz_ == 1) FN<double, 32>(__VA_ARGS__);                         \
      else if (sz_ == 2) FN<double, 64>(__VA_ARGS__);                         \
      else FN<double, 128>(__VA_ARGS__);                                      \
    } else {                                                                  \
      if (sz_ == 0) FN<float, 16>(__VA_ARGS__);                               \
      else if (sz_ == 1) FN<float, 32>(__VA_ARGS__);                          \
      else if (sz_ == 2) FN<float, 64>(__VA_ARGS__);                          \
      else FN<float, 128>(__VA_ARGS__);                                       \
    }                                                                         \
  } while (0)

// The analysis kernel of a class (P = precision path, M = padded size).
#define LETKF_ANA_KERNEL(cls, FN)                                   \
  do {                                                              \
    const int prec_ = (cls) / 4, sz_ = (cls) % 4;                   \
    if (prec_ == 0) {                                               \
      if (sz_ == 0) FN((k_analysis<0, 16>));                        \
      else if (sz_ == 1) FN((k_analysis<0, 32>));                   \
      else if (sz_ == 2) FN((k_analysis<0, 64>));                   \
      else FN((k_analysis<0, 128>));                                \
    } else if (prec_ == 1) {                                        \
      if (sz_ == 0) FN((k_analysis<1, 16>));                        \
      else if (sz_ == 1) FN((k_analysis<1, 32>));                   \
      else if (sz_ == 2) FN((k_analysis<1, 64>));                   \
      else FN((k_analysis<1, 128>));                                \
    } else if (prec_ == 2) {                                        \
      if (sz_ == 0) FN((k_analysis<2, 16>));                        \
      else if (sz_ == 1) FN((k_analysis<2, 32>));                   \
      else if (sz_ == 2) FN((k_analysis<2, 64>));                   \
      else FN((k_analysis<2, 128>));                                \
    } else {                                                        \
      if (sz_ == 0) FN((k_analysis<3, 16>));                        \
      else if (sz_ == 1) FN((k_analysis<3, 32>));                   \
      else if (sz_ == 2) FN((k_analysis<3, 64>));                   \
      else FN((k_analysis<3, 128>));                                \
    }                                                               \
  } while (0)

void launch_slopes(int cls, int rows, const InstDesc* tab, BatchHdr* hdr, hipStream_t s, const double* y) {
  LETKF_DISPATCH(launch_slopes_t, cls, rows, tab, hdr, cls, s, y);
}
void launch_pistons(int cls, int items, const InstDesc* tab, BatchHdr* hdr, hipStream_t s) {
  const int grid = min(items, kItemGridCap);
  if (grid <= 0) return;
  if (cls / 4 == 0 || cls == kBigClass) hipLaunchKernelGGL(k_piston_rhs<double>, dim3(grid), dim3(256), 0, s, tab, hdr, cls);
  else hipLaunchKernelGGL(k_piston_rhs<float>, dim3(grid), dim3(256), 0, s, tab, hdr, cls);
  hipLaunchKernelGGL(k_piston_solve, dim3(grid), dim3(256), 0, s, tab, hdr, cls);
}

void launch_rows(int cls, int mode, int rows, const InstDesc* tab, BatchHdr* hdr, hipStream_t s, const HostMeans& out) {
  LETKF_DISPATCH(launch_rows_t, cls, mode, rows, tab, hdr, cls, s, out);
}

void launch_big_analysis(int items, int rows_max, int m_max, const InstDesc* tab, BatchHdr* hdr, hipStream_t s) {
  if (items <= 0) return;
  const int cls = kBigClass, nt = (m_max + 15) / 16;
  hipLaunchKernelGGL(k_big_gram, dim3(nt * (nt + 1) / 2, items), dim3(64 * kGramWaves), 0, s, tab, hdr, cls);
  for (int st = 0; st < kBigStages; ++st) {
    hipLaunchKernelGGL(k_big_mul<0>, dim3(16 * nt, items), dim3(256), 0, s, tab, hdr, cls, st);
    hipLaunchKernelGGL(k_big_mul<1>, dim3(16 * nt, items), dim3(256), 0, s, tab, hdr, cls, st);
    hipLaunchKernelGGL(k_big_mul<2>, dim3(16 * nt, items, st == 0 ? 1 : 2), dim3(256), 0, s, tab, hdr, cls, st);
    hipLaunchKernelGGL(k_big_mul<4>, dim3(16 * nt, items), dim3(256), 0, s, tab, hdr, cls, st);
  }
  hipLaunchKernelGGL(k_big_slow, dim3(items), dim3(256), 0, s, tab, hdr, cls);
  hipLaunchKernelGGL(k_big_wbar, dim3(items), dim3(1024), 0, s, tab, hdr, cls);
  hipLaunchKernelGGL(k_big_update, dim3((rows_max + 15) / 16, (nt + 3) / 4, items), dim3(256), 0, s, tab, hdr, cls);
}

void launch_big_lambda(int domain, int m_max, const InstDesc* tab, BatchHdr* hdr, hipStream_t s) {
  const int cls = kBigClass, nb = 2 * ((m_max + 31) / 32);
  hipLaunchKernelGGL(k_big_chol, dim3(1), dim3(64 * kBigCholWaves), 0, s, tab, hdr, cls, domain);
  for (int sw = 0; sw < kBigMaxSweeps; ++sw) {
    for (int r = 0; r < nb - 1; ++r)
      hipLaunchKernelGGL(k_big_round, dim3(nb / 2), dim3(256), 0, s, tab, hdr, cls, domain, nb, r);
    hipLaunchKernelGGL(k_big_sweep, dim3(1), dim3(1), 0, s, tab, hdr, cls, domain);
  }
  hipLaunchKernelGGL(k_big_lambda, dim3(1), dim3(256), 0, s, tab, hdr, cls, domain);
}

#define LETKF_POLY_KERNEL(cls, FN)             \
  do {                                         \
    const int sz_ = (cls) % 4;                 \
    if (sz_ == 0) FN(k_analysis_poly<16>);     \
    else if (sz_ == 1) FN(k_analysis_poly<32>); \
    else if (sz_ == 2) FN(k_analysis_poly<64>); \
    else FN(k_analysis_poly<128>);             \
  } while (0)

void launch_analysis(int cls, int grid, int kinds, const InstDesc* tab, BatchHdr* hdr, hipStream_t s, int fair) {
  if (grid <= 0 || cls == kBigClass) return;  // the m > 128 class runs launch_big_analysis
  if (kinds & kKindPoly) {
    const bool m128 = cls % 4 == 3;
    const int pgrid = min(grid, analysis_max_grid(cls, kKindPoly));
#define LETKF_LAUNCH_POLY(K) hipLaunchKernelGGL(K, dim3(pgrid), dim3(m128 ? 512 : 256), 0, s, tab, hdr, cls)
    LETKF_POLY_KERNEL(cls, LETKF_LAUNCH_POLY);
#undef LETKF_LAUNCH_POLY
  }
  if (!(kinds & kKindJacobi)) return;
#define LETKF_LAUNCH_ANA(K) hipLaunchKernelGGL(K, dim3(grid), dim3(cls % 4 == 3 ? AnaCfg<128>::NT : 256), 0, s, tab, hdr, cls, fair)
  LETKF_ANA_KERNEL(cls, LETKF_LAUNCH_ANA);
#undef LETKF_LAUNCH_ANA
}

void launch_lambda(int cls, const InstDesc* inst, int domain, hipStream_t s) {
  const int sz = cls % 4;
  if (sz == 0) hipLaunchKernelGGL(k_lambda<16>, dim3(1), dim3(256), 0, s, inst, domain);
  else if (sz == 1) hipLaunchKernelGGL(k_lambda<32>, dim3(1), dim3(256), 0, s, inst, domain);
  else if (sz == 2) hipLaunchKernelGGL(k_lambda<64>, dim3(1), dim3(256), 0, s, inst, domain);
  else hipLaunchKernelGGL(k_lambda<128>, dim3(1), dim3(AnaCfg<128>::NT), 0, s, inst, domain);
}

int analysis_blocks_per_cu(int cls, int kinds) {
  if (cls == kBigClass) return 1;
  int n = 0, least = 0;
  hipError_t e = hipSuccess;
#define LETKF_OCC(K) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, K, cls % 4 == 3 ? 512 : 256, 0)
  static_assert(AnaCfg<128>::NT == 512 && PolyCfg<128>::NT == 512, "workgroups of M = 128");
  if (kinds & kKindPoly) {
    LETKF_POLY_KERNEL(cls, LETKF_OCC);
    least = (e == hipSuccess && n > 0) ? n : 1;
  }
  if (kinds & kKindJacobi) {
    LETKF_ANA_KERNEL(cls, LETKF_OCC);
    if (e != hipSuccess || n < 1) n = 1;
    least = least ? min(least, n) : n;
  }
#undef LETKF_OCC
  return least ? least : 1;
}

int analysis_max_grid(int cls, int kinds) { return cls % 4 == 3 && kinds == kKindPoly ? kParkSlots : 65535; }

}  // namespace letkf
