// Monte-Carlo (q)EHVI over a disjoint box decomposition.
//
// Paper: "Constrained qNEHVI" paragraph — the acquisition is the expected
// hypervolume improvement over samples of the joint posterior, estimated by
// Monte-Carlo integration, optionally restricted to feasible samples. With
// the region the front does not dominate split into disjoint boxes
// [lo, lo + w):
//   HVI(y)  = sum_c prod_k clamp(y_k - lo_ck, 0, w_ck)
//   qHVI(Y) = sum_{J != {}} (-1)^{|J|+1} sum_c prod_k min_{a in J} clamp(y_ak - lo_ck, 0, w_ck)
// (the clamp is monotone, so the minimum over batch members commutes with it).
//
// Feasibility (the constrained form): the constraints bound the objectives
// themselves, y_k >= t_k on the maximised objectives, and a sample (a batch
// member) counts only where all of them hold. An infeasible member's first
// objective is replaced by -inf: every clamp of it is then 0, so each box
// product, and each subset term that contains the member, vanishes — the
// same as multiplying those terms by the member's indicator.
//
// Mapping: one lane per candidate batch; the S base samples and the boxes
// are the same for every lane. Two objectives (fronts of a few points): both
// sit in LDS, every read is a broadcast, samples are processed in chunks held
// in registers and each box is read once per chunk, which leaves a branch-free
// VALU loop of 2m + (m-1) + 1 ops per (sample, box) for q = 1; for q > 1 a box
// that only one member reaches (on any lane and sample of the chunk) adds that
// member's own extent product. Three objectives (fronts of a hundred points,
// two boxes a point): sample by sample, the boxes that no lane of the wave
// reaches culled 64 at a time (k_ehvi3). No cross-lane reduction is needed: a
// lane owns the terms of its batch.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bo_internal.h"
#include "hvi_cull.h"

namespace bo {

size_t ehvi_lds_bytes(int S, int q, int m, int nbox) {
  return sizeof(float) * ((size_t)S * q * m + (size_t)nbox * 2 * m);
}

namespace {

constexpr int kThreads = 256;
constexpr size_t kLdsBytes = 160 * 1024;

__device__ inline float clamp_ext(float y, float lo, float w) {
  return __builtin_amdgcn_fmed3f(y - lo, 0.0f, w);
}

// Member feasibility: all objectives at or above their thresholds.
template <int MO>
__device__ __forceinline__ float mask_infeasible(const float (&y)[MO], const EhviArgs& a) {
  bool ok = true;
#pragma unroll
  for (int k = 0; k < MO; ++k) ok = ok && (y[k] >= a.lower[k]);
  return ok ? y[0] : -__builtin_inff();
}

// q = 1. The samples fall into kGroups groups of whole chunks of SC, each
// group's terms are summed on their own and the group sums added in group
// order, so the result does not depend on how the groups are spread: W waves
// (a power of two, blockDim.x = 64 max(W, 4)) share 64 candidates, each taking
// kGroups / W consecutive groups, and meet in LDS. Bound by vector issue when
// the chip is full (W = 1); a small batch has too few candidates for that
// (8192 are 128 waves on 1024 SIMDs), and its time is one lane's serial walk
// over its samples, which W divides. One wave per candidate set against the
// rule of q1_waves (m = 2): M = 4096, S = 128: 22.2 -> 5.1 us; M = 8192,
// S = 512: 78.4 -> 9.2 us; M = 65536, S = 256: 58.7 -> 26.9 us; M = 1048576,
// S = 512 (W = 1 either way): 326 and 319 us.
constexpr int kGroups = 16;
template <int SC, bool CONS>
__global__ __launch_bounds__(1024) void k_ehvi_q1(EhviArgs a, int W) {
  extern __shared__ float sm[];
  constexpr int MO = 2;
  float* zs = sm;                                   // [S][MO]
  float* bx = sm + a.S * MO;                        // [nbox][2*MO]
  float* part = bx + a.nbox * 2 * MO;               // W > 1: [64 max(W, 4) / (64 W)][kGroups][64]
  const int nt = blockDim.x;
  for (int i = threadIdx.x; i < a.S * MO; i += nt) zs[i] = a.Z[i];
  for (int i = threadIdx.x; i < a.nbox * 2 * MO; i += nt) bx[i] = a.boxes[i];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sub = wave / W, ws = wave % W;          // candidate set of this wave, its share
  const int64_t b = ((int64_t)blockIdx.x * (nt / 64 / W) + sub) * 64 + lane;
  const bool valid = b < a.nbat;
  float mu[MO], sd[MO];
  bool nan_in = false;      // a NaN posterior gives a NaN acquisition
#pragma unroll
  for (int k = 0; k < MO; ++k) {
    mu[k] = valid ? a.mu[b * a.mu_ps + k * a.mu_ks] : 0.f;
    sd[k] = valid ? a.sd[b * a.sd_ps + k * a.sd_ks] : 0.f;
    nan_in = nan_in || (mu[k] != mu[k]) || (sd[k] != sd[k]);
  }
  const int gs = (a.S + kGroups * SC - 1) / (kGroups * SC) * SC;   // samples per group
  float tot = 0.f;
  for (int g = ws * (kGroups / W); g < (ws + 1) * (kGroups / W); ++g) {
    float acc = 0.f;
    for (int s0 = g * gs; s0 < min(a.S, (g + 1) * gs); s0 += SC) {
      float y[SC][MO];
#pragma unroll
      for (int j = 0; j < SC; ++j)
#pragma unroll
        for (int k = 0; k < MO; ++k) {
          const int s = s0 + j;
          const int sl = (s < a.S) ? s : (a.S - 1);
          // samples past S get -inf: every extent clamps to 0
          y[j][k] = (s < a.S) ? fmaf(sd[k], zs[sl * MO + k], mu[k]) : -__builtin_inff();
        }
      if constexpr (CONS) {
#pragma unroll
        for (int j = 0; j < SC; ++j) y[j][0] = mask_infeasible<MO>(y[j], a);
      }
      for (int c = 0; c < a.nbox; ++c) {
        float lo[MO], w[MO];
#pragma unroll
        for (int k = 0; k < MO; ++k) {
          lo[k] = bx[c * 2 * MO + k];
          w[k] = bx[c * 2 * MO + MO + k];
        }
#pragma unroll
        for (int j = 0; j < SC; ++j) {
          float t = clamp_ext(y[j][0], lo[0], w[0]);
#pragma unroll
          for (int k = 1; k < MO; ++k) t *= clamp_ext(y[j][k], lo[k], w[k]);
          acc += t;
        }
      }
    }
    if (W == 1) tot += acc;
    else part[(sub * kGroups + g) * 64 + lane] = acc;
  }
  if (W > 1) {
    __syncthreads();
    if (ws != 0) return;
    for (int g = 0; g < kGroups; ++g) tot += part[(sub * kGroups + g) * 64 + lane];
  }
  if (valid) a.ehvi[b] = nan_in ? __builtin_nanf("") : tot / static_cast<float>(a.S);
}

// Waves per 64 candidates at q = 1: the fewest that give the chip's 1024
// SIMDs four waves each, at most one per sample group.
int q1_waves(int64_t nbat) {
  const int64_t sets = (nbat + 63) / 64;
  int W = 1;
  while (W < kGroups && sets * W < 4096) W *= 2;
  return W;
}

// q-batch version (two objectives): lane owns a batch of Q points; y_s[a][k] is sampled with
// the lower factor of objective k, then the 2^Q - 1 member subsets are
// expanded by inclusion-exclusion per box. Batches are few (131,072 at the
// q = 4 workload: two waves per SIMD at one lane each), so the four waves of
// a workgroup share its 64 batches and split the samples; their partial sums
// are added in LDS in wave order.
constexpr int kQWaves = kThreads / 64;
template <int Q, int SC, bool CONS>
__global__ __launch_bounds__(kThreads) void k_ehvi_q(EhviArgs a) {
  extern __shared__ float sm[];
  constexpr int MO = 2;
  constexpr int T = Q * (Q + 1) / 2;
  constexpr int NS = (1 << Q);
  float* zs = sm;                                   // [S][Q][MO]
  float* bx = sm + a.S * Q * MO;                    // [nbox][2*MO]
  for (int i = threadIdx.x; i < a.S * Q * MO; i += kThreads) zs[i] = a.Z[i];
  for (int i = threadIdx.x; i < a.nbox * 2 * MO; i += kThreads) bx[i] = a.boxes[i];
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t b = (int64_t)blockIdx.x * 64 + lane;
  const bool valid = b < a.nbat;
  // this wave's samples: a quarter of S, in whole chunks of SC
  const int sw = (a.S + kQWaves * SC - 1) / (kQWaves * SC) * SC;
  const int sbeg = wave * sw, send = min(a.S, sbeg + sw);
  float mu[Q][MO];
  float C[MO][T];
  bool nan_in = false;      // a NaN posterior gives a NaN acquisition
#pragma unroll
  for (int i = 0; i < Q; ++i)
#pragma unroll
    for (int k = 0; k < MO; ++k) {
      mu[i][k] = valid ? a.mu[(b * Q + i) * a.mu_ps + k * a.mu_ks] : 0.f;
      nan_in = nan_in || (mu[i][k] != mu[i][k]);
    }
#pragma unroll
  for (int k = 0; k < MO; ++k)
#pragma unroll
    for (int e = 0; e < T; ++e) {
      C[k][e] = valid ? a.chol[(k * a.nbat + b) * T + e] : 0.f;
      nan_in = nan_in || (C[k][e] != C[k][e]);
    }

  float acc_pos = 0.f, acc_neg = 0.f;
  for (int s0 = sbeg; s0 < send; s0 += SC) {
    float y[SC][Q][MO];
#pragma unroll
    for (int j = 0; j < SC; ++j) {
      const int s = s0 + j;
      const int sl = (s < send) ? s : (send - 1);
#pragma unroll
      for (int k = 0; k < MO; ++k)
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          float v = mu[i][k];
#pragma unroll
          for (int t = 0; t <= i; ++t) v = fmaf(C[k][i * (i + 1) / 2 + t], zs[(sl * Q + t) * MO + k], v);
          y[j][i][k] = (s < send) ? v : -__builtin_inff();
        }
      if constexpr (CONS) {
#pragma unroll
        for (int i = 0; i < Q; ++i) y[j][i][0] = mask_infeasible<MO>(y[j][i], a);
      }
    }
    // per sample, the batch's best value in each objective: a box whose
    // lower corner no member exceeds in some objective adds exactly zero
    float ymax[SC][MO];
#pragma unroll
    for (int j = 0; j < SC; ++j)
#pragma unroll
      for (int k = 0; k < MO; ++k) {
        float v = y[j][0][k];
#pragma unroll
        for (int i = 1; i < Q; ++i) v = fmaxf(v, y[j][i][k]);
        ymax[j][k] = v;
      }
    for (int c = 0; c < a.nbox; ++c) {
      float lo[MO], w[MO];
#pragma unroll
      for (int k = 0; k < MO; ++k) {
        lo[k] = bx[c * 2 * MO + k];
        w[k] = bx[c * 2 * MO + MO + k];
      }
      bool live = false;
#pragma unroll
      for (int j = 0; j < SC; ++j) {
        bool nz = true;
#pragma unroll
        for (int k = 0; k < MO; ++k) nz = nz && (ymax[j][k] > lo[k]);
        live = live || nz;
      }
      if (__ballot(live) == 0) continue;   // the whole wave would add zeros
      // the members that reach the box (above its lower corner in every
      // objective) on some lane and sample of the chunk; a member subset with
      // any other member adds exactly zero. Mostly one member reaches a box:
      // then only its own extent product is formed (the same sum, the other
      // terms being zeros)
      int rmask = 0;
#pragma unroll
      for (int i = 0; i < Q; ++i) {
        bool r = false;
#pragma unroll
        for (int j = 0; j < SC; ++j) {
          bool rj = true;
#pragma unroll
          for (int k = 0; k < MO; ++k) rj = rj && (y[j][i][k] > lo[k]);
          r = r || rj;
        }
        if (__ballot(r) != 0) rmask |= 1 << i;
      }
      if (rmask == 0) continue;
      if ((rmask & (rmask - 1)) == 0) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          if (rmask == (1 << i)) {
#pragma unroll
            for (int j = 0; j < SC; ++j) {
              float t = clamp_ext(y[j][i][0], lo[0], w[0]);
#pragma unroll
              for (int k = 1; k < MO; ++k) t *= clamp_ext(y[j][i][k], lo[k], w[k]);
              acc_pos += t;
            }
          }
        }
        continue;
      }
#pragma unroll
      for (int j = 0; j < SC; ++j) {
        float ext[NS][MO];
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
          for (int k = 0; k < MO; ++k) ext[1 << i][k] = clamp_ext(y[j][i][k], lo[k], w[k]);
#pragma unroll
        for (int mask = 1; mask < NS; ++mask) {
          const int low = mask & (-mask);
          if (mask != low) {
#pragma unroll
            for (int k = 0; k < MO; ++k) ext[mask][k] = fminf(ext[mask ^ low][k], ext[low][k]);
          }
          float t = ext[mask][0];
#pragma unroll
          for (int k = 1; k < MO; ++k) t *= ext[mask][k];
          if (__builtin_popcount(mask) & 1) acc_pos += t;
          else acc_neg += t;
        }
      }
    }
  }
  // the waves' partial sums, added in wave order (the samples' LDS is done)
  __syncthreads();
  float* part = sm;                                 // [kQWaves][64]
  part[wave * 64 + lane] = acc_pos - acc_neg;
  __syncthreads();
  if (wave == 0) {
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < kQWaves; ++w) tot += part[w * 64 + lane];
    if (valid) a.ehvi[b] = nan_in ? __builtin_nanf("") : tot / static_cast<float>(a.S);
  }
}

// Three objectives, any q, every size: a lane per batch, W waves (blockDim.x = 64 W) share
// 64 batches and the sample groups as in k_ehvi_q1 (kGroups groups of
// consecutive samples, group sums added in group order), and each sample's
// boxes are culled per wave (hvi_cull.h). Lanes past the batch sit at -inf.
// Bound by vector and scalar issue. Against testing box after box in chunks of
// 2 to 16 samples (the two-objective kernels' way): 131072 batches of 4, 512
// samples, 235 boxes 10.40 -> 1.79 ms; 33331 pairs, 300 samples, 137 boxes,
// constrained 1.14 -> 0.163 ms; 256 samples, 6 dimensions, lengthscales 0.3 and
// 1.5 (the latter: small variances, candidates far apart), 145 boxes: 65536
// single points 0.65 -> 0.38 and 0.65 -> 0.46 ms, 32768 pairs 1.33 -> 0.40 and
// 1.36 -> 0.52, 16384 batches of 4 2.93 -> 0.89 and 3.05 -> 1.06; 3 boxes 51 -> 29
// and 49 -> 27 us, 36 -> 21 and 39 -> 21, 68 -> 55 and 79 -> 60.
template <int Q, bool CONS>
__device__ __forceinline__ void ehvi3(const EhviArgs& a, bool lds_lo) {
  extern __shared__ float sm[];
  constexpr int T = Q * (Q + 1) / 2;
  const int nt = blockDim.x, W = nt / 64;
  const int nb64 = (a.nbox + 63) / 64 * 64;
  float* zs = sm;                                   // [S][Q][3]
  float* ls = sm + a.S * Q * 3;                     // lds_lo: [3][nb64] lower corners, +inf past nbox
  for (int i = threadIdx.x; i < a.S * Q * 3; i += nt) zs[i] = a.Z[i];
  if (lds_lo)
    for (int i = threadIdx.x; i < 3 * nb64; i += nt) {
      const int k = i / nb64, c = i - k * nb64;
      ls[i] = c < a.nbox ? a.boxes[6 * c + k] : __builtin_huge_valf();
    }
  __syncthreads();
  auto corner = [&](int c, float (&l)[3]) {
    if (lds_lo) {
#pragma unroll
      for (int k = 0; k < 3; ++k) l[k] = ls[k * nb64 + c];
    } else {
      load_corner(a.boxes, a.nbox, c, l);
    }
  };
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t b = (int64_t)blockIdx.x * 64 + lane;
  const bool valid = b < a.nbat;
  float mu[Q][3], C[3][T];               // q = 1: C[k][0] = sigma_k
  bool nan_in = false;                   // a NaN posterior gives a NaN acquisition
#pragma unroll
  for (int i = 0; i < Q; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      mu[i][k] = valid ? a.mu[(b * Q + i) * a.mu_ps + k * a.mu_ks] : -__builtin_huge_valf();
      nan_in = nan_in || (mu[i][k] != mu[i][k]);
    }
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int e = 0; e < T; ++e) {
      if (Q == 1) C[k][e] = valid ? a.sd[b * a.sd_ps + k * a.sd_ks] : 0.f;
      else C[k][e] = valid ? a.chol[(k * a.nbat + b) * T + e] : 0.f;
      nan_in = nan_in || (C[k][e] != C[k][e]);
    }
  const int gs = (a.S + kGroups - 1) / kGroups;      // samples per group
  float sum[kGroups / 4] = {};                       // this wave's groups (W >= 4)
  CullState cull;
#pragma unroll 1                                     // one copy of the boxes' code
  for (int gi = 0; gi < kGroups / W; ++gi) {
    const int g = wave * (kGroups / W) + gi;
    HviSums<Q> h;
    for (int s = g * gs; s < min(a.S, (g + 1) * gs); ++s) {
      float y[Q][3];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < Q; ++i) {
          float v = mu[i][k];
#pragma unroll
          for (int t = 0; t <= i; ++t)
            v = fmaf(C[k][i * (i + 1) / 2 + t], zs[(s * Q + t) * 3 + k], v);
          y[i][k] = v;
        }
      if constexpr (CONS) {
#pragma unroll
        for (int i = 0; i < Q; ++i) y[i][0] = mask_infeasible<3>(y[i], a);
      }
      box_terms3<Q>(y, a.boxes, a.nbox, corner, cull, h);
    }
    const float t = h.total();
#pragma unroll
    for (int j = 0; j < kGroups / 4; ++j) sum[j] = j == gi ? t : sum[j];
  }
  // the group sums, added in group order (the samples' LDS is done with)
  __syncthreads();
#pragma unroll
  for (int gi = 0; gi < kGroups / 4; ++gi)
    if (gi < kGroups / W) sm[(wave * (kGroups / W) + gi) * 64 + lane] = sum[gi];
  __syncthreads();
  if (wave != 0) return;
  float tot = 0.f;
  for (int g = 0; g < kGroups; ++g) tot += sm[g * 64 + lane];
  if (valid) a.ehvi[b] = nan_in ? __builtin_nanf("") : tot / static_cast<float>(a.S);
}

template <int Q, bool CONS>
__global__ __launch_bounds__(1024) BO_CULL_SGPRS void k_ehvi3(EhviArgs a, bool lds_lo) {
  ehvi3<Q, CONS>(a, lds_lo);
}
template <bool CONS>
__global__ __launch_bounds__(1024) void k_ehvi3_q4(EhviArgs a, bool lds_lo) {
  ehvi3<4, CONS>(a, lds_lo);
}

// Waves per 64 batches with three objectives: eight waves a SIMD for a full
// chip, at most one per sample group.
int waves3(int64_t nbat) {
  const int64_t sets = (nbat + 63) / 64;
  int W = 4;
  while (W < kGroups && sets * W < 8192) W *= 2;
  return W;
}

// Launch with the dynamic-LDS limit raised for that kernel (set on every
// launch, so that it holds on whichever device is current).
template <typename K, typename... A>
hipError_t launch_k(K kern, unsigned grid, unsigned threads, size_t lds, hipStream_t st, A... a) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, st, a...);
  return hipGetLastError();
}

template <bool CONS>
hipError_t launch_2(const EhviArgs& a, hipStream_t st) {
  const size_t lds = ehvi_lds_bytes(a.S, a.q, 2, a.nbox);
  if (a.q == 1) {
    // the group sums of W > 1 waves come after the boxes (at most 4096 samples
    // and 2049 boxes: 81 KiB in all)
    const int W = q1_waves(a.nbat);
    const int per = 64 * (W < 4 ? 4 / W : 1);       // candidates per workgroup
    const size_t part = W > 1 ? sizeof(float) * kGroups * per : 0;
    if (lds + part > kLdsBytes) return hipErrorInvalidValue;
    const unsigned grid = static_cast<unsigned>((a.nbat + per - 1) / per);
    return launch_k(&k_ehvi_q1<16, CONS>, grid, 64 * std::max(W, 4), lds + part, st, a, W);
  }
  // q > 1: a workgroup per 64 batches (LDS: at least the waves' partial sums,
  // which reuse the space at the end)
  const unsigned grid = static_cast<unsigned>((a.nbat + 63) / 64);
  const size_t ldsq = std::max<size_t>(lds, sizeof(float) * kThreads);
  switch (a.q) {
    case 2: return launch_k(&k_ehvi_q<2, 4, CONS>, grid, kThreads, ldsq, st, a);
    case 4: return launch_k(&k_ehvi_q<4, 2, CONS>, grid, kThreads, ldsq, st, a);
    default: return hipErrorInvalidValue;
  }
}

template <bool CONS>
hipError_t launch_3(const EhviArgs& a, hipStream_t st) {
  const unsigned grid = static_cast<unsigned>((a.nbat + 63) / 64);
  const unsigned threads = 64 * waves3(a.nbat);
  // corners in LDS unless the samples leave no room (the last few hundred
  // bytes of the limit that ehvi_lds_bytes sets), group sums over them at the end
  const size_t zs = sizeof(float) * a.S * a.q * 3, lo = sizeof(float) * 3 * ((a.nbox + 63) / 64 * 64);
  const bool lds_lo = zs + lo <= kLdsBytes;
  const size_t lds = std::max<size_t>(zs + (lds_lo ? lo : 0), sizeof(float) * kGroups * 64);
  switch (a.q) {
    case 1: return launch_k(&k_ehvi3<1, CONS>, grid, threads, lds, st, a, lds_lo);
    case 2: return launch_k(&k_ehvi3<2, CONS>, grid, threads, lds, st, a, lds_lo);
    case 4: return launch_k(&k_ehvi3_q4<CONS>, grid, threads, lds, st, a, lds_lo);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_ehvi(const EhviArgs& a, hipStream_t st) {
  if (a.nbat <= 0) return hipSuccess;
  if (a.m == 2) return a.constrained ? launch_2<true>(a, st) : launch_2<false>(a, st);
  if (a.m == 3) return a.constrained ? launch_3<true>(a, st) : launch_3<false>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace bo
