// Hypervolume terms of three objectives over many boxes, culled per wave.
//
// A lane holds one candidate batch and all lanes of a wave are at the same
// sample, so their draws differ only by the candidates' means and factors: of
// the 140-290 boxes of a three-objective front a sample reaches about 12% on
// a lane and 16% on any lane of the wave (2048 observations, 24 dimensions),
// and nearly always with one member of the batch. Testing box after box costs
// more than the terms do. Here the lanes test 64 boxes at a time instead: each
// member's largest value per objective over the wave is reduced with DPP, lane
// i compares box c0 + i's lower corner with it, and the ballots are one 64-bit
// mask of the boxes that the member may reach. The waves then visit only those
// boxes, in order, by which members reach them: one (its own extent product),
// two (two products less their intersection), more (all 2^Q - 1 subsets).
// Every term left out is exactly zero on every lane, and a lane adds the others
// box after box whatever the way taken: which boxes and ways these are depends
// on the batches that share the wave, a batch's sum does not. A box's corner and widths come
// through the scalar cache (its address is uniform) as scalar operands; the
// visits are bound by scalar issue (mask and address), so one box at a time or
// four measured 2-13% slower than two.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace bo {
namespace {

// Largest of v over the wave (NaN lanes do not count), in every lane's reach.
__device__ __forceinline__ float wave_max(float v) {
#define BO_DPP_MAX(ctrl)                                                                       \
  v = fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), \
                                                          ctrl, 0xF, 0xF, false)))
  BO_DPP_MAX(0x111);   // row_shr:1
  BO_DPP_MAX(0x112);   // row_shr:2
  BO_DPP_MAX(0x114);   // row_shr:4
  BO_DPP_MAX(0x118);   // row_shr:8
  BO_DPP_MAX(0x142);   // row_bcast:15
  BO_DPP_MAX(0x143);   // row_bcast:31
#undef BO_DPP_MAX
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

typedef const float __attribute__((address_space(4)))* const_floats;

// When a wave's lanes are far apart (candidates with spread-out means and small
// variances) most boxes are marked and walking all of them in order is cheaper:
// no masks, addresses that only count up, no test. A tested sample that cost
// more than the walk lets the next kWalkSamples walk without a test (the lanes
// stay as far apart as they are), and a front so small that the test alone
// costs more is always walked. A walk adds the zeros that a visit leaves out,
// nothing else changes. Issue costs in quarters of a box that one member
// reaches: two members, all members (q = 4), the test, a box of the walk.
template <int Q>
struct CullCost {
  static constexpr int kOwn = 4, kPair = 8, kAll = 28;
  static constexpr int kTest = Q == 1 ? 20 : Q == 2 ? 34 : 60;
  static constexpr int kWalk = Q == 1 ? 3 : Q == 2 ? 6 : 26;
};
constexpr int kWalkSamples = 15;

// Terms of the boxes boxes[0 .. nbox) ([c][6]: lower corner, then widths; the
// address is uniform) for the members' values y[a][k] of this lane, into pos
// and neg (odd and even subsets). lo(c, k): lower corner k of box c, a vector
// load by lane, +inf for c >= nbox. walk: samples to come that are walked
// without a test (0 at first).
template <int Q, typename Lo>
__device__ __forceinline__ void box_terms3(const float (&y)[Q][3], const float* boxes, int nbox,
                                           Lo lo, int& walk, float& pos, float& neg) {
  using Cost = CullCost<Q>;
  const const_floats bx = (const_floats)(uintptr_t)boxes;
  struct Box { float lo[3], w[3]; };
  auto box = [&](unsigned c) {
    const const_floats p = bx + 6u * c;
    return Box{{p[0], p[1], p[2]}, {p[3], p[4], p[5]}};
  };
  auto extents = [&](const float (&v)[3], const Box& b, float (&e)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) e[k] = __builtin_amdgcn_fmed3f(v[k] - b.lo[k], 0.0f, b.w[k]);
  };
  auto own = [&](const float (&v)[3], const Box& b) {
    float e[3];
    extents(v, b, e);
    pos = fmaf(e[0] * e[1], e[2], pos);
  };
  auto pair = [&](const float (&v)[3], const float (&u)[3], const Box& b) {
    float e[3], f[3];
    extents(v, b, e);
    extents(u, b, f);
    pos = fmaf(e[0] * e[1], e[2], pos);
    pos = fmaf(f[0] * f[1], f[2], pos);
    neg = fmaf(fminf(e[0], f[0]) * fminf(e[1], f[1]), fminf(e[2], f[2]), neg);
  };
  auto all = [&](const Box& b) {
    if constexpr (Q == 1) {
      own(y[0], b);
    } else if constexpr (Q == 2) {
      pair(y[0], y[1], b);
    } else {
      constexpr int NS = 1 << Q;
      float ext[NS][3];
#pragma unroll
      for (int a = 0; a < Q; ++a) extents(y[a], b, ext[1 << a]);
#pragma unroll
      for (int mask = 1; mask < NS; ++mask) {
        const int low = mask & (-mask);
        if (mask != low) {
#pragma unroll
          for (int k = 0; k < 3; ++k) ext[mask][k] = fminf(ext[mask ^ low][k], ext[low][k]);
        }
        const float t = ext[mask][0] * ext[mask][1];
        if (__builtin_popcount(mask) & 1) pos = fmaf(t, ext[mask][2], pos);
        else neg = fmaf(t, ext[mask][2], neg);
      }
    }
  };

  if (walk == 0) walk = (Cost::kTest >= Cost::kWalk * nbox) ? 1 : 0;
  float top[Q][3];
  if (walk == 0) {
    // An infinite value times an extent of zero is NaN, so a box that a lane
    // does not reach counts as well then: every box, whatever the lanes beside
    // it hold. (Bits of floats: +inf is above every number.)
    int largest = 0;
#pragma unroll
    for (int a = 0; a < Q; ++a)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        top[a][k] = wave_max(y[a][k]);
        largest = max(largest, __float_as_int(top[a][k]));
      }
    walk = largest >= 0x7f800000 ? 1 : 0;
  }
  if (walk > 0) {
    --walk;
#pragma unroll(Q == 1 ? 4 : 2)
    for (unsigned c = 0; c < (unsigned)nbox; ++c) all(box(c));
    return;
  }
  const int lane = threadIdx.x & 63;
  int cost = Cost::kTest;
  for (int c0 = 0; c0 < nbox; c0 += 64) {
    float l[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) l[k] = lo(c0 + lane, k);
    uint64_t m[Q], any = 0, two = 0, more = 0;
#pragma unroll
    for (int a = 0; a < Q; ++a) {
      m[a] = __builtin_amdgcn_ballot_w64(l[0] < top[a][0]) & __builtin_amdgcn_ballot_w64(l[1] < top[a][1]) &
             __builtin_amdgcn_ballot_w64(l[2] < top[a][2]);
      more |= two & m[a];
      two |= any & m[a];
      any |= m[a];
    }
    cost += Cost::kOwn * __builtin_popcountll(any);
    if (Q > 1) cost += (Cost::kPair - Cost::kOwn) * __builtin_popcountll(two);
    if (Q > 2) cost += (Cost::kAll - Cost::kPair) * __builtin_popcountll(more);
    // box i of the chunk, by the members that reach it
    auto visit = [&](unsigned i, const Box& b) {
      const uint64_t bit = 1ull << i;
      if (Q == 1) {
        own(y[0], b);
      } else if (!(two & bit)) {
        if (Q == 4 && ((m[Q - 1] | m[Q - 2]) & bit)) {
          if (m[Q - 1] & bit) own(y[Q - 1], b);
          else own(y[Q - 2], b);
        } else {
          if (m[Q > 1] & bit) own(y[Q > 1], b);
          else own(y[0], b);
        }
      } else if (Q > 2 && !(more & bit)) {
#pragma unroll
        for (int a = 0; a < Q; ++a)
#pragma unroll
          for (int d = a + 1; d < Q; ++d)
            if (m[a] & m[d] & bit) pair(y[a], y[d], b);
      } else {
        all(b);
      }
    };
    // two boxes at a time, so that one's corner is on its way while the other
    // is used
    uint64_t r = any;
    while (r) {
      const unsigned i0 = __builtin_ctzll(r);
      r &= r - 1;
      const bool second = r != 0;
      const unsigned i1 = second ? __builtin_ctzll(r) : i0;
      r &= r - 1;
      const Box b0 = box(c0 + i0), b1 = box(c0 + i1);
      visit(i0, b0);
      if (second) visit(i1, b1);
    }
  }
  if (cost >= Cost::kWalk * nbox) walk = kWalkSamples;
}

}  // namespace
}  // namespace bo
