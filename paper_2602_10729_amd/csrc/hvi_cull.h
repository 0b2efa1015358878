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
// mask of the boxes that the member may reach. The boxes that one member reaches
// are visited member by member for its own extent product; a box that two or
// more reach is visited for all its subsets' terms, after those before it of its
// members. Every term left out is exactly zero on every lane. Each member's own
// products and the larger subsets' terms have sums of their own (HviSums), and
// each sum takes its boxes in order: which boxes are visited, and by which loop,
// depends on the batches that share the wave, a batch's sums do not. What that
// order costs: where single boxes went first, then pairs, 32768 batches of 4,
// 279 boxes, 512 samples took 0.68 ms, now 0.72 (50 boxes reached a sample, 5 by
// two members), with a composite model 2.1, now 3.1 (173 reached, 54 by two, 20
// by more; a test box by box 5.9 and 10.2). One sum, the members chosen box by
// box, is slower by its branches (33331 constrained pairs, 137 boxes, 300 samples
// 249 us when these loops took 184). A box's corner and widths come through the
// scalar cache (its address is uniform) as scalar operands; the visits are bound
// by scalar issue (mask and address), so the address is a 32-bit offset in bytes,
// which the load adds itself (the pairs: 184 -> 164 us), and one box at a time or
// four measured 2-13% slower than two.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

// The kernels with q = 1 and 2 keep to 80 scalar registers: with more, only one
// of their workgroups of 16 waves fits a CU instead of two (the pairs above: 254
// us against 184 then). With q = 4 the vector registers leave room for one anyway.
#define BO_CULL_SGPRS __attribute__((amdgpu_num_sgpr(80)))

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

// Lower corner of box c, +inf (not reached) for c >= nbox.
__device__ __forceinline__ void load_corner(const float* boxes, int nbox, int c, float (&l)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) l[k] = c < nbox ? boxes[6 * c + k] : __builtin_huge_valf();
}

// When a wave's lanes are far apart (candidates with spread-out means and small
// variances) most boxes are marked and walking all of them in order is cheaper:
// no masks, addresses that only count up. For q <= 2 that is decided for each
// chunk of 64 from its masks (for q = 4 the second copy of the subsets' code in
// that loop costs more than it gives). The test itself is saved, too, where it
// keeps costing more than it saves: after two such samples in a row one is
// walked without a test, after three 3, then 7, then 15 (a sample's reach
// varies with its draw; 15 after the first such sample took 331 us for the
// pairs above). A front so small that the test alone costs more is always
// walked. A walk adds the zeros that a visit leaves out, nothing else changes.
// Issue costs in quarters of a box that one member reaches: two members, all
// members (q = 4), the test, a box of the walk.
template <int Q>
struct CullCost {
  static constexpr int kOwn = 4, kPair = 8, kAll = 28;
  static constexpr int kTest = Q == 1 ? 20 : Q == 2 ? 34 : 60;
  static constexpr int kWalk = Q == 1 ? 3 : Q == 2 ? 6 : 26;
};

// What a wave carries from sample to sample.
struct CullState {
  int skip = 0;     // samples to come that are walked without a test
  int run = 0;      // 2^i - 1 after i tested samples in a row that cost more
};

// The sums of a lane's terms: each member's own extent products, the
// intersections of three members, those of two and four.
template <int Q>
struct HviSums {
  float own[Q] = {}, odd = 0.f, even = 0.f;
  __device__ __forceinline__ float total() const {
    float v = own[0];
#pragma unroll
    for (int a = 1; a < Q; ++a) v += own[a];
    return Q > 2 ? (v + odd) - even : v - even;
  }
};

// Terms of the boxes boxes[0 .. nbox) ([c][6]: lower corner, then widths; the
// address is uniform) for the members' values y[a][k] of this lane, into h.
// corner(c, l): lower corner of box c, vector loads by lane, +inf for c >= nbox.
template <int Q, typename Corner>
__device__ __forceinline__ void box_terms3(const float (&y)[Q][3], const float* boxes, int nbox,
                                           Corner corner, CullState& st, HviSums<Q>& h) {
  using Cost = CullCost<Q>;
  typedef const char __attribute__((address_space(4)))* const_bytes;
  const const_bytes bx = (const_bytes)(uintptr_t)boxes;
  struct Box { float lo[3], w[3]; };
  auto box = [&](unsigned c) {
    // (a 32-bit offset in bytes: the load adds it to the base itself)
    const const_floats p = (const_floats)(bx + 24u * c);
    return Box{{p[0], p[1], p[2]}, {p[3], p[4], p[5]}};
  };
  auto extents = [&](const float (&v)[3], const Box& b, float (&e)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) e[k] = __builtin_amdgcn_fmed3f(v[k] - b.lo[k], 0.0f, b.w[k]);
  };
  auto own = [&](int a, const Box& b) {
    float e[3];
    extents(y[a], b, e);
    h.own[a] = fmaf(e[0] * e[1], e[2], h.own[a]);
  };
  auto pair = [&](int a, int d, const Box& b) {
    float e[3], f[3];
    extents(y[a], b, e);
    extents(y[d], b, f);
    h.own[a] = fmaf(e[0] * e[1], e[2], h.own[a]);
    h.own[d] = fmaf(f[0] * f[1], f[2], h.own[d]);
    h.even = fmaf(fminf(e[0], f[0]) * fminf(e[1], f[1]), fminf(e[2], f[2]), h.even);
  };
  auto all = [&](const Box& b) {
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
      float& sum = mask == low                       ? h.own[__builtin_ctz(mask)]
                   : (__builtin_popcount(mask) & 1) ? h.odd
                                                    : h.even;
      sum = fmaf(ext[mask][0] * ext[mask][1], ext[mask][2], sum);
    }
  };
  auto walk = [&](unsigned c, unsigned c1) {
#pragma unroll(Q == 1 ? 4 : 2)
    for (; c < c1; ++c) all(box(c));
  };

  if (st.skip > 0 || Cost::kTest >= Cost::kWalk * nbox) {
    st.skip = max(st.skip - 1, 0);
    walk(0, nbox);
    return;
  }
  // An infinite value, or the product of two that overflows, times an extent of
  // zero is NaN, so a box that a lane does not reach counts as well then: every
  // box, whatever the lanes beside it hold. Below 2^62 no product of two extents
  // overflows (the lower corners are observations' or the reference's values).
  // Bits of floats: their order is the numbers'.
  float top[Q][3];
  int largest = 0;
#pragma unroll
  for (int a = 0; a < Q; ++a)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      top[a][k] = wave_max(y[a][k]);
      largest = max(largest, __float_as_int(top[a][k]));
    }
  if (largest >= 0x5e800000) {
    walk(0, nbox);
    return;
  }
  const int lane = threadIdx.x & 63;
  int cost = Cost::kTest;
  for (int c0 = 0; c0 < nbox; c0 += 64) {
    float l[3];
    corner(c0 + lane, l);
    uint64_t m[Q], any = 0, two = 0, more = 0;
#pragma unroll
    for (int a = 0; a < Q; ++a) {
      m[a] = __builtin_amdgcn_ballot_w64(l[0] < top[a][0]) & __builtin_amdgcn_ballot_w64(l[1] < top[a][1]) &
             __builtin_amdgcn_ballot_w64(l[2] < top[a][2]);
      more |= two & m[a];
      two |= any & m[a];
      any |= m[a];
    }
    int visits = Cost::kOwn * __builtin_popcountll(any);
    if (Q > 1) visits += (Cost::kPair - Cost::kOwn) * __builtin_popcountll(two);
    if (Q > 2) visits += (Cost::kAll - Cost::kPair) * __builtin_popcountll(more);
    cost += visits;
    if constexpr (Q <= 2) {
      const int left = min(nbox - c0, 64);
      if (visits >= Cost::kWalk * left) {
        walk(c0, c0 + left);
        continue;
      }
    }
    // member a's boxes in r, two at a time (after an odd first one), both
    // requested before either is used
    auto visit = [&](uint64_t r, int a) {
      if (__builtin_popcountll(r) & 1) {
        own(a, box(c0 + __builtin_ctzll(r)));
        r &= r - 1;
      }
      while (r != 0) {
        const Box b0 = box(c0 + __builtin_ctzll(r));
        r &= r - 1;
        const Box b1 = box(c0 + __builtin_ctzll(r));
        r &= r - 1;
        __builtin_amdgcn_sched_barrier(0);
        own(a, b0);
        own(a, b1);
      }
    };
    if (two == 0) {
#pragma unroll
      for (int a = 0; a < Q; ++a) visit(m[a], a);
    } else if constexpr (Q > 1) {
      // a shared box waits for the boxes before it of its own members only
      uint64_t left[Q];                              // single boxes to come
#pragma unroll
      for (int a = 0; a < Q; ++a) left[a] = m[a] & ~two;
      for (uint64_t r = two; r != 0; r &= r - 1) {
        const unsigned i = __builtin_ctzll(r);
        const uint64_t below = (1ull << i) - 1;
        auto in = [&](uint64_t mask) { return (mask >> i) & 1; };
        const Box b = box(c0 + i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < Q; ++a)
          if (Q == 2 || in(m[a])) {
            const uint64_t now = left[a] & below;
            if (now != 0) {
              visit(now, a);
              left[a] &= ~now;
            }
          }
        if (Q == 2 || in(more)) {
          all(b);
        } else if (in(m[0])) {
          if (in(m[1])) pair(0, 1, b);
          else if (in(m[Q - 2])) pair(0, Q - 2, b);
          else pair(0, Q - 1, b);
        } else if (in(m[1])) {
          if (in(m[Q - 2])) pair(1, Q - 2, b);
          else pair(1, Q - 1, b);
        } else {
          pair(Q - 2, Q - 1, b);
        }
      }
#pragma unroll
      for (int a = 0; a < Q; ++a) visit(left[a], a);
    }
  }
  st.run = cost >= Cost::kWalk * nbox ? min(2 * st.run + 1, 31) : 0;
  st.skip = st.run >> 1;
}

}  // namespace
}  // namespace bo
