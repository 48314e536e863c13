// gv_probe.h -- look-ahead pruning of a chunk's pending children before their
// lists are written.
//
// A kept child's list is written by the compaction, read once by its own
// count pass, and dropped there when none of its children can still beat the
// best key.  Near the leaves that is what happens to nearly every list.  The
// probe decides it from the parent's list alone: it repeats the child's test
// on every parent entry, canonizes the survivors in registers and counts
// them over the child's own children, and it stops as soon as
//   - every grandchild's count plus the child entries not yet seen stays
//     below the bound (counts only shrink down the tree: no leaf below this
//     child can become the best, so the child is dropped), or
//   - a grandchild's share of the entries seen so far points above the bound
//     (the child is kept and takes the ordinary path).
// The first is exact, the second only chooses who does the work, so no
// result depends on the probe.
#pragma once
#include "gv_kernels.h"
#include "gv_subtree.h"

// Smallest count with which a leaf of the subtree of the child (index bits
// `pre` of level m + 1) can beat the best key: a larger count, or the same
// count at a lower leaf index.
__device__ inline uint32_t probe_need(uint64_t best, int B, uint64_t idxmask, uint64_t pre, int rem_next) {
  const uint64_t bc = best >> B, low = idxmask - (pre << rem_next);
  return (uint32_t)(bc + (low > (best & idxmask) ? 0ull : 1ull));
}

// v with lane L's value replaced by the wave-uniform x
template <int L> __device__ inline uint32_t put_lane(uint32_t v, uint32_t x) {
  asm("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(x), "n"(L));
  return v;
}

// PLANE3D, unit-weight lists, every axis splitting at the parent's level
// (lv) and the children's (lv2).  One wave takes a parent cell and reads its
// list once for all eight children, G rows of 64 entries at a time.  As in
// the compaction, with x = 2F + b1 K1 + b2 K2 - b0 H an entry passes child
// (b1, b2, b0) iff x + pad + S lies in [0, R], and its canonical height there
// is rne(x / 2); K1', K2' are the same in every child.  Lane 8 i + g of the
// wave holds the state of grandchild g of child i: its count so far and its
// child's entries seen, total and needed count.
// Bound by the vector unit (about 28 instructions a row and child, two scalar
// ones per grandchild beside them).  The counters as vector lanes, filled
// once per block, keep the scalar registers free: as scalars they spilled
// (two or four children a wave) and the pass took 459 instead of 319 ms of a
// plane3d_1m solve.  G = 4, 6 and 8 rows measured 331, 316 and 319 ms, and
// 266, 257 and 255 on another input.
template <typename E>
__global__ void __launch_bounds__(256) k_probe_p3(LevelC lv, LevelC lv2, int B, uint64_t idxmask,
                                                  const Cell* __restrict__ cells, uint32_t ncell,
                                                  const E* __restrict__ ents, const uint32_t* __restrict__ rank_of,
                                                  const uint32_t* __restrict__ cnent, uint32_t r0, uint32_t r1,
                                                  const unsigned long long* __restrict__ best, uint32_t* keepc,
                                                  uint64_t* csize, unsigned long long* __restrict__ tests,
                                                  unsigned long long* __restrict__ reads) {
  constexpr int G = 8;
  const uint32_t lane = lane_id(), child = lane >> 3;
  const uint32_t wave = uniform_u32((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const uint32_t nwaves = (gridDim.x * blockDim.x) >> 6;
  const int32_t H = lv.H[2], pad = lv.padu[2], H2 = lv2.H[2], pad2 = lv2.padu[2];
  uint64_t ntests = 0, nread = 0;
  for (uint32_t c = wave; c < ncell; c += nwaves) {
    const uint64_t off = uniform_u64(cells[c].off), prefix = uniform_u64(cells[c].prefix);
    const uint32_t len = uniform_u32(cells[c].len);
    const uint32_t rank = rank_of[c * 8 + child];
    const bool pend = rank >= r0 && rank < r1 && keepc[rank - r0];
    uint64_t open = __builtin_amdgcn_ballot_w64(pend);  // children undecided (eight bits each)
    if (!open) continue;
    const uint32_t tot = cnent[c * 8 + child];
    const uint32_t need = probe_need(best[cells[c].prob], B, idxmask, (prefix << 3) | child, lv.rem_next);
    const float hope = 1.125f * (float)need / (float)max(tot, 1u);  // share of the seen that points an eighth above need
    uint32_t cnt = 0, seen = 0;
    uint64_t drop = 0;
    for (uint32_t k0 = 0; k0 < len && open; k0 += 64 * G) {
      E ev[G];
      if (k0 + 64 * G <= len) {
#pragma unroll
        for (int j = 0; j < G; j++) ev[j] = ents[off + k0 + 64 * j + lane];
      } else {
#pragma unroll
        for (int j = 0; j < G; j++) {
          const uint32_t k = k0 + 64 * j + lane;
          ev[j] = E{};
          if (k < len) ev[j] = ents[off + k];
        }
      }
      nread += min(len - k0, 64u * G);
      // X = 2F, SP = pad + S, and in the child SB = pad' + S', RR = R'.
      // Lanes past the list's end get an SP that passes nothing.
      int32_t X[G], KA[G], KB[G], KA1[G], KB1[G], SB[G];
      uint32_t SP[G], R[G], RR[G];
#pragma unroll
      for (int j = 0; j < G; j++) {
        const LinS s = load_ent<FAM_PLANE3D>(ev[j]);
        const int32_t S = imax32(s.K[0][0], 0) + imax32(s.K[0][1], 0);
        X[j] = 2 * s.F[0];
        KA[j] = s.K[0][0];
        KB[j] = s.K[0][1];
        SP[j] = k0 + 64 * j + lane < len ? (uint32_t)(pad + S) : GV_NOWHERE;
        R[j] = (uint32_t)(2 * S + (H + 2 * pad) - (KA[j] + KB[j]));
        KA1[j] = rne_half(KA[j]);
        KB1[j] = rne_half(KB[j]);
        const int32_t S1 = imax32(KA1[j], 0) + imax32(KB1[j], 0);
        SB[j] = pad2 + S1;
        RR[j] = (uint32_t)(2 * S1 + (H2 + 2 * pad2) - (KA1[j] + KB1[j]));
      }
      uint32_t dn = 0;  // this block's counts, lane 8 i + g
#define GV_PROBE_CHILD(I)                                                                                              \
  if ((open >> (8 * I)) & 1u) {                                                                                        \
    uint32_t got = 0, n[8] = {0, 0, 0, 0, 0, 0, 0, 0};                                                                 \
    _Pragma("unroll") for (int j = 0; j < G; j++) {                                                                    \
      const int32_t x = X[j] + ((I & 4) ? KA[j] : 0) + ((I & 2) ? KB[j] : 0) - ((I & 1) ? H : 0);                      \
      const bool p = in_range(x, SP[j], R[j]);                                                                         \
      got += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(p));                                                       \
      /* 2 rne(x / 2) + pad' + S'; out of every grandchild's range where the child's own test fails */                 \
      const int32_t U = p ? ((x + ((x >> 1) & 1)) & ~1) + SB[j] : (int32_t)0x40000000;                                 \
      _Pragma("unroll") for (int q = 0; q < 4; q++) {                                                                  \
        const int32_t uu = U + ((q & 2) ? KA1[j] : 0) + ((q & 1) ? KB1[j] : 0);                                        \
        n[2 * q] += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64((uint32_t)uu <= RR[j]));                            \
        n[2 * q + 1] += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64((uint32_t)(uu - H2) <= RR[j]));                 \
      }                                                                                                                \
    }                                                                                                                  \
    ntests += 8u * got;                                                                                                \
    seen += child == I ? got : 0u;                                                                                     \
    dn = put_lane<8 * I>(dn, n[0]);                                                                                    \
    dn = put_lane<8 * I + 1>(dn, n[1]);                                                                                \
    dn = put_lane<8 * I + 2>(dn, n[2]);                                                                                \
    dn = put_lane<8 * I + 3>(dn, n[3]);                                                                                \
    dn = put_lane<8 * I + 4>(dn, n[4]);                                                                                \
    dn = put_lane<8 * I + 5>(dn, n[5]);                                                                                \
    dn = put_lane<8 * I + 6>(dn, n[6]);                                                                                \
    dn = put_lane<8 * I + 7>(dn, n[7]);                                                                                \
  }
      GV_PROBE_CHILD(0)
      GV_PROBE_CHILD(1)
      GV_PROBE_CHILD(2)
      GV_PROBE_CHILD(3)
      GV_PROBE_CHILD(4)
      GV_PROBE_CHILD(5)
      GV_PROBE_CHILD(6)
      GV_PROBE_CHILD(7)
#undef GV_PROBE_CHILD
      cnt += dn;
      // a child with no grandchild that can still get there is dropped; one
      // with a grandchild on its way is left to the ordinary path
      uint64_t can = __builtin_amdgcn_ballot_w64(cnt + (tot - seen) >= need);
      uint64_t will = __builtin_amdgcn_ballot_w64(seen >= 1024u && (float)cnt >= hope * (float)seen);
      for (int o = 1; o < 8; o <<= 1) {  // any bit of a child's eight, in its lowest
        can |= can >> o;
        will |= will >> o;
      }
      can = (can & 0x0101010101010101ull) * 0xffull;
      will = (will & 0x0101010101010101ull) * 0xffull;
      drop |= open & ~can;
      open &= can & ~will;
    }
    if ((lane & 7u) == 0 && ((drop >> lane) & 1ull)) {
      keepc[rank - r0] = 0;
      csize[rank - r0] = 0;
    }
  }
  if (lane == 0 && ntests) atomicAdd(tests, (unsigned long long)ntests);
  if (lane == 0 && nread) atomicAdd(reads, (unsigned long long)nread * sizeof(E));
}

// The popcounts of the wave's mask bits L..N-1 in lanes L..N-1
template <int N, int L = 0> __device__ inline uint32_t bit_counts(uint32_t mask, uint32_t v = 0) {
  if constexpr (L < N) {
    const bool p = (mask >> L) & 1u;
    return bit_counts<N, L + 1>(mask, put_lane<L>(v, (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(p))));
  } else {
    return v;
  }
}

// Pose families, unit-weight lists, every axis splitting at the children's
// level (lv2).  One wave takes one pending child (rank r).  It reads the
// parent's pass masks, queues the child's survivors (their places in the
// parent's list) in LDS, and tests them 64 at a time against the child's own
// children, reading the entries from the parent's list; lane g < NCH counts
// grandchild g.  The waves of a workgroup mostly hold children of one parent.
// min_blocks as for the count kernels.
template <int FAM, typename E> constexpr int probe_min_blocks() {
  return FAM == FAM_POSE5DOF ? pose5_min_blocks<E>() : 4;
}
template <int FAM, typename E>
__global__ void __launch_bounds__(256, (probe_min_blocks<FAM, E>())) k_probe_pose(
    const ProbC* __restrict__ Ptab, int m, LevelC lv, LevelC lv2, int B, uint64_t idxmask,
    const Cell* __restrict__ cells, const E* __restrict__ ents, const typename RecOf<E>::T* __restrict__ rec,
    const typename SubFam<FAM>::M* __restrict__ masks, const double* __restrict__ m64, uint64_t n_root, const uint32_t* __restrict__ order,
    const uint32_t* __restrict__ cnent, uint32_t r0, uint32_t r1, const unsigned long long* __restrict__ best,
    uint32_t* keepc, uint64_t* csize, unsigned long long* __restrict__ tests, unsigned long long* __restrict__ reads,
    unsigned long long* __restrict__ rechecks) {
  using F = SubFam<FAM>;
  constexpr int NCH = F::NCH;
  constexpr uint64_t KIDS = NCH == 32 ? 0xffffffffull : 0xffffull;
  __shared__ uint32_t queue[4][128];  // one wave each: at most 63 waiting and 64 new
  const uint32_t lane = lane_id(), nch = 1u << lv.abits;
  uint32_t* const q = queue[threadIdx.x >> 6];
  const uint32_t wave = uniform_u32((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
  const uint32_t nwaves = (gridDim.x * blockDim.x) >> 6;
  uint64_t ntests = 0, nread = 0;
  uint32_t nre = 0;
  for (uint32_t r = r0 + wave; r < r1; r += nwaves) {
    if (!uniform_u32(keepc[r - r0])) continue;
    const uint32_t k = uniform_u32(order[r]), c = k / nch, ch = k % nch;
    Cell C = cells[c];
    const uint64_t off = C.off;
    const uint32_t len = C.len, tot = uniform_u32(cnent[k]);
    const ProbC& P = Ptab[C.prob];
    const uint32_t need = probe_need(uniform_u64(best[C.prob]), B, idxmask, (C.prefix << lv.abits) | ch, lv.rem_next);
    const float hope = 1.125f * (float)need / (float)max(tot, 1u);
    const uint32_t cb = lv.cbits[ch];
    for (int a = 0; a < GV_MAXD; a++) C.c[a] = lv.split[a] ? 2 * C.c[a] + (int32_t)((cb >> a) & 1u) : C.c[a];
    typename F::Boxes Bx;
    float Bf[F::NBF];
    F::boxes(P, lv2, C, m + 1, Bx, Bf);
    uint32_t cnt = 0, seen = 0, head = 0, tail = 0;
    bool open = true, drop = false;
    uint32_t mk = lane < len ? (uint32_t)masks[off + lane] : 0u;
    for (uint32_t k0 = 0; k0 < len && open; k0 += 64) {
      const uint32_t kn = k0 + 64 + lane;
      const uint32_t mkn = kn < len ? (uint32_t)masks[off + kn] : 0u;  // the next row's, on its way
      const bool p = (mk >> ch) & 1u;
      const uint64_t bal = __builtin_amdgcn_ballot_w64(p);
      if (p) q[(tail + mbcnt64(bal)) & 127u] = k0 + lane;
      tail += (uint32_t)__popcll(bal);
      mk = mkn;
      const bool last = k0 + 64 >= len;
      if (tail - head < 64u && !last) continue;
      __builtin_amdgcn_wave_barrier();
      // (the last row may leave more than 64 waiting)
      do {
        const uint32_t n = min(tail - head, 64u);
        uint32_t mask = 0;
        if (lane < n) {
          const typename RecOf<E>::T e = pose_rec(ents, off + q[(head + lane) & 127u], rec);
          mask = F::template mask_as<true, typename RecOf<E>::T>(P, lv2, C, m + 1, Bx, Bf, e, m64, n_root, nre);
        }
        head += n;
        seen += n;
        cnt += bit_counts<NCH>(mask);
        if (!(__builtin_amdgcn_ballot_w64(cnt + (tot - seen) >= need) & KIDS)) {
          drop = true;
          open = false;
        } else if (seen >= 512u && (__builtin_amdgcn_ballot_w64((float)cnt >= hope * (float)seen) & KIDS)) {
          open = false;
        }
      } while (last && open && tail != head);
      __builtin_amdgcn_wave_barrier();
    }
    ntests += (uint64_t)NCH * seen;
    nread += seen;
    if (drop && lane == 0) {
      keepc[r - r0] = 0;
      csize[r - r0] = 0;
    }
  }
  if (lane == 0 && ntests) {
    atomicAdd(tests, (unsigned long long)ntests);
    atomicAdd(reads, (unsigned long long)nread * (RecOf<E>::idx ? sizeof(E) + sizeof(typename RecOf<E>::T) : sizeof(E)));
  }
  const uint32_t re = wave_sum_u32(nre);
  if (lane == 0 && re) atomicAdd(rechecks, (unsigned long long)re);
}
