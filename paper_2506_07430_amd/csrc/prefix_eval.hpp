// Prefix-shared local energies: the loop over a sample's parents and entries (the scheme is in
// prefix.hpp), for either precision. Net supplies the network: its value types, one pass over
// rows of a tile (rows), the log-softmax of one orbital (step), the ratio of one entry, and
// where a wave reads from (Sources).
//
// Measured against kernels that run every entry's whole network (k_eval_bf16, k_eval_f64), whole
// calls on one MI355X (where it is taken: prefix_pays in api.cpp):
//   60 orbitals, 256x3, 128 samples   BF16 72.9 -> 30.5 ms   17 samples  FP64 119 -> 29.0 ms
//   40 orbitals, 256x3, 512 samples   BF16 43.7 -> 22.5 ms (with the gradient)
//   24 orbitals, 128x2, 4096 samples  BF16 14.7 -> 10.0 ms (with the gradient)   1024 samples FP64 38.1 -> 13.4 ms
// At 60 orbitals 8.8 of 29.75 matrix instructions per entry are left and two waves per SIMD
// wait 31% of their cycles; at 24 orbitals vector issue (33 instructions per entry, 2.4 of
// them products) bounds the kernel, whose checkpoints (18 KB a wave) stream through the
// last-level cache at 3 TB/s.
#pragma once
#include <type_traits>

#include "elocal_internal.hpp"
#include "kernels.hpp"
#include "made_bf16.hpp"
#include "prefix.hpp"

namespace elocal {

// The kernel arguments through the constant address space: scalar loads. `opaque` hides where
// the pointer comes from, so that the loads stay where they are written: hoisted out of the
// loops, the tables of every pass variant together overflow the scalar registers, and each
// use then costs a v_readlane.
typedef const __attribute__((address_space(4))) PrefixArgs CArgs;
__device__ __forceinline__ CArgs* opaque(CArgs* p) {
  asm volatile("" : "+s"(p));
  return p;
}

// The same for the lane index: what is derived from it (shuffle addresses, lane-group offsets)
// is cheaper to compute again than to hold in registers, or in spill slots, across the kernel.
__device__ __forceinline__ int opaque(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  // word 3 = 0x00020000: raw (untyped) buffer access on the gfx9 family
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// The output layer of these networks: 4(n - 1) logits (the last orbital's conditional is 1)
// and the phase row.
__device__ __forceinline__ int prefix_phase_row(int n) { return 4 * (n - 1); }

// What a wave keeps of the sample its current work item belongs to.
template <int NW>
struct PrefixSample {
  int64_t b;
  uint64_t xs[NW];
  SpinMasks m;
  double sig_x, ed;
  const double* Fs;
};

// Adds the 64 lanes' terms to a slot of the wave's sums: lane `slot` keeps the real part, lane
// 32 + slot the imaginary part. A segment's groups go to the slots in turn and the slots are
// added in a fixed order, so that the sum is the same whether one wave runs the segment or
// 2^k waves each run every 2^k-th of its groups.
__device__ __forceinline__ void add_to_slot(double re, double im, uint32_t slot, int lane0, double& sum) {
  const int lane = opaque(lane0);
  const double v = wave_sum_complex(re, im);
  sum += (uint32_t)(lane & 31) == (slot & 31u) ? v : 0.0;
}

// One group of up to 64 entries of class b, one per lane: the network in passes of NC tiles,
// then the lane's term H exp(dA + i dphi), added to the slot's sum.
template <class Net, int NB, int NC, int NW, bool BASE>
__device__ __forceinline__ void run_group(CArgs* args, const SysDev& S, const typename Net::Sources& src,
                                          PrefixWave& pw, const PrefixSample<NW>& st, uint32_t stot, int b, int rows,
                                          const uint64_t (&xo)[NW], int parent, int p0, int p2, double hv, int lane0,
                                          uint32_t slot, double& sum) {
  typedef typename Net::Real Real;
  const int n = S.n, na = S.na, nb = S.nb;
  const int ob_phi = prefix_phase_row(n) >> 4, g_phi = (prefix_phase_row(n) & 15) >> 2;
  const int p2_row = row_min(p2);
  double dA_own = 0.0;
  Real zp_own = 0;
  // the entry's epilogue state at the class's first output block, once per entry: a pass
  // only advances it to its own first block and to the lane group's orbital
  const int obq = opaque(args)->px.cls[b].obq;
  const RowCursor<NW> own = cursor_at<NW>(xo, 4 * obq);
  const uint32_t own_cnt = (uint32_t)(own.cu | own.cd << 16);
#pragma unroll 1
  for (int h = 0; h * 16 * NC < rows; ++h) {
    const int lane = opaque(lane0), g = lane >> 4, r16 = lane & 15;
    uint64_t xr[NC][NW];
    int p0r[NC];
    uint32_t cko[NC];
    RowCursor<NW> cr[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int src_lane = 16 * NC * h + 16 * c + r16;
#pragma unroll
      for (int w = 0; w < NW; ++w) xr[c][w] = __shfl(xo[w], src_lane);
      p0r[c] = __shfl(p0, src_lane);
#pragma unroll
      for (int w = 0; w < NW; ++w) cr[c].bits[w] = __shfl(own.bits[w], src_lane);
      const uint32_t cnt = (uint32_t)__shfl((int)own_cnt, src_lane);
      cr[c].cu = cnt & 0xFFFFu;
      cr[c].cd = cnt >> 16;
      cko[c] = (uint32_t)__shfl(parent, src_lane) * stot * Net::kSlotBytes + Net::kSlotBytes / 4u * g;
    }
    int obf = __builtin_amdgcn_readlane(p2_row, 16 * NC * h);
#pragma unroll
    for (int c = 1; c < NC; ++c) obf = min(obf, __builtin_amdgcn_readlane(p2_row, 16 * NC * h + 16 * c));
    obf = sgpr(min(obf >> 2, ob_phi));
    double dA[NC];
    Real zp[NC];
    RowCursor<NW> rc[NC];
    auto pre = [&] {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        dA[c] = 0.0;
        zp[c] = 0;
        rc[c] = cr[c];
        for (int ob = obq; ob < obf; ++ob) cursor_advance4<NW>(rc[c], (uint32_t)rc[c].bits[0] & 0xFFu);
        cursor_advance<NW>(rc[c], g);
      }
    };
    Net::template rows<NB, NC, NW, BASE>(args, src, xr, lane, b, cko, obf, NB, false, pre,
                                         [&](int ob, const typename Net::Acc (&a)[NC]) {
      const int p = 4 * ob + g;
      if (p < n - 1) {   // the last orbital's conditional is 1
        const int ta = na - (n - p - 1), tb = nb - (n - p - 1);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const Real lp = Net::template step<NW>(rc[c], ta, tb, na, nb, a[c]);
          Real d = p >= p0r[c] ? lp : (Real)0;
          asm volatile("" : "+v"(d));   // keeps the select in the type of lp (before the convert)
          dA[c] += (double)d;
        }
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) zp[c] = a[c][0];   // the phase row is the last block's
    });
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      dA[c] += __shfl_xor(dA[c], 16);
      dA[c] += __shfl_xor(dA[c], 32);
      zp[c] = __shfl(zp[c], g_phi * 16 + r16);
    }
    if (lane / (16 * NC) == h) {
      const int c = (lane >> 4) % NC;
      double dsel = dA[0];
      Real zsel = zp[0];
#pragma unroll
      for (int cc = 1; cc < NC; ++cc)
        if (c == cc) { dsel = dA[cc]; zsel = zp[cc]; }
      // the orbitals below the pass's first block are the parent's
      dA_own = dsel + pw.ag[parent][obf];
      zp_own = zsel;
    }
  }
  double2 r = make_double2(0.0, 0.0);
  if (hv != 0.0) r = Net::ratio(hv, zp_own, st.sig_x, dA_own);   // (invalid lanes have H = 0)
  add_to_slot(r.x, r.y, slot, lane0, sum);
}

// Calls f(integral_constant<nblk>), LO <= nblk <= NB.
template <int NB, int LO, class F>
__device__ __forceinline__ void with_blocks(int nblk, F&& f) {
  if constexpr (NB > LO) {
    if (nblk < NB) {
      with_blocks<NB - 1, LO>(nblk, f);
      return;
    }
  }
  f(std::integral_constant<int, NB>{});
}

// One segment: up to 16 parents of one class of c2. Their tile runs first (checkpoints, the
// parents' own single excitations), then the entries class by class in groups of 64. The wave
// takes every (mask + 1)-th group, from `part` on; the parents' excitations are group 0.
// LO: the fewest blocks of a network that the kernel takes.
template <class Net, int HB, int LO, int NW>
__device__ __forceinline__ void run_segment(const PrefixArgs& P, CArgs* args, const typename Net::Sources& src,
                                            PrefixWave& pw, const PrefixSample<NW>& st, uint32_t seg, uint32_t part,
                                            uint32_t mask, int lane0, double& sum) {
  typedef typename Net::Real Real;
  const SysDev& S = P.sys;
  CArgs* q = opaque(args);
  const int n = S.n, na = S.na, nb = S.nb, nblk = q->px.nblk;
  const int g_phi = (prefix_phase_row(n) & 15) >> 2;
  int cls = 0;
  while (cls + 1 < nblk && seg >= q->px.seg0[cls + 1]) ++cls;
  const int ng = q->px.ng[cls];
  const uint32_t r0 = q->px.rank0[cls] + (seg - q->px.seg0[cls]) * (uint32_t)ng;
  const int np = (int)min((uint32_t)ng, q->px.rank0[cls + 1] - r0);   // parents of this segment
  const uint32_t stot = q->px.stot[cls];
  const int bst = max(1, cls);
  // each lane's parent (lane % 16) is derived again where it is needed, which is cheaper
  // than holding it in registers through the network
  auto parent = [&](int r16, int& c1, int& c2, int& k1, int& k2) {
    unrank_parent(r0 + (uint32_t)min(r16, np - 1), c1, c2);
    k1 = getbit<NW>(st.xs, c1);
    k2 = getbit<NW>(st.xs, c2);
  };
  // ---- the parents
  {
    const int lane = opaque(lane0), g = lane >> 4, r16 = lane & 15;
    double v = lane < n - 1 ? Net::sample_lp(P, st.b * n + lane) : 0.0;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double u = __shfl_down(v, off);
      if (lane + off < 64) v += u;
    }
    wave_sync_lds();     // the last class's rectangles are no longer read
    pw.sfx[lane] = v;    // lanes >= n - 1 sum nothing: 0
    wave_sync_lds();
    int c1, c2, k1, k2;
    parent(r16, c1, c2, k1, k2);
    uint64_t xg[1][NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) xg[0][w] = st.xs[w];
    flip<NW>(xg[0], c1);
    flip<NW>(xg[0], c2);
#pragma unroll
    for (int w = 0; w < NW; ++w)
      if (g == w) pw.xg[r16][w] = xg[0][w];
    const int p0 = c1 >> 1;
    const int obf = sgpr(__builtin_amdgcn_readlane(row_min(p0), 0) >> 2);
    const uint32_t cko[1] = {(uint32_t)r16 * stot * Net::kSlotBytes + Net::kSlotBytes / 4u * g};
    RowCursor<NW> rc;
    double dA = 0.0;
    Real zp = 0;
    auto pre = [&] {
      rc = cursor_at<NW>(xg[0], min(4 * obf + g, n - 1));
      dA = g == 0 ? -pw.sfx[p0] : 0.0;
    };
    auto epi = [&](int ob, const typename Net::Acc (&a)[1]) {
      double t = dA;
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);
      if (g == 0) pw.ag[r16][ob] = t;
      const int p = 4 * ob + g;
      if (p < n - 1) {
        const int ta = na - (n - p - 1), tb = nb - (n - p - 1);
        const Real lp = Net::template step<NW>(rc, ta, tb, na, nb, a[0]);
        dA += (double)(p >= p0 ? lp : (Real)0);
      }
      zp = a[0][0];
    };
    with_blocks<HB, LO>(nblk, [&](auto nbc) {
      Net::template rows<decltype(nbc)::value, 1, NW, true>(args, src, xg, lane, 0, cko, obf, bst, r16 < np, pre, epi);
    });
    dA += __shfl_xor(dA, 16);
    dA += __shfl_xor(dA, 32);
    zp = __shfl(zp, g_phi * 16 + r16);
    double2 r = make_double2(0.0, 0.0);
    Excitation e;
    const bool single = parent_single(S, st.m, c1, c2, k1, k2, e);
    if (single && lane < np) {
      uint64_t xp[NW];
      const int sn = apply_excitation<NW>(st.xs, e, xp);
      const double v = excitation_value(S, e, st.Fs, st.ed);
      const double hv = sn < 0 ? -v : v;
      if (hv != 0.0) r = Net::ratio(hv, zp, st.sig_x, dA);
    }
    if (part == 0) add_to_slot(r.x, r.y, 0, lane0, sum);
  }
  // checkpoints and the table above are read by other lanes of this wave
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  // ---- their entries
  Segment sg;
  {
    const int lane = opaque(lane0), r16 = lane & 15;
    int c1, c2, k1, k2;
    parent(r16, c1, c2, k1, k2);
    sg = make_segment<NW>(st.xs, st.m, c1, c2, k1, k2, (lane >> 4) & 1, r16, r16 < np);
  }
  uint32_t gi = 0;
  for (int b = cls, bn; b < nblk; b = bn) {
    uint32_t total;
    for (bn = b + 1;;) {
      const int lane = opaque(lane0);
      wave_sync_lds();   // the previous class's rectangles are no longer read
      total = post_class(pw, sg, q->px.cls[b].qb, q->px.cls[bn].qb, lane);
      // a group that the next class's entries still fit in takes them along (their own
      // boundary is a later one; an earlier one is as good)
      if (bn >= nblk || total > 48u) break;
      const uint32_t more = post_class(pw, sg, q->px.cls[b].qb, q->px.cls[bn + 1].qb, lane);
      if (more > 64u) {
        total = post_class(pw, sg, q->px.cls[b].qb, q->px.cls[bn].qb, lane);
        break;
      }
      ++bn;
      total = more;
      if (bn >= nblk) break;
    }
    wave_sync_lds();
    for (uint32_t t0 = 0; t0 < total; t0 += 64u) {
      if ((++gi & mask) != part) continue;
      const int lane = opaque(lane0);
      const int rows = (int)min(64u, total - t0);
      uint64_t xo[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) xo[w] = st.xs[w];
      double hv = 0.0;
      int par = 0, p0 = n, p2 = n;
      if (lane < rows) {
        const PrefixEntry<NW> en = prefix_entry<NW>(S, pw, t0 + lane);
#pragma unroll
        for (int w = 0; w < NW; ++w) xo[w] = en.x[w];
        hv = en.h;
        par = en.parent;
        p0 = en.p0;
        p2 = en.p2;
      }
      auto go = [&](auto nbc, auto basec) {
        constexpr int NB = decltype(nbc)::value;
        constexpr bool BASE = decltype(basec)::value;
        run_group<Net, NB, BASE ? 1 : Net::cols(NB), NW, BASE>(args, S, src, pw, st, stot, b, rows, xo, par, p0, p2, hv,
                                                               lane, gi, sum);
      };
      if (b == 0) with_blocks<HB, LO>(nblk, [&](auto nbc) { go(nbc, std::true_type{}); });
      else with_blocks<HB - 1, 1>(nblk - b, [&](auto nbc) { go(nbc, std::false_type{}); });
    }
  }
}

// What of a sample its part `part` runs: segments [s0, s1), of every segment the groups
// k, k + mask + 1, ...
struct ItemSpan {
  uint32_t s0, s1, k, mask;
};
__device__ __forceinline__ ItemSpan item_span(const PrefixArgs& P, uint32_t part) {
  const uint32_t spi = P.px.spi;
  if (spi != 0) return {part * spi, min(P.px.seg0[P.px.nblk], part * spi + spi), 0u, 0u};
  int c = 0;
  while (c + 1 < P.px.nblk && part >= P.px.item0[c + 1]) ++c;
  const uint32_t i = part - P.px.item0[c], mask = (1u << P.px.lgk[c]) - 1u, s0 = P.px.seg0[c] + (i >> P.px.lgk[c]);
  return {s0, s0 + 1u, i & mask, mask};
}

// One ticket: of one sample (or, in a batch of more work items than tickets, of samples
// P.px.bt apart) P.px.spi segments, or (spi = 0) a part of one of them. The partial sums go to
// P.partial.
template <class Net, int HB, int LO, int NW>
__device__ __forceinline__ void run_item(const PrefixArgs& P, CArgs* args, const typename Net::Sources& src,
                                         PrefixWave& pw, uint32_t ticket, PrefixSample<NW>& st, int lane) {
  const SysDev& S = P.sys;
  // parts of segments: the same part of every sample in turn, so that the long ones (of the
  // first classes) are run first and the short ones fill the launch's end
  const uint32_t by = P.px.spi == 0 ? P.px.bt : P.ips, hi = ticket / by, lo = ticket - hi * by;
  uint32_t part = P.px.spi == 0 ? hi : lo;
#pragma unroll 1
  for (int64_t b = P.px.spi == 0 ? lo : hi; b < P.B; b += P.px.bt) {
    if (b != st.b) {
      wave_sync_lds();
#pragma unroll
      for (int w = 0; w < NW; ++w) st.xs[w] = w < S.W ? P.x[b * S.W + w] : 0ull;
      st.m = spin_lists<NW>(st.xs, S.n, lane, pw.c);
      wave_sync_lds();
      st.sig_x = sigmoid64(P.zphi[b]);
      st.ed = P.ediag[b];
      st.Fs = P.F + (size_t)b * (S.nSa + S.nSb);
      st.b = b;
    }
    double total = 0.0;
    {
      const ItemSpan it = item_span(P, part);
      for (uint32_t seg = it.s0; seg < it.s1; ++seg) {
        double sum = 0.0;
        run_segment<Net, HB, LO, NW>(P, args, src, pw, st, (uint32_t)sgpr((int)seg), (uint32_t)sgpr((int)it.k),
                                     (uint32_t)sgpr((int)it.mask), lane, sum);
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
        total += sum;
      }
    }
    // (derived again: held across the segments, the 64-bit positions cost registers)
    part = (uint32_t)sgpr((int)part);
    asm volatile("" : "+s"(part));
    const ItemSpan it = item_span(P, part);
    int64_t at = st.b * P.ips + part, end = at + 1;
    if (P.px.spi == 0) {
      const int64_t seg = st.b * P.px.seg0[P.px.nblk] + it.s0;
      at = (seg << P.px.lgp) + it.k;
      end = (seg + 1) << P.px.lgp;   // a segment of fewer parts than others: zeros after them
    }
    for (; at < end; at += it.mask + 1) {
      if ((lane & 31) == 0) P.partial[2 * at + (lane >> 5)] = total;
      total = 0.0;
    }
  }
}

// Takes the launch's next ticket (wave-uniform); false once all are taken. Every wave's last
// ticket is past the end: the host keeps their number and the waves of the grid below 2^32.
__device__ __forceinline__ bool next_ticket(const PrefixDev& X, int lane, uint32_t& t) {
  t = 0;
  if (lane == 0) t = atomicAdd(X.queue, 1u);
  t = (uint32_t)sgpr((int)t);
  return t < X.tickets;
}

}  // namespace elocal
