// Prefix-shared evaluation: the list entries of a sample, grouped by what they share.
//
// A single or double excitation changes spin-orbitals c1 < c2 (< c3 < c4), two per spin
// created and annihilated in equal number. The pair (c1, c2) is the entry's parent: x with c1
// and c2 changed. In an autoregressive network everything that depends on orbitals below
// c3's only is the parent's: hidden units of low degree, the conditionals of those orbitals,
// and the partial sums of every later unit over the low-degree units. So a wave runs a tile
// of up to 16 parents through the network once, keeping the accumulators at every class
// boundary (checkpoints), and each of their entries continues from there. An entry of
// class b costs the (nblk - b)-block triangle at the end of each layer instead of the whole
// layer; over a list the first three changes are spread like order statistics of uniform
// orbitals, which leaves about a quarter of the products (60 orbitals: 146 of 526 matrix
// instructions per 16 entries) and 0.43 of the conditionals. Accumulation orders are those of
// the whole network, so every logit is bit for bit what it was.
//
// The entries of a parent are products of suffixes of the sample's occupied and virtual
// lists: c3 and c4 complete the excitation, both above c2.
//   c1, c2 of different spin: one change of each spin, of the kind opposite to the parent's
//     change of that spin (segment A);
//   same spin, same kind: a pair from that spin's list of the opposite kind (segment A);
//   same spin, opposite kinds: the parent is itself a single excitation; an occupied and a
//     virtual orbital of the same spin (A), or of the other spin (B).
// With u_q (v_q) the length of the suffix from orbital q on, u_q v_q pairs have both members
// at or above q, so those whose smaller member lies in class b form an L of two rectangles.
#pragma once
#include "elocal_internal.hpp"
#include "kernels.hpp"

namespace elocal {

constexpr int kTileParents = 16;

// Occupied (kind 0) and virtual (kind 1) orbitals of the sample, list 2 * kind + spin at
// entry 64 * (2 * kind + spin): bits 0..5 the orbital, bit 7 the parity of the number of
// occupied spin-orbitals below that spin-orbital.
struct SampleLists {
  uint8_t e[4 * kMaxOrb];
};

// Entries of one rectangle of a segment (see post_class).
struct Rect {
  uint32_t lists;   // first entry of the two lists: u | v << 16
  uint32_t sel;     // byte selector that puts (c1, c2, u, v) into the roles (i, j, a, b)
  uint32_t fix;     // orbitals of c1, c2 (6 bits each), tile parent << 12, sign << 16, their order's
                    // share of the sign << 17, same spin << 18, triangle << 19, spins of u, v << 20, 21,
                    // entries per row << 24
  uint32_t start;   // number of entries before it
};

// Per-wave LDS state.
struct PrefixWave {
  SampleLists c;
  double ag[kTileParents][16];              // parent's part of log2 p below each output block
  uint64_t xg[kTileParents][2];             // the parents' words
  union {
    Rect rect[64];                          // rectangles of the current class
    double sfx[kMaxOrb];                    // before that: sum_{p >= q} log2 p_p(s_p) of the sample
  };
  uint32_t end[64];                         // running number of entries up to and with each
};

static_assert(sizeof(PrefixWave) == kPrefixWaveBytes, "per-wave LDS state");

// Occupied (0) and virtual (1) orbitals per spin, wave-uniform.
struct SpinMasks {
  uint64_t a0, a1, b0, b1;   // alpha occupied, alpha virtual, beta occupied, beta virtual
  __device__ __forceinline__ uint64_t get(int spin, int kind) const {
    return spin ? (kind ? b1 : b0) : (kind ? a1 : a0);
  }
};

__device__ __forceinline__ uint64_t mask_below(int p) { return p >= 64 ? ~0ull : (1ull << p) - 1ull; }

// The sample's masks (returned) and lists (written to LDS; lane p handles orbital p).
template <int NW>
__device__ __forceinline__ SpinMasks spin_lists(const uint64_t (&x)[NW], int n, int lane, SampleLists& c) {
  SpinMasks r;
  const bool in = lane < n;
  const bool oa = in && getbit<NW>(x, 2 * lane), ob = in && getbit<NW>(x, 2 * lane + 1);
  r.a0 = __ballot(oa);
  r.b0 = __ballot(ob);
  const uint64_t all = n >= 64 ? ~0ull : (1ull << n) - 1ull;
  r.a1 = all & ~r.a0;
  r.b1 = all & ~r.b0;
  const uint64_t below = mask_below(lane);
  const int ia = __popcll(r.a0 & below), ib = __popcll(r.b0 & below);
  if (in) {
    const int pa = (ia + ib) & 1, pb = pa ^ (oa ? 1 : 0);
    c.e[oa ? ia : 2 * kMaxOrb + lane - ia] = (uint8_t)(lane | pa << 7);
    c.e[kMaxOrb + (ob ? ib : 2 * kMaxOrb + lane - ib)] = (uint8_t)(lane | pb << 7);
  }
  return r;
}

// Parent of rank r: c2 (c2 - 1) / 2 + c1, c1 < c2.
__device__ __forceinline__ void unrank_parent(uint32_t r, int& c1, int& c2) {
  int c = (int)((1.f + sqrtf(1.f + 8.f * (float)r)) * 0.5f);
  c -= (uint32_t)(c * (c - 1) / 2) > r;
  c += (uint32_t)((c + 1) * c / 2) <= r;
  c2 = c;
  c1 = (int)r - c * (c - 1) / 2;
}

// One lane's segment: the suffixes of two lists above c2, and what its entries share.
struct Segment {
  uint64_t mu, mv;       // the lists' orbitals (0: no entries)
  int iu, iv;            // first index of the suffix
  int lu, lv;            // first entry of the lists
  int pair;              // both lists are one: its pairs
  uint32_t sel, fix;     // as in Rect (without triangle and entries per row)
};

// Segment `half` (0: A, 1: B) of parent (c1, c2) with kinds k1, k2 (1: occupied in x);
// `tp`: the parent's place in its tile.
template <int NW>
__device__ __forceinline__ Segment make_segment(const uint64_t (&x)[NW], const SpinMasks& m, int c1, int c2, int k1,
                                                int k2, int half, int tp, bool valid) {
  Segment s;
  const int s1 = c1 & 1, s2 = c2 & 1;
  int su, ku, sv, kv;   // spin and kind (0 occupied, 1 virtual) of the two lists
  // roles as byte selectors: 0 = c1, 1 = c2, 2 = u, 3 = v
  int ri, rj, ra, rb;
  bool any = valid;
  s.pair = 0;
  if (s1 != s2) {
    // each spin: one change by the parent, the opposite one by the entry
    const int ca = s1, cb = 1 - s1;   // which of c1 (0), c2 (1) is the alpha (beta) change
    const int ka = ca ? k2 : k1, kb = cb ? k2 : k1;
    su = 0; ku = ka;    // an occupied one was removed -> a virtual one is needed
    sv = 1; kv = kb;
    ri = ka ? ca : 2; ra = ka ? 2 : ca;
    rj = kb ? cb : 3; rb = kb ? 3 : cb;
    any = any && half == 0;
  } else if (k1 == k2) {
    s.pair = 1;
    su = sv = s1; ku = kv = k1;
    ri = k1 ? 0 : 2; rj = k1 ? 1 : 3;
    ra = k1 ? 2 : 0; rb = k1 ? 3 : 1;
    any = any && half == 0;
  } else {
    su = sv = half == 0 ? s1 : 1 - s1;
    ku = 0; kv = 1;
    const int og = k1 ? 0 : 1, vg = 1 - og;
    const bool swap = half == 1 && s1 == 1;   // alpha first
    ri = swap ? 2 : og; ra = swap ? 3 : vg;
    rj = swap ? og : 2; rb = swap ? vg : 3;
  }
  const bool same = s1 == s2 && half == 0;
  s.mu = any ? m.get(su, ku) : 0ull;
  s.mv = any ? m.get(sv, kv) : 0ull;
  // spin-orbitals above c2
  s.iu = __popcll(s.mu & mask_below(((c2 - su) >> 1) + 1));
  s.iv = __popcll(s.mv & mask_below(((c2 - sv) >> 1) + 1));
  s.lu = kMaxOrb * (2 * ku + su);
  s.lv = kMaxOrb * (2 * kv + sv);
  s.sel = (uint32_t)(ri | rj << 8 | ra << 16 | rb << 24);
  // Sign of a+_a a+_b a_j a_i: the occupation parities below the four spin-orbitals, and for
  // every two of them, f applied before g, one more if f < g. With c1 < c2 < u, v only the
  // order of u and v is open. pos[r]: when the spin-orbital of selector r is applied.
  int pos = 0;   // 4 bits each
  pos |= 0 << (4 * ri) | 1 << (4 * rj) | 2 << (4 * rb) | 3 << (4 * ra);
  const int t0 = pos & 15, t1 = (pos >> 4) & 15, t2 = (pos >> 8) & 15, t3 = (pos >> 12) & 15;
  int sg = (t0 < t1) + (t0 < t2) + (t0 < t3) + (t1 < t2) + (t1 < t3);
  sg += parity_below<NW>(x, c1) + parity_below<NW>(x, c2);
  const int uv = t2 < t3;   // [u < v] adds to the sign, else [v < u] = 1 - [u < v]
  sg += 1 - uv;
  s.fix = (uint32_t)((c1 >> 1) | (c2 >> 1) << 6 | tp << 12 | (sg & 1) << 16 | (same ? 1 : 0) << 18 | su << 20 | sv << 21);
  return s;
}

// Posts the rectangles of the entries whose smaller new orbital lies in [q0, q1) and returns
// their number. Lane r * 32 + half * 16 + parent posts rectangle r of its segment: with
// suffix starts u0, v0 (at q0) and u1, v1 (at q1) the entries are u in [u0, u1), v >= v0 and
// u >= u1, v in [v0, v1); of pairs, u in [u0, u1), v >= u1 and the triangle u < v in [u0, u1).
__device__ __forceinline__ uint32_t post_class(PrefixWave& pw, const Segment& s, int q0, int q1, int lane) {
  const uint64_t m0 = mask_below(q0), m1 = mask_below(q1);
  const int u0 = max(s.iu, (int)__popcll(s.mu & m0)), u1 = max(s.iu, (int)__popcll(s.mu & m1));
  const int v0 = max(s.iv, (int)__popcll(s.mv & m0)), v1 = max(s.iv, (int)__popcll(s.mv & m1));
  const int nu = __popcll(s.mu), nv = __popcll(s.mv);
  const bool second = lane >= 32, tri = second && s.pair;
  const int bu = second && !s.pair ? u1 : u0, bv = !second && s.pair ? u1 : second && s.pair ? u0 : v0;
  const int rows = second && !s.pair ? nu - u1 : u1 - u0;
  const int cols = second ? (s.pair ? 0 : v1 - v0) : nv - bv;
  const uint32_t own = tri ? (uint32_t)(rows * (rows - 1) / 2) : (uint32_t)(rows * cols);
  uint32_t v = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t u = __shfl_up(v, off);
    if (lane >= off) v += u;
  }
  pw.end[lane] = v;
  pw.rect[lane] = Rect{(uint32_t)((s.lu + bu) | (s.lv + bv) << 16), s.sel,
                       s.fix | (uint32_t)(tri ? 1 : 0) << 19 | (uint32_t)max(cols, 1) << 24, v - own};
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Entry t of the posted class: x', H_{x x'}, its parent's place in the tile, the orbitals of
// c1 and of the lower of its two new changes.
template <int NW>
struct PrefixEntry {
  uint64_t x[NW];
  double h;
  int parent, p0, p2;
};

template <int NW>
__device__ __forceinline__ PrefixEntry<NW> prefix_entry(const SysDev& S, const PrefixWave& pw, uint32_t t) {
  int s = 0;
#pragma unroll
  for (int step = 32; step >= 1; step >>= 1)
    if (pw.end[s + step - 1] <= t) s += step;
  const Rect d = pw.rect[s];
  const int w = (int)(t - d.start), cols = (int)(d.fix >> 24);
  int q = (int)((float)w * __builtin_amdgcn_rcpf((float)cols));
  int r = w - q * cols;
  q -= r < 0; r += r < 0 ? cols : 0;
  q += r >= cols; r -= r >= cols ? cols : 0;
  if ((d.fix >> 19) & 1) unrank_parent((uint32_t)w, q, r);   // pairs q < r, rank r (r - 1) / 2 + q
  const uint32_t eu = pw.c.e[(d.lists & 0xFFFFu) + (uint32_t)q], ev = pw.c.e[(d.lists >> 16) + (uint32_t)r];
  const int pu = eu & 63, pv = ev & 63, p1 = d.fix & 63, p2 = (d.fix >> 6) & 63;
  const int U = 2 * pu + (int)((d.fix >> 20) & 1), V = 2 * pv + (int)((d.fix >> 21) & 1);
  PrefixEntry<NW> e;
  e.parent = (d.fix >> 12) & 15;
  e.p0 = p1;
  e.p2 = min(pu, pv);
#pragma unroll
  for (int k = 0; k < NW; ++k) e.x[k] = pw.xg[e.parent][k];
  flip<NW>(e.x, U);
  flip<NW>(e.x, V);
  const uint32_t roles = __builtin_amdgcn_perm(0u, (uint32_t)(p1 | p2 << 8 | pu << 16 | pv << 24), d.sel);
  const uint32_t n = (uint32_t)S.n, i = roles & 0xFFu, j = (roles >> 8) & 0xFFu, a = (roles >> 16) & 0xFFu,
                 b = roles >> 24;
  const uint32_t ab = a * n + b, nn = n * n;
  double h = S.S[(i * n + j) * nn + ab];
  if ((d.fix >> 18) & 1) h -= S.S[(j * n + i) * nn + ab];
  const uint32_t neg = (eu >> 7) ^ (ev >> 7) ^ (d.fix >> 16) ^ (U < V ? 1u : 0u);
  e.h = (neg & 1u) ? -h : h;
  return e;
}

// The single excitation that parent (c1, c2) is, if its spins agree and its kinds differ.
__device__ __forceinline__ bool parent_single(const SysDev& S, const SpinMasks& m, int c1, int c2, int k1, int k2,
                                              Excitation& e) {
  e.kind = KIND_SINGLE;
  e.spin = c1 & 1;
  e.i = (k1 ? c1 : c2) >> 1;
  e.a = (k1 ? c2 : c1) >> 1;
  e.j = e.b = e.J = e.Bq = -1;
  e.I = 2 * e.i + e.spin;
  e.A = 2 * e.a + e.spin;
  const uint64_t mo = m.get(e.spin, 0), mv = m.get(e.spin, 1);
  const int qi = __popcll(mo & mask_below(e.i)), qa = __popcll(mv & mask_below(e.a));
  e.sidx = (uint32_t)((e.spin ? (int)S.nSa : 0) + qi * (e.spin ? S.vb : S.va) + qa);
  return ((c1 ^ c2) & 1) == 0 && k1 != k2;
}

}  // namespace elocal
