// Prefix-shared local energies of the two-term BF16 mode (the scheme is in prefix.hpp; the
// network, its packing and its precision are those of made_bf16.hip). One translation unit
// per kernel class instantiates it.
#pragma once
#include <algorithm>
#include <type_traits>

#include "elocal_internal.hpp"
#include "kernels.hpp"
#include "made_bf16.hpp"
#include "prefix.hpp"
#include "prefix_eval.hpp"

namespace elocal {

// Packed weight fragments: through a buffer resource (the lane's offset in one register, the
// fragment's a scalar: no address arithmetic per load) or from LDS.
struct WeightsGlobal {
  static constexpr bool kLds = false;
  __amdgpu_buffer_rsrc_t r;
  uint32_t voff;   // 16 * lane
  // fragment f + k (k known at compile time: in the instruction's 12-bit offset)
  __device__ __forceinline__ h16x8 operator()(int f, int k) const {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, voff + (uint32_t)(k & 3) * 1024u,
                                                         (uint32_t)(f + (k & ~3)) * 1024u, 0);
    h16x8 w;
    __builtin_memcpy(&w, &v, 16);
    return w;
  }
};
struct WeightsLds {
  static constexpr bool kLds = true;
  const h16x8* p;   // the lane's place in fragment 0
  int kb0, kin0;    // first input block held (of layer 0)
  __device__ __forceinline__ h16x8 operator()(int f, int k) const { return p[(f + k) * 64]; }
};

// Checkpoints of one wave.
struct Checkpoints {
  __amdgpu_buffer_rsrc_t r;
  // slot + k (k known at compile time)
  __device__ __forceinline__ f32x4 load(uint32_t voff, uint32_t slot, int k) const {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, voff + (uint32_t)k * 64u, slot * 64u, 0);
    f32x4 a;
    __builtin_memcpy(&a, &v, 16);
    return a;
  }
  __device__ __forceinline__ void store(const f32x4& a, uint32_t voff, uint32_t slot) const {
    decltype(__builtin_amdgcn_raw_buffer_load_b128(r, 0, 0, 0)) v;
    __builtin_memcpy(&v, &a, 16);
    __builtin_amdgcn_raw_buffer_store_b128(v, r, voff, slot * 64u, 0);
  }
};

__device__ __forceinline__ int ke_of(uint64_t ke, int ob) { return (int)((ke >> (4 * ob)) & 15u); }

// Network on NC 16-row tiles (tile c: row r of lane r) from class b = nblk - NB on, and
// epi(ob, a[NC]) for the output blocks ob >= ob_first, after pre() (row state that only the
// epilogue needs). Accumulators start from the rows' checkpoints (byte offset cko[c] of the
// row's 16 B of this lane group). BASE: whole rows (b = 0, NB = nblk), accumulators start
// from the biases, and the checkpoints of the boundaries >= bst are stored by the lanes with
// st_ok.
//
// A pass is a short chain of dependent layers, so what bounds it is the latency of the loads
// between them, not their bandwidth: every load is issued one step ahead of its use (the next
// pair's weights and the next layer's checkpoint before a pair is split into fp16 terms, the
// next output block's before an epilogue; with AHEAD also layer 1's checkpoint and the first
// output block's at the start of the pass), and the packing pads the k-ranges to ones known
// at compile time (layer 0: all input blocks; pair j of a hidden layer: j + 2 blocks for its
// second o-block, j + 1 + x for its first), so that no branch separates a load from its use.
template <int NB, int NT, int NC, int NW, bool BASE, bool AHEAD, class Weights, class Pre, class Epi>
__device__ __forceinline__ void net_rows(CArgs* args, const Weights& wt, const float* bias, const Checkpoints& ck,
                                         const uint64_t (&xr)[NC][NW], int lane, int b, const uint32_t (&cko)[NC],
                                         int ob_first, const uint64_t* xlut, int bst, bool st_ok, Pre&& pre,
                                         Epi&& epi) {
  CArgs* q = opaque(args);
  const int g = lane >> 4, L = q->made.L, x = q->px.extra;
  int kb0 = 0, kin0 = 0;
  if constexpr (Weights::kLds) { kb0 = wt.kb0; kin0 = wt.kin0; }
  h16x8 act[NT][NC][NB];
  f32x4 acc[NB][2][NC], nxt[AHEAD ? NB : 1][2][NC];
  h16x8 hw[2][NB], wo[NB];
  f32x4 no[NC];
  auto from_ck = [&](uint32_t slot, int k, f32x4 (&a)[NC]) {
#pragma unroll
    for (int c = 0; c < NC; ++c) a[c] = ck.load(cko[c], slot, k);
  };
  auto from_bias = [&](uint32_t row, f32x4 (&a)[NC]) {
    const f32x4 v = load_bias4(bias, row + 4 * g);
#pragma unroll
    for (int c = 0; c < NC; ++c) a[c] = v;
  };
  auto store = [&](uint32_t slot, const f32x4& a) {
    if (st_ok) ck.store(a, cko[0], slot);
  };
  const uint32_t soff = BASE ? 0u : q->px.cls[b].soff;
  const int nob = q->made.nob[L];
  int ob = sgpr(ob_first);
  int fo_out = (Weights::kLds ? q->px.tout[ob] : q->px.fout[ob]) + b - kb0;
  const uint32_t so_out = BASE ? 0u : q->px.cls[b].oslot, bb_out = q->px.lay[L].boff;
  auto load_out = [&](int o, int f) {
    if (BASE) from_bias(bb_out + 16 * o, no);
    else from_ck(so_out + o, 0, no);
#pragma unroll
    for (int kk = 0; kk < NB; ++kk) wo[kk] = wt(f, kk);   // (past the block's range: read, not used)
  };
  // weights of pair jj of hidden layer l (fo: fragment offset past its second o-block)
  auto load_pair = [&](int jj, int& fo) {
    const int c1 = min(b + jj + 2, b + NB) - kb0, c0 = min(b + jj + 1 + x, b + NB) - kb0;
    const int f1 = fo - c1, f0 = f1 - c0;
    fo = f0;
#pragma unroll
    for (int kk = 0; kk < NB; ++kk) {
      if (kk <= jj + 1) hw[1][kk] = wt(f1 + b - kb0, kk);
      if (kk <= jj) hw[0][kk] = wt(f0 + b - kb0, kk);
    }
    return f0 + b - kb0;
  };
  auto hidden_end = [&](int l) { return Weights::kLds ? q->px.lay[l].tend : q->px.lay[l].fend; };
  int fo = 0, f0 = 0;   // hidden layers: running fragment offset, the pair's first fragment
  // ---- layer 0: exact 0/1 inputs; every pair of blocks at once, one input block at a time
  {
    const int nk = q->made.nk[0], kin = BASE ? 0 : q->px.cls[b].kin;
    const int f = (Weights::kLds ? q->px.cls[b].t0 : q->px.cls[b].f0) - kin0;
    const uint32_t bb = q->px.lay[0].boff;
    h16x8 w0[NB][2], xin[NC];
    auto load_in = [&](int kb) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const uint32_t b8 = bits8_at<NW>(xr[c], 32 * kb + 8 * g);
        const uint64_t w2[2] = {xlut[b8 & 15u], xlut[b8 >> 4]};
        __builtin_memcpy(&xin[c], w2, 16);
      }
#pragma unroll
      for (int jj = 0; jj < NB; ++jj)
#pragma unroll
        for (int h = 0; h < 2; ++h) w0[jj][h] = wt(f + kb + (2 * jj + h) * (nk - kin0), 0);
    };
    load_in(kin);
#pragma unroll
    for (int jj = 0; jj < NB; ++jj)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (BASE) from_bias(bb + 32 * jj + 16 * h, acc[jj][h]);
        else from_ck(soff, 2 * jj + h, acc[jj][h]);
      }
    if constexpr (AHEAD) {
      if (L > 1) {
#pragma unroll
        for (int jj = NB - 1; jj >= 0; --jj)
#pragma unroll
          for (int h = 0; h < 2; ++h) from_ck(soff + 2 * NB, 2 * jj + h, nxt[jj][h]);
      }
      load_out(ob, fo_out);
    }
#pragma unroll 1
    for (int kb = kin;;) {
      if (BASE) {
        for (int bp = bst; bp < NB; ++bp)
          if (q->px.cls[bp].kin == kb) {
            const uint32_t sp = q->px.cls[bp].soff;
#pragma unroll
            for (int jj = 0; jj < NB; ++jj)
              if (jj >= bp) {
                store(sp + 2 * (jj - bp), acc[jj][0][0]);
                store(sp + 2 * (jj - bp) + 1, acc[jj][1][0]);
              }
          }
      }
#pragma unroll
      for (int jj = 0; jj < NB; ++jj)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int c = 0; c < NC; ++c) acc[jj][h][c] = mfma_f16(w0[jj][h], xin[c], acc[jj][h][c]);
      if (++kb >= nk) break;
      load_in(kb);
    }
    if (L > 1) {
      fo = hidden_end(1);
      f0 = load_pair(NB - 1, fo);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int jj = NB - 1; jj >= 0; --jj) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        h16x8 t[NT];
        split_relu<NT>(acc[jj][0][c], acc[jj][1][c], t);
#pragma unroll
        for (int i = 0; i < NT; ++i) act[i][c][jj] = t[i];
      }
      if (!BASE && !AHEAD) {
        if (L > 1) {
#pragma unroll
          for (int h = 0; h < 2; ++h) from_ck(soff + 2 * NB, 2 * jj + h, acc[jj][h]);
        }
      }
    }
  }
  auto& start = [&]() -> f32x4 (&)[NB][2][NC] {
    if constexpr (AHEAD) return nxt;
    else return acc;
  }();
  // ---- hidden layers 1..L-1 in place: pairs from the last to the first; pair jj reads
  // blocks up to jj + 1 (host-checked), so its result waits until pair jj - 1 is done
#pragma unroll 1
  for (int l = 1; l < L; ++l) {
    const uint32_t bb = q->px.lay[l].boff;
    // the next layer (the last hidden layer loads its own again)
    const int ln = min(l + 1, L - 1);
    const uint32_t so = soff + (uint32_t)(2 * NB * ln);
    f32x4 r0[NC], r1[NC];   // pair jj + 1's sums; its slot is free once pair jj is multiplied
    auto put = [&](int jj) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        h16x8 t[NT];
        split_relu<NT>(r0[c], r1[c], t);
#pragma unroll
        for (int i = 0; i < NT; ++i) act[i][c][jj] = t[i];
      }
    };
#pragma unroll
    for (int jj = NB - 1; jj >= 0; --jj) {
      f32x4 a0[NC], a1[NC];
      if (BASE) {
        from_bias(bb + 32 * jj, a0);
        from_bias(bb + 32 * jj + 16, a1);
      } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) { a0[c] = start[jj][0][c]; a1[c] = start[jj][1][c]; }
      }
#pragma unroll
      for (int kk = 0; kk <= jj + 1 && kk < NB; ++kk) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int i = 0; i < NT; ++i) a1[c] = mfma_f16(hw[1][kk], act[i][c][kk], a1[c]);
        if (kk <= jj) {
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int i = 0; i < NT; ++i) a0[c] = mfma_f16(hw[0][kk], act[i][c][kk], a0[c]);
        } else if (x) {
          const h16x8 w = wt(f0, kk);
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int i = 0; i < NT; ++i) a0[c] = mfma_f16(w, act[i][c][kk], a0[c]);
        }
        if (BASE && kk < jj && kk + 1 >= bst) {   // boundary kk + 1
          const uint32_t sp = q->px.cls[kk + 1].soff + (uint32_t)(2 * (NB - kk - 1) * l + 2 * (jj - kk - 1));
          store(sp, a0[0]);
          store(sp + 1, a1[0]);
        }
      }
      if (jj == 0) fo = hidden_end(ln);
      f0 = load_pair(jj == 0 ? NB - 1 : jj - 1, fo);
      if (!BASE) {
        from_ck(so, 2 * jj, start[jj][0]);
        from_ck(so, 2 * jj + 1, start[jj][1]);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (jj + 1 < NB) put(jj + 1 < NB ? jj + 1 : 0);
#pragma unroll
      for (int c = 0; c < NC; ++c) { r0[c] = a0[c]; r1[c] = a1[c]; }
    }
    put(0);
  }
  // ---- output layer
  if (!AHEAD) load_out(ob, fo_out);
  const uint64_t kes = q->px.lay[L].ke;
  pre();
#pragma unroll 1
  for (;;) {
    const int ke = ke_of(kes, ob);
    f32x4 a[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) a[c] = no[c];
#pragma unroll
    for (int kk = 0; kk < NB; ++kk) {
      if (b + kk >= ke) break;   // the k-range is a prefix (from class b on it may be empty)
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < NT; ++i) a[c] = mfma_f16(wo[kk], act[i][c][kk], a[c]);
      if (BASE && kk + 1 < NB && kk + 1 >= bst) {
        const int bp = kk + 1 < NB ? kk + 1 : 0;
        if (ob >= q->px.cls[bp].obq) store(q->px.cls[bp].oslot + (uint32_t)ob, a[0]);
      }
    }
    const int o = ob;
    if (ob + 1 < nob) {
      ++ob;
      fo_out += ke - kb0;
    }
    load_out(ob, fo_out);   // (after the last block: that block's again)
    __builtin_amdgcn_sched_barrier(0);
    epi(o, a);
    if (o + 1 >= nob) break;
  }
}

// 16-row tiles per network pass of NB blocks, and whether a pass loads layer 1's checkpoint at
// its start, in a kernel of CAP: 4 is built for 128 registers per lane, 8 for 256.
constexpr int prefix_cols(int nb, int cap) {
  return cap >= 8 ? (nb == 1 ? 4 : nb == 2 ? 2 : 1) : 1;
}
constexpr bool prefix_ahead(int nb, int cap) { return cap >= 8 ? nb <= 5 : nb <= 2; }

// The two-term BF16 network of kernel class HB with COLS tiles per pass.
template <int HB, int COLS, int LMODE>
struct NetBf16 {
  typedef float Real;
  typedef f32x4 Acc;
  static constexpr uint32_t kSlotBytes = 64;   // checkpoint of a 16-unit block of one row
  static constexpr int kCap = prefix_waves_bf16(32 * HB, COLS) == 16 ? 4 : 8;
  struct Sources {
    WeightsGlobal glob;
    WeightsLds ldsw;
    const float* bias;
    Checkpoints ck;
    const uint64_t* xlut;
  };
  static constexpr int cols(int nb) { return prefix_cols(nb, kCap); }
  static __device__ __forceinline__ double sample_lp(const PrefixArgs& P, int64_t i) { return (double)P.lpx[i]; }
  template <int NW>
  static __device__ __forceinline__ float step(RowCursor<NW>& rc, int ta, int tb, int na, int nb, const f32x4& z) {
    return cond_log2p_step<NW>(rc, ta, tb, na, nb, z);
  }
  static __device__ __forceinline__ double2 ratio(double hv, float zp, double sig_x, double dA) {
    return ratio_term(hv, zp, sig_x, dA);
  }
  template <int NB, int NC, int NW, bool BASE, class Pre, class Epi>
  static __device__ __forceinline__ void rows(CArgs* args, const Sources& src, const uint64_t (&xr)[NC][NW], int lane,
                                              int b, const uint32_t (&cko)[NC], int ob_first, int bst, bool st_ok,
                                              Pre&& pre, Epi&& epi) {
    constexpr bool AHEAD = !BASE && prefix_ahead(NB, kCap);
    constexpr bool IN_LDS = LMODE == 1 || (LMODE == 2 && !BASE && NB <= prefix_lds_blocks(32 * HB));
    if constexpr (IN_LDS)
      net_rows<NB, 2, NC, NW, BASE, AHEAD>(args, src.ldsw, src.bias, src.ck, xr, lane, b, cko, ob_first, src.xlut, bst,
                                           st_ok, pre, epi);
    else
      net_rows<NB, 2, NC, NW, BASE, AHEAD>(args, src.glob, src.bias, src.ck, xr, lane, b, cko, ob_first, src.xlut, bst,
                                           st_ok, pre, epi);
  }
};

// LMODE 2: copies the fragments of the last classes (input blocks >= bs, o-blocks that
// read them) to LDS. (Only the parents' passes read biases: those stay in global memory.)
__device__ __forceinline__ void stage_top(const PrefixArgs& P, unsigned char* smem) {
  const MadeDev& M = P.made;
  const PrefixTop& T = P.top;
  h16x8* sw = (h16x8*)smem;
  const h16x8* gw = (const h16x8*)M.wfrag;
  for (int l = 0; l <= M.L; ++l) {
    const int k0 = l == 0 ? T.kin0 : T.kb0;
    for (int ob = T.ob0[l]; ob < M.nob[l]; ++ob) {
      const int cnt = T.foff[l][ob + 1] - T.foff[l][ob];
      for (int i = threadIdx.x; i < cnt * 64; i += blockDim.x)
        sw[(size_t)T.foff[l][ob] * 64 + i] = gw[(size_t)(M.foff[l][ob] + k0) * 64 + i];
    }
  }
}

template <int LMODE>
__device__ __forceinline__ void stage_prefix(const PrefixArgs& P, unsigned char* smem) {
  if (LMODE == 1) stage_weights(P.made, P.lds_frag, smem, P.lds_bias_off);
  if (LMODE == 2) stage_top(P, smem);
}

// What a wave reads its weights, biases and checkpoints from.
template <int HB, int COLS, int LMODE>
__device__ __forceinline__ typename NetBf16<HB, COLS, LMODE>::Sources wave_sources(const PrefixArgs& P,
                                                                                 const unsigned char* smem, int wid,
                                                                                 int lane, const uint64_t* xlut) {
  typename NetBf16<HB, COLS, LMODE>::Sources s;
  s.xlut = xlut;
  s.glob = WeightsGlobal{buffer_of(P.made.wfrag, P.made.nfrag * 1024u), (uint32_t)lane * 16u};
  s.ldsw = WeightsLds{(const h16x8*)smem + lane, LMODE == 2 ? P.top.kb0 : 0, LMODE == 2 ? P.top.kin0 : 0};
  s.bias = LMODE == 1 ? (const float*)(smem + P.lds_bias_off) : (const float*)P.made.bias;
  // (made scalar explicitly: a resource in vector registers costs a loop around every access)
  const uint32_t wave = blockIdx.x * (blockDim.x >> 6) + (uint32_t)wid;
  const uint64_t base = (uint64_t)(P.px.scratch + (size_t)wave * P.px.stride);
  const uint64_t sbase = (uint64_t)(uint32_t)sgpr((int)(uint32_t)base) | (uint64_t)(uint32_t)sgpr((int)(base >> 32)) << 32;
  s.ck = Checkpoints{buffer_of((const void*)sbase, (uint32_t)sgpr((int)(P.px.stride * 4u)))};
  return s;
}

// One system: waves take work items from a queue (parents with early changes have far more
// entries than late ones) until it is empty.
template <int HB, int COLS, int NW, int LMODE>
__global__ void __launch_bounds__(64 * prefix_waves_bf16(32 * HB, COLS), 1) k_prefix_bf16(PrefixArgs P) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wid = sgpr(threadIdx.x >> 6);
  const uint64_t* xlut = fill_xlut(smem, P.lds_lut_off);
  stage_prefix<LMODE>(P, smem);
  __syncthreads();
  PrefixWave& pw = ((PrefixWave*)(smem + P.lds_ctx_off))[wid];
  CArgs* args = (CArgs*)__builtin_amdgcn_kernarg_segment_ptr();   // P, the only argument
  typedef NetBf16<HB, COLS, LMODE> Net;
  const typename Net::Sources src = wave_sources<HB, COLS, LMODE>(P, smem, wid, lane, xlut);
  PrefixSample<NW> st;
  st.b = -1;
  for (uint32_t t; next_ticket(P.px, lane, t);)
    run_item<Net, HB, HB / 2 + 1, NW>(P, args, src, pw, t, st, lane);
}

// Several systems in one persistent launch: every block goes through the systems in order
// (most expensive first), restaging its LDS weights, and its waves take items from the
// system's queue until that is empty. LDS offsets are those of system 0's arguments.
template <int HB, int COLS, int LMODE>
__global__ void __launch_bounds__(64 * prefix_waves_bf16(32 * HB, COLS), 1)
    k_prefix_multi_bf16(const PrefixArgs* __restrict__ args, int n_sys) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wid = sgpr(threadIdx.x >> 6);
  const uint64_t* xlut = fill_xlut(smem, args[0].lds_lut_off);
  PrefixWave& pw = ((PrefixWave*)(smem + args[0].lds_ctx_off))[wid];
  // A block starts with the system that its index gives it (shares by cost, see plan_multi) and
  // goes on to the next ones that have items left. All blocks in one system after the other
  // left the chip idle at each system's end: eight systems of 8 to 25 orbitals, 4 to 95 samples
  // 1017 us, 770 so; of 12 to 40, 256 to 347 samples 19.9 and 19.1 ms for the whole call.
  int s = 0;
  while (s + 1 < n_sys && blockIdx.x >= args[s + 1].px.block0) ++s;
  for (int i = 0; i < n_sys; ++i, s = s + 1 < n_sys ? s + 1 : 0) {
    const PrefixArgs& P = args[s];
    // (the barrier: every wave is done with the previous system's weights)
    const bool left = threadIdx.x == 0 && __hip_atomic_load(P.px.queue, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                                              P.px.tickets;
    if (!__syncthreads_or(left)) continue;
    stage_prefix<LMODE>(P, smem);
    __syncthreads();
    typedef NetBf16<HB, COLS, LMODE> Net;
    const typename Net::Sources src = wave_sources<HB, COLS, LMODE>(P, smem, wid, lane, xlut);
    // (two-word determinants for every system: a second copy of the code would cost more
    // registers than the empty second word)
    PrefixSample<2> st;
    st.b = -1;
    for (uint32_t t; next_ticket(P.px, lane, t);)
      run_item<Net, HB, 2, 2>(P, (CArgs*)(uintptr_t)&P, src, pw, t, st, lane);
  }
}

// ----------------------------------------------------------------------------- launchers
// lmode 0 or LM (the class's LDS mode).
template <int HB, int COLS, int LM>
static hipError_t launch_prefix_class(const PrefixArgs& A, int lmode, size_t lds, unsigned grid, int waves,
                                      hipStream_t st) {
  auto go = [&](auto kern) {
    const hipError_t e = allow_lds(kern, lds);
    if (e != hipSuccess) return e;
    const int w = std::max(1, std::min(waves, prefix_waves_bf16(32 * HB, COLS)));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * w), lds, st, A);
    return hipGetLastError();
  };
  if (lmode)
    return A.sys.W == 1 ? go(k_prefix_bf16<HB, COLS, 1, LM>) : go(k_prefix_bf16<HB, COLS, 2, LM>);
  return A.sys.W == 1 ? go(k_prefix_bf16<HB, COLS, 1, 0>) : go(k_prefix_bf16<HB, COLS, 2, 0>);
}

template <int HB, int COLS, int LM>
static hipError_t launch_prefix_multi_class(const PrefixArgs* args, int n_sys, int lmode, size_t lds, unsigned grid,
                                            int waves, hipStream_t st) {
  auto kern = lmode ? k_prefix_multi_bf16<HB, COLS, LM> : k_prefix_multi_bf16<HB, COLS, 0>;
  const hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  const int w = std::max(1, std::min(waves, prefix_waves_bf16(32 * HB, COLS)));
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * w), lds, st, args, n_sys);
  return hipGetLastError();
}

#define ELOCAL_PREFIX_CLASS(name, HB, COLS, LM)                                                                     \
  hipError_t launch_prefix_##name(const PrefixArgs& A, int lmode, size_t lds, unsigned grid, int waves,               \
                                  hipStream_t st) {                                                                 \
    return launch_prefix_class<HB, COLS, LM>(A, lmode, lds, grid, waves, st);                                        \
  }                                                                                                                 \
  hipError_t launch_prefix_multi_##name(const PrefixArgs* args, int n_sys, int lmode, size_t lds, unsigned grid,      \
                                        int waves, hipStream_t st) {                                                \
    return launch_prefix_multi_class<HB, COLS, LM>(args, n_sys, lmode, lds, grid, waves, st);                        \
  }

}  // namespace elocal
