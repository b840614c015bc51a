// Prefix-shared local energies of the all-FP64 mode (the scheme is in prefix.hpp; the network
// is that of made_f64.hip).
//
// A 16-row tile of the whole network is bound by the FP64 matrix cores (32 cycles per
// 16x16x4 product, 1,970 products at 60 orbitals, 3 x 256), so the products that sharing
// removes are the gain. Classes are those of the BF16 kernels (32 units, two o-blocks). Up to
// three blocks a pass takes two tiles: each weight fragment then feeds twice the rows (one
// tile's weights alone would take the whole 64 B per cycle of a CU's vector memory path at
// the matrix cores' rate) and four product chains are in flight.
//
// Packing: fragment (ob, kb) holds the 16 x 16 block of o-block ob and input block kb, lane
// (g, rho) the four k-steps of its row: 32 B, two vector loads. Input block kb of layer 0 is
// input bits 16 kb .. 16 kb + 15. The output layer has 4(n - 1) logits and the phase row.
#include <algorithm>

#include "made_f64.hpp"
#include "prefix_eval.hpp"

namespace elocal {

__global__ void k_pack_prefix_f64(MadeDev M, ThetaLayout T, const double* __restrict__ theta, double* __restrict__ frag,
                                  double* __restrict__ bias, uint32_t* __restrict__ queue) {
  const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
  const int n = M.n, L = M.L, nm1 = n - 1;
  if (gid == 0) *queue = 0u;
  if (gid < M.nfrag * 64u) {
    const uint32_t f = gid >> 6;
    const int lane = gid & 63, rho = lane & 15, g = lane >> 4;
    int l = 0;
    while (l < L && f >= M.woff[l + 1]) ++l;
    const uint32_t local = f - M.woff[l];
    const int ob = local / M.nk[l], kb = local % M.nk[l];
    // the FP64 product returns row 4 i + lane / 16 of the block in register i
    const int opos = 16 * ob + 4 * (rho & 3) + (rho >> 2);
    const int o = opos >= M.nout[l] ? -1 : l < L ? sorted_unit(n, M.nout[l], opos) : opos;
    double v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int kpos = l == 0 ? 16 * kb + 4 * i + g : 16 * kb + 4 * g + i;
      const int k = kpos >= M.nin[l] ? -1 : l > 0 ? sorted_unit(n, M.nin[l], kpos) : kpos;
      bool ok = o >= 0 && k >= 0;
      const bool phase = l == L && o == 4 * nm1;
      if (l == 0) ok = ok && (o % nm1) + 1 >= k / 2 + 1;
      else if (l < L) ok = ok && (o % nm1) >= (k % nm1);
      else ok = ok && (phase || (o / 4) + 1 > (k % nm1) + 1);
      v[i] = !ok ? 0.0 : phase ? theta[T.offwphi + k] : theta[T.offW[l] + (uint32_t)o * M.nin[l] + k];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) frag[(size_t)gid * 4 + i] = v[i];
  }
  if (gid < M.nbias) {
    int l = 0;
    while (l < L && gid >= M.boff[l + 1]) ++l;
    const int opos = gid - M.boff[l];
    double v = 0.0;
    if (opos < M.nout[l]) {
      const int o = l < L ? sorted_unit(n, M.nout[l], opos) : opos;
      v = l == L && o == 4 * nm1 ? theta[T.offbphi] : theta[T.offb[l] + o];
    }
    bias[gid] = v;
  }
}

struct NetF64 {
  typedef double Real;
  typedef f64x4 Acc;
  static constexpr uint32_t kSlotBytes = 128;
  struct Sources {
    __amdgpu_buffer_rsrc_t w, bias, ck;
  };
  static constexpr int cols(int nb) { return nb <= 2 ? 2 : 1; }
  static __device__ __forceinline__ double sample_lp(const PrefixArgs& P, int64_t i) { return P.lpx64[i]; }
  static __device__ __forceinline__ double2 ratio(double hv, double zp, double sig_x, double dA) {
    return ratio_term64(hv, zp, sig_x, dA);
  }

  template <int NW>
  static __device__ __forceinline__ double step(RowCursor<NW>& rc, int ta, int tb, int na, int nb, const f64x4& z) {
    return cond_step64<NW>(rc, ta, tb, na, nb, z);
  }

  static __device__ __forceinline__ f64x4 load32(const __amdgpu_buffer_rsrc_t& r, uint32_t voff, uint32_t soff) {
    const auto lo = __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0);
    const auto hi = __builtin_amdgcn_raw_buffer_load_b128(r, voff + 16u, soff, 0);
    double d[4];
    __builtin_memcpy(d, &lo, 16);
    __builtin_memcpy(d + 2, &hi, 16);
    return f64x4{d[0], d[1], d[2], d[3]};
  }
  static __device__ __forceinline__ void store32(const __amdgpu_buffer_rsrc_t& r, const f64x4& a, uint32_t voff,
                                                 uint32_t soff) {
    double d[4] = {a[0], a[1], a[2], a[3]};
    decltype(__builtin_amdgcn_raw_buffer_load_b128(r, 0, 0, 0)) lo, hi;
    __builtin_memcpy(&lo, d, 16);
    __builtin_memcpy(&hi, d + 2, 16);
    __builtin_amdgcn_raw_buffer_store_b128(lo, r, voff, soff, 0);
    __builtin_amdgcn_raw_buffer_store_b128(hi, r, voff + 16u, soff, 0);
  }

  // One pass (see net_rows in prefix_bf16.hpp): rows of class b = nblk - NB, or with BASE
  // whole rows whose checkpoints are stored.
  template <int NB, int NC, int NW, bool BASE, class Pre, class Epi>
  static __device__ __forceinline__ void rows(CArgs* args, const Sources& src, const uint64_t (&xr)[NC][NW], int lane,
                                              int b, const uint32_t (&cko)[NC], int ob_first, int bst, bool st_ok,
                                              Pre&& pre, Epi&& epi) {
    CArgs* q = opaque(args);
    const int g = lane >> 4, L = q->made.L;
    const uint32_t wv = 32u * (uint32_t)lane, bv = 32u * (uint32_t)g;
    f64x4 cur[NC][2 * NB];
    auto frag = [&](int f) { return load32(src.w, wv, (uint32_t)f * 2048u); };
    auto start = [&](uint32_t slot, int k, uint32_t row, f64x4 (&a)[NC]) {
      if (BASE) {
        const f64x4 v = load32(src.bias, bv, row * 8u);
#pragma unroll
        for (int c = 0; c < NC; ++c) a[c] = v;
      } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) a[c] = load32(src.ck, cko[c] + 128u * (uint32_t)k, slot * 128u);
      }
    };
    auto store = [&](uint32_t slot, const f64x4& a) {
      if (st_ok) store32(src.ck, a, cko[0], slot * 128u);
    };
    auto mul = [&](f64x4& a, const f64x4& w, const f64x4& x) {
#pragma unroll
      for (int i = 0; i < 4; ++i) a = __builtin_amdgcn_mfma_f64_16x16x4f64(w[i], x[i], a, 0, 0, 0);
    };
    auto relu = [](const f64x4& a) {
      f64x4 r;
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = a[i] > 0.0 ? a[i] : 0.0;
      return r;
    };
    const uint32_t soff = BASE ? 0u : q->px.cls[b].soff;
    // ---- layer 0: exact 0/1 inputs
    {
      const int nk = q->made.nk[0], kin = BASE ? 0 : q->px.cls[b].kin;
      const uint64_t kes = q->px.lay[0].ke;
      const uint32_t bb = q->px.lay[0].boff;
#pragma unroll
      for (int jj = 0; jj < NB; ++jj) {
        const int f0 = q->px.cls[b].f0 + 2 * jj * nk, f1 = f0 + nk;
        const int ke = 1 + (int)((kes >> (4 * (2 * (b + jj) + 1))) & 15u);   // both blocks of the pair
        f64x4 a0[NC], a1[NC];
        start(soff, 2 * jj, bb + 32 * jj, a0);
        start(soff, 2 * jj + 1, bb + 32 * jj + 16, a1);
        f64x4 w0 = frag(f0 + kin), w1 = frag(f1 + kin);
        auto boundary = [&](int kb) {
          if (BASE)
            for (int bp = bst; bp <= jj; ++bp)
              if (q->px.cls[bp].kin == kb) {
                const uint32_t sp = q->px.cls[bp].soff + (uint32_t)(2 * (jj - bp));
                store(sp, a0[0]);
                store(sp + 1, a1[0]);
              }
        };
#pragma unroll 1
        for (int kb = kin; kb < ke; ++kb) {
          boundary(kb);
          const f64x4 v0 = w0, v1 = w1;
          w0 = frag(f0 + kb + 1);   // (past the pair's range: read, not used)
          w1 = frag(f1 + kb + 1);
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            f64x4 xb;
#pragma unroll
            for (int i = 0; i < 4; ++i) xb[i] = (double)getbit<NW>(xr[c], 16 * kb + 4 * i + g);
            mul(a0[c], v0, xb);
            mul(a1[c], v1, xb);
          }
        }
        boundary(ke);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          cur[c][2 * jj] = relu(a0[c]);
          cur[c][2 * jj + 1] = relu(a1[c]);
        }
      }
    }
    // ---- hidden layers in place: pairs from the last to the first; o-block ob reads input
    // blocks up to ob + 1 (host-checked), so a pair's sums wait until the pair below is done
#pragma unroll 1
    for (int l = 1; l < L; ++l) {
      const uint64_t kes = q->px.lay[l].ke;
      const uint32_t bb = q->px.lay[l].boff, so = soff + (uint32_t)(2 * NB * l);
      const int nk = q->made.nk[l], fl = q->px.lay[l].fend + 2 * b * nk + 2 * b;
      // the next pair's start is loaded ahead where registers are left for it
      constexpr bool AHEAD = NB * NC <= 5;
      f64x4 r0[NC], r1[NC], n0[NC], n1[NC];
      if (AHEAD) {
        start(so, 2 * NB - 2, bb + 32 * (NB - 1), n0);
        start(so, 2 * NB - 1, bb + 32 * (NB - 1) + 16, n1);
      }
      f64x4 w0 = frag(fl + 2 * (NB - 1) * nk), w1 = frag(fl + (2 * NB - 1) * nk);
#pragma unroll
      for (int jj = NB - 1; jj >= 0; --jj) {
        const int f0 = fl + 2 * jj * nk, f1 = f0 + nk, ob = 2 * (b + jj);
        const int e0 = 1 + (int)((kes >> (4 * ob)) & 15u) - 2 * b, e1 = 1 + (int)((kes >> (4 * ob + 4)) & 15u) - 2 * b;
        f64x4 a0[NC], a1[NC];
        if (!AHEAD) {
          start(so, 2 * jj, bb + 32 * jj, a0);
          start(so, 2 * jj + 1, bb + 32 * jj + 16, a1);
        } else {
#pragma unroll
          for (int c = 0; c < NC; ++c) { a0[c] = n0[c]; a1[c] = n1[c]; }
        }
        if (AHEAD && jj > 0) {
          start(so, 2 * jj - 2, bb + 32 * (jj - 1), n0);
          start(so, 2 * jj - 1, bb + 32 * (jj - 1) + 16, n1);
        }
#pragma unroll
        for (int kb = 0; kb <= 2 * jj + 2 && kb < 2 * NB; ++kb) {
          // block 0 reads 2 jj + 1 or + 2 blocks, block 1 one more of each
          const bool need0 = kb <= 2 * jj || (kb == 2 * jj + 1 && kb < e0), need1 = kb <= 2 * jj + 1 || kb < e1;
          const f64x4 v0 = w0, v1 = w1;
          const bool last = kb == 2 * jj + 2 || kb == 2 * NB - 1;
          if (!last) {
            if (kb <= 2 * jj) w0 = frag(f0 + kb + 1);
            w1 = frag(f1 + kb + 1);
          } else if (jj > 0) {
            w0 = frag(f0 - 2 * nk);
            w1 = frag(f1 - 2 * nk);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            if (need1) mul(a1[c], v1, cur[c][kb]);
            if (kb <= 2 * jj + 1 && need0) mul(a0[c], v0, cur[c][kb]);
          }
          if (BASE && (kb & 1) && (kb + 1) / 2 <= jj && (kb + 1) / 2 >= bst) {
            const int bp = (kb + 1) / 2;
            const uint32_t sp = q->px.cls[bp].soff + (uint32_t)(2 * (NB - bp) * l + 2 * (jj - bp));
            store(sp, a0[0]);
            store(sp + 1, a1[0]);
          }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          if (jj + 1 < NB) {
            cur[c][jj + 1 < NB ? 2 * (jj + 1) : 0] = relu(r0[c]);
            cur[c][jj + 1 < NB ? 2 * (jj + 1) + 1 : 0] = relu(r1[c]);
          }
          r0[c] = a0[c];
          r1[c] = a1[c];
        }
      }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        cur[c][0] = relu(r0[c]);
        cur[c][1] = relu(r1[c]);
      }
    }
    // ---- output layer
    {
      const uint64_t kes = q->px.lay[L].ke;
      const uint32_t bb = q->px.lay[L].boff, so = BASE ? 0u : q->px.cls[b].oslot;
      const int nk = q->made.nk[L], nob = q->made.nob[L], fl = q->px.lay[L].fend + 2 * b;
      int ob = sgpr(ob_first);
      f64x4 no[NC];
      start(so + ob, 0, bb + 16 * ob, no);
      f64x4 w = frag(fl + ob * nk);
      pre();
#pragma unroll 1
      for (;;) {
        const int e = 1 + (int)((kes >> (4 * ob)) & 15u) - 2 * b;
        f64x4 a[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) a[c] = no[c];
#pragma unroll
        for (int kb = 0; kb < 2 * NB; ++kb) {
          if (kb >= e) break;   // (from class b on the range may be empty)
          const f64x4 v = w;
          w = frag(fl + ob * nk + kb + 1);
#pragma unroll
          for (int c = 0; c < NC; ++c) mul(a[c], v, cur[c][kb]);
          if (BASE && (kb & 1) && (kb + 1) / 2 < NB && (kb + 1) / 2 >= bst) {
            const int bp = (kb + 1) / 2;
            if (ob >= q->px.cls[bp].obq) store(q->px.cls[bp].oslot + (uint32_t)ob, a[0]);
          }
        }
        const int o = ob;
        if (ob + 1 < nob) ++ob;
        start(so + ob, 0, bb + 16 * ob, no);   // (after the last block: that block's again)
        w = frag(fl + ob * nk);
        __builtin_amdgcn_sched_barrier(0);
        epi(o, a);
        if (o + 1 >= nob) break;
      }
    }
  }
};

__device__ __forceinline__ NetF64::Sources wave_sources_f64(const PrefixArgs& P, int wid) {
  const uint32_t wave = blockIdx.x * (blockDim.x >> 6) + (uint32_t)wid;
  const uint64_t base = (uint64_t)(P.px.scratch + (size_t)wave * P.px.stride);
  const uint64_t sbase = (uint64_t)(uint32_t)sgpr((int)(uint32_t)base) | (uint64_t)(uint32_t)sgpr((int)(base >> 32)) << 32;
  return NetF64::Sources{buffer_of(P.made.wfrag, P.made.nfrag * 2048u), buffer_of(P.made.bias, P.made.nbias * 8u),
                         buffer_of((const void*)sbase, (uint32_t)sgpr((int)(P.px.stride * 4u)))};
}

// (see k_prefix_bf16)
template <int HB, int NW>
__global__ void __launch_bounds__(64 * kPrefixWavesF64, 1) k_prefix_f64(PrefixArgs P) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wid = sgpr(threadIdx.x >> 6);
  PrefixWave& pw = ((PrefixWave*)smem)[wid];
  CArgs* args = (CArgs*)__builtin_amdgcn_kernarg_segment_ptr();   // P, the only argument
  const NetF64::Sources src = wave_sources_f64(P, wid);
  PrefixSample<NW> st;
  st.b = -1;
  for (uint32_t t; next_ticket(P.px, lane, t);)
    run_item<NetF64, HB, HB / 2 + 1, NW>(P, args, src, pw, t, st, lane);
}

template <int HB>
__global__ void __launch_bounds__(64 * kPrefixWavesF64, 1)
    k_prefix_multi_f64(const PrefixArgs* __restrict__ args, int n_sys) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wid = sgpr(threadIdx.x >> 6);
  PrefixWave& pw = ((PrefixWave*)smem)[wid];
  // (a wave starts with its block's system and goes on to the others, see k_prefix_multi_bf16)
  int s = 0;
  while (s + 1 < n_sys && blockIdx.x >= args[s + 1].px.block0) ++s;
  for (int i = 0; i < n_sys; ++i, s = s + 1 < n_sys ? s + 1 : 0) {
    const PrefixArgs& P = args[s];
    const NetF64::Sources src = wave_sources_f64(P, wid);
    PrefixSample<2> st;
    st.b = -1;
    for (uint32_t t; next_ticket(P.px, lane, t);)
      run_item<NetF64, HB, 2, 2>(P, (CArgs*)(uintptr_t)&P, src, pw, t, st, lane);
  }
}

hipError_t launch_pack_prefix_f64(const MadeDev& M, const ThetaLayout& T, const double* theta, void* frag,
                                  double* bias, uint32_t* queue, hipStream_t st) {
  const uint32_t total = std::max(M.nfrag * 64u, M.nbias);
  hipLaunchKernelGGL(k_pack_prefix_f64, dim3((total + 255) / 256), dim3(256), 0, st, M, T, theta, (double*)frag, bias,
                     queue);
  return hipGetLastError();
}

hipError_t launch_prefix_f64(const PrefixArgs& A, int hmax, unsigned grid, hipStream_t st) {
  if (A.n_items <= 0) return hipSuccess;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kPrefixWavesF64), kPrefixWavesF64 * sizeof(PrefixWave), st, A);
    return hipGetLastError();
  };
  const bool one = A.sys.W == 1;
  if (hmax == 64) return one ? go(k_prefix_f64<2, 1>) : go(k_prefix_f64<2, 2>);
  if (hmax == 128) return one ? go(k_prefix_f64<4, 1>) : go(k_prefix_f64<4, 2>);
  return one ? go(k_prefix_f64<8, 1>) : go(k_prefix_f64<8, 2>);
}

hipError_t launch_prefix_multi_f64(const PrefixArgs* args, int n_sys, int hmax, unsigned grid, hipStream_t st) {
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kPrefixWavesF64), kPrefixWavesF64 * sizeof(PrefixWave), st, args,
                       n_sys);
    return hipGetLastError();
  };
  if (hmax == 64) return go(k_prefix_multi_f64<2>);
  if (hmax == 128) return go(k_prefix_multi_f64<4>);
  return go(k_prefix_multi_f64<8>);
}

}  // namespace elocal
