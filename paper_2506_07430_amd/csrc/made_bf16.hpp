// Device code shared by the BF16-mode kernels (made_bf16.hip, prefix_bf16.hip): operand
// conversion, matrix-core products, the log-softmax epilogue, the FP64 ratio and the LDS
// staging of packed weights.
#pragma once
#include "elocal_internal.hpp"
#include "kernels.hpp"

namespace elocal {

// Output layer of the BF16 packing: rows 4p..4p+3 hold the logits of orbital p < n - 1 and
// row 4(n - 1) the phase head. The last orbital needs no logits: with no orbital left after
// it exactly one occupation keeps both electron counts reachable, so its conditional is 1.
__device__ __forceinline__ int phase_row_bf16(int n) { return 4 * (n - 1); }

__device__ __forceinline__ h16x8 bits_to_h16x8(uint32_t v) {
  uint32_t w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    w[q] = (((v >> (2 * q)) & 1u) * 0x3C00u) | ((((v >> (2 * q + 1)) & 1u) * 0x3C00u) << 16);
  h16x8 r;
  __builtin_memcpy(&r, w, sizeof(r));
  return r;
}

typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));

// ReLU of a pair, then NT fp16 terms whose sum represents each value: t[0] = fp16(a),
// t[1] = fp16(a - t[0]), t[2] = fp16(a - t[0] - t[1]) (one packed convert for the first
// term of both values; each later term is one fused multiply-add with an fp16 operand
// that rounds straight to fp16, a - t[0] being exact in FP32). Two terms leave at most
// 2^-22 |a| for |a| >= 2^-3 and 2^-25 in absolute terms below (fp16 subnormals), three
// terms far less. Values must stay below 65504 (the fp16 range).
template <int NT>
__device__ __forceinline__ void split_pair(float u, float v, uint32_t (&t)[NT]) {
  u = __int_as_float(max(__float_as_int(u), 0));     // ReLU: negative floats are negative ints
  v = __int_as_float(max(__float_as_int(v), 0));
  // a 1.0 the optimiser cannot fold: fma(-t, one, a) then stays one mixed-precision FMA
  float one;
  asm("s_mov_b32 %0, 1.0" : "=s"(one));
  h16x2 h;
  h[0] = (_Float16)u;
  h[1] = (_Float16)v;
  uint32_t hb;
  __builtin_memcpy(&hb, &h, 4);
  // opaque to the optimiser: the residuals below read the packed value, not a second convert
  asm volatile("" : "+v"(hb));
  t[0] = hb;
  if (NT > 1) {
    h16x2 hh;
    __builtin_memcpy(&hh, &hb, 4);
    const float ru = __builtin_fmaf(-(float)hh[0], one, u);
    const float rv = __builtin_fmaf(-(float)hh[1], one, v);
    h16x2 l;
    l[0] = (_Float16)ru;
    l[1] = (_Float16)rv;
    uint32_t lb;
    __builtin_memcpy(&lb, &l, 4);
    t[1] = lb;
    if (NT > 2) {
      asm volatile("" : "+v"(lb));
      h16x2 ll;
      __builtin_memcpy(&ll, &lb, 4);
      const float su = __builtin_fmaf(-(float)ll[0], one, ru);
      const float sv = __builtin_fmaf(-(float)ll[1], one, rv);
      h16x2 m;
      m[0] = (_Float16)su;
      m[1] = (_Float16)sv;
      __builtin_memcpy(&t[NT > 2 ? 2 : 0], &m, 4);
    }
  }
}

// Units 4g..4g+3 of block a and of block a+1 -> the 8 k-slots of the next layer, as NT
// fp16 terms.
template <int NT>
__device__ __forceinline__ void split_relu(const f32x4& a, const f32x4& b, h16x8 (&out)[NT]) {
  uint32_t t[4][NT];
  split_pair<NT>(a[0], a[1], t[0]);
  split_pair<NT>(a[2], a[3], t[1]);
  split_pair<NT>(b[0], b[1], t[2]);
  split_pair<NT>(b[2], b[3], t[3]);
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const uint32_t w[4] = {t[0][i], t[1][i], t[2][i], t[3][i]};
    __builtin_memcpy(&out[i], w, 16);
  }
}

__device__ __forceinline__ int sgpr(int v) { return __builtin_amdgcn_readfirstlane(v); }

// k-range of o-block ob (wave-uniform) from the three packed words of its layer.
__device__ __forceinline__ int kend_packed(uint32_t k0, uint32_t k1, uint32_t k2, int ob) {
  const uint32_t w = ob < 8 ? k0 : ob < 16 ? k1 : k2;
  return (int)((w >> (4 * (ob & 7))) & 15u);
}

__device__ __forceinline__ f32x4 mfma_f16(const h16x8& a, const h16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 load_bias4(const float* bias, uint32_t off) {
  f32x4 r;
  r[0] = bias[off]; r[1] = bias[off + 1]; r[2] = bias[off + 2]; r[3] = bias[off + 3];
  return r;
}

// Per-row state of the epilogue at the lane's current orbital p: the row's occupation
// bits from orbital p on (bit 0 = alpha of p) and the electrons of each spin before p.
// Advanced by four orbitals per output block.
template <int NW>
struct RowCursor {
  uint64_t bits[NW];
  int cu, cd;
};

template <int NW>
__device__ __forceinline__ RowCursor<NW> cursor_at(const uint64_t (&x)[NW], int p) {
  RowCursor<NW> r;
  r.cu = count_spin_below<NW>(x, p, 0);
  r.cd = count_spin_below<NW>(x, p, 1);
  const int k = 2 * p;   // < 64 NW for every orbital the epilogue visits
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    uint64_t v = 0;
#pragma unroll
    for (int u = w; u < NW; ++u) {
      const int sh = 64 * (u - w) - k;   // bit i of word u lands at 64(u - w) + i - k
      if (sh >= 0 && sh < 64) v |= x[u] << sh;
      else if (sh < 0 && sh > -64) v |= x[u] >> (-sh);
    }
    r.bits[w] = v;
  }
  return r;
}

template <int NW>
__device__ __forceinline__ void cursor_advance4(RowCursor<NW>& r, uint32_t b8) {
  r.cu += __popc(b8 & 0x55u);
  r.cd += __popc(b8 & 0xAAu);
#pragma unroll
  for (int w = 0; w < NW; ++w) r.bits[w] = (r.bits[w] >> 8) | (w + 1 < NW ? r.bits[w + 1] << 56 : 0ull);
}

// By k < 4 orbitals.
template <int NW>
__device__ __forceinline__ void cursor_advance(RowCursor<NW>& r, int k) {
  const uint32_t low = (uint32_t)r.bits[0] & ((1u << (2 * k)) - 1u);
  r.cu += __popc(low & 0x55u);
  r.cd += __popc(low & 0xAAu);
#pragma unroll
  for (int w = 0; w < NW; ++w)
    r.bits[w] = (r.bits[w] >> (2 * k)) | (w + 1 < NW ? (r.bits[w + 1] << 1) << (63 - 2 * k) : 0ull);
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr double kLn2 = 0.6931471805599453094;

// log2 p_p(s_p) of the row at the cursor's orbital, then advance the cursor by four
// orbitals. The softmax runs over the occupations that keep both electron counts
// reachable: alpha must be taken if cu < ta (= n_alpha - orbitals after p), may be
// taken if cu < na (same for beta). Base 2 on the native exp2/log2 units (one rescale
// to natural log per row, by the caller), shifted by the taken occupation's logit:
// log2 p = -log2(sum over allowed s of 2^(y_s - y_taken)), where the taken term is 1, so
// the sum is >= 1; it overflows only when p is below 2^-128, and then gives -inf, the
// right limit for a ratio (that entry's amplitude is 0 to double precision).
template <int NW>
__device__ __forceinline__ float cond_log2p_step(RowCursor<NW>& rc, int ta, int tb, int na, int nb,
                                                 const f32x4& z) {
  const uint32_t b8 = (uint32_t)rc.bits[0] & 0xFFu;
  const bool a_must = rc.cu < ta, a_may = rc.cu < na;
  const bool b_must = rc.cd < tb, b_may = rc.cd < nb;
  const bool ok0 = !a_must && !b_must, ok1 = a_may && !b_must;
  const bool ok2 = !a_must && b_may, ok3 = a_may && b_may;
  // the taken logit in log2 units; each exponent is one fused multiply-add
  const float z01 = (b8 & 1u) ? z[1] : z[0];
  const float z23 = (b8 & 1u) ? z[3] : z[2];
  const float ys = ((b8 & 2u) ? z23 : z01) * kLog2e;
  const float e0 = ok0 ? __builtin_amdgcn_exp2f(__builtin_fmaf(z[0], kLog2e, -ys)) : 0.f;
  const float e1 = ok1 ? __builtin_amdgcn_exp2f(__builtin_fmaf(z[1], kLog2e, -ys)) : 0.f;
  const float e2 = ok2 ? __builtin_amdgcn_exp2f(__builtin_fmaf(z[2], kLog2e, -ys)) : 0.f;
  const float e3 = ok3 ? __builtin_amdgcn_exp2f(__builtin_fmaf(z[3], kLog2e, -ys)) : 0.f;
  const float sum = (e0 + e1) + (e2 + e3);
  cursor_advance4<NW>(rc, b8);
  return -__builtin_amdgcn_logf(sum);
}

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int row_min(int v) {   // least over the lane's 16-lane row
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) v = min(v, __shfl_xor(v, off));
  return v;
}

// H exp(dA ln2 / 2 + i 2 pi (sigmoid(zp) - sig_x)) in FP64. The phase difference 2 pi d has
// |d| < 1, so sincospi needs no large-argument reduction; the magnitude with dA in log2
// units is exp2(dA / 2). Not inlined (nor is the sample's sigmoid): inlined, the compiler
// keeps the constants of the FP64 functions in registers across the whole kernel, and at
// four waves per SIMD they spill to scratch memory.
static __device__ __attribute__((noinline)) double sigmoid64(double z) { return 1.0 / (1.0 + exp(-z)); }

static __device__ __attribute__((noinline)) double2 ratio_term(double hv, float zp, double sig_x, double dA) {
  const double d = 1.0 / (1.0 + exp(-(double)zp)) - sig_x;
  double sn, cs;
  sincospi(2.0 * d, &sn, &cs);
  const double mag = hv * exp2(0.5 * dA);
  return make_double2(mag * cs, mag * sn);
}

// Copies the packed weights of every staged layer (lds[l] >= 0: fragment offset in LDS)
// and the biases into LDS.
__device__ __forceinline__ void stage_weights(const MadeDev& M, const int32_t* lds, unsigned char* smem,
                                              uint32_t bias_off) {
  h16x8* sw = (h16x8*)smem;
  const h16x8* gw = (const h16x8*)M.wfrag;
  for (int l = 0; l <= M.L; ++l) {
    const int32_t lf = lds[l];
    if (lf < 0) continue;
    const uint32_t f0 = (uint32_t)M.foff[l][0], nf = (uint32_t)M.foff[l][M.nob[l]] - f0;
    for (uint32_t i = threadIdx.x; i < nf * 64u; i += blockDim.x) sw[(size_t)lf * 64 + i] = gw[(size_t)f0 * 64 + i];
  }
  float* sb = (float*)(smem + bias_off);
  const float* gb = (const float*)M.bias;
  for (uint32_t i = threadIdx.x; i < M.nbias; i += blockDim.x) sb[i] = gb[i];
}

// Fills the input-expansion table (every thread of the block takes part; the caller
// synchronises the block before the table is read): entry v (4 bits) holds the four fp16
// values bit j of v ? 1 : 0.
__device__ __forceinline__ uint64_t* fill_xlut(unsigned char* smem, uint32_t lut_off) {
  uint64_t* lut = (uint64_t*)(smem + lut_off);
  for (uint32_t v = threadIdx.x; v < 16u; v += blockDim.x) {
    uint64_t e = 0;
    for (int j = 0; j < 4; ++j) e |= (uint64_t)(((v >> j) & 1u) * 0x3C00u) << (16 * j);
    lut[v] = e;
  }
  return lut;
}

template <class K>
static hipError_t allow_lds(K kern, size_t lds) {
  if (lds <= 65536) return hipSuccess;
  return hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

}  // namespace elocal
