// H on full-sector vectors as matrix products over the two spins' strings.
//
// A determinant is a pair of strings (occupied orbitals of one spin) Ia, Ib, and a vector a
// matrix V[Ia][Ib]. With the orbitals ordered alpha first, H is
//   (H V)[Ia][Ib] = sum_Ja Ha[Ia][Ja] V[Ja][Ib] + sum_Jb Hb[Ib][Jb] V[Ia][Jb]
//                 + sum_{pq,rs} (pq|rs) <Ia|E_pq|Ja> <Ib|E_rs|Jb> V[Ja][Jb]:
// Ha and Hb (one-body part and same-spin repulsion) are sparse matrices over strings, tabled
// once per call, and the last sum is, for every Ia, a dense product of the integrals with the
// rows V[Ja] that one E_pq reaches, from which every Ib then gathers its E_rs:
//   W[rs][Jb] = sum_{pq} (pq|rs) <Ia|E_pq|Ja> V[Ja][Jb].
// The library orders spin-orbitals alpha and beta in turn; a vector in the order above is
// multiplied by (-1)^(pairs of an occupied alpha orbital p and a beta orbital below p).
//
// At (12, 6a, 6b), 853776 rows of 1819 entries, one product with H takes 0.42 ms (two
// sparse products of 115 us, the dense one with its gathers 179 us, which is 70 us of matrix
// instructions); from lists of entries (kpm.hip), 1.6e9 gathered values with their ranks, 8 ms.
#include <algorithm>
#include <initializer_list>

#include "elocal_internal.hpp"
#include "kernels.hpp"

namespace elocal {

// String of rank r: the greedy unranking of sector_unrank, one spin.
__device__ __forceinline__ uint64_t string_unrank(const uint32_t* __restrict__ binom, int n, int k, uint32_t r) {
  uint64_t s = 0;
  int o = n - 1;
  for (int i = k; i >= 1; --i) {
    while (binom[o * 65 + i] > r) --o;
    r -= binom[o * 65 + i];
    s |= 1ull << o;
    --o;
  }
  return s;
}

__device__ __forceinline__ uint32_t string_rank(const uint32_t* __restrict__ binom, uint64_t s) {
  uint32_t r = 0;
  for (int i = 1; s; ++i, s &= s - 1) r += binom[(__ffsll((unsigned long long)s) - 1) * 65 + i];
  return r;
}

__device__ __forceinline__ int parity_under(uint64_t s, int p) { return __popcll(s & ((1ull << p) - 1ull)) & 1; }

// Row r, column s of pair k = s (s + 1) / 2 + r, r <= s.
__device__ __forceinline__ void pair_of(uint32_t k, int& r, int& s) {
  s = (int)((sqrtf(8.0f * (float)k + 1.0f) - 1.0f) * 0.5f);
  while ((uint32_t)((s + 1) * (s + 2) / 2) <= k) ++s;
  while ((uint32_t)(s * (s + 1) / 2) > k) --s;
  r = (int)k - s * (s + 1) / 2;
}

__device__ __forceinline__ uint32_t pair_index(int p, int q) {
  const int lo = min(p, q), hi = max(p, q);
  return (uint32_t)(hi * (hi + 1) / 2 + lo);
}

// Row stride of W in LDS: the neighbouring rows that the four lane groups of a matrix result
// write are 64 B apart in the banks.
__host__ __device__ inline uint32_t couple_ldw(uint32_t ndb) { return (ndb + 15) / 16 * 16 + 8; }
// A column of W that stays zero.
__host__ __device__ inline uint32_t couple_zero(uint32_t ndb) { return (ndb + 15) / 16 * 16; }

// The integrals by pairs, two[pq][rs] = (pq|rs), rows padded to 16: the operand of
// k_sector_couple, whose lanes read 16 neighbouring rs. After the pairs' rows come those of the
// alpha strings' diagonals, sum_{p in Ia} (pp|rs) (k_string_tables), and a row of zeros.
__global__ void __launch_bounds__(256) k_pair_integrals(SysDev S, SectorTables T) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < T.ldp) T.two[(size_t)(T.npair + T.nda) * T.ldp + i] = 0.0;
  if (i >= T.npair * T.ldp) return;
  const uint32_t pq = i / T.ldp, rs = i % T.ldp;
  int p, q, r = 0, s = 0;
  pair_of(pq, p, q);
  if (rs < T.npair) pair_of(rs, r, s);
  const int n = S.n;
  T.two[i] = rs < T.npair ? S.S[(uint32_t)(((p * n + r) * n + q) * n + s)] : 0.0;
}

// Tables of one spin's strings, one wave per string:
//  * mask[I]: V's sign is the parity of mask_alpha[Ia] & mask_beta[Ib] (bits below every
//    occupied alpha orbital, xor-ed; the beta string itself);
//  * row I of the string's H: col/val[I][e], the diagonal, the singles, the doubles;
//  * alpha, one[I][k]: the strings Ja with <I|E_pq|Ja> != 0 and their row of `two` | sign << 31
//    (singles, the diagonal as one row, zeros);
//  * beta, hop[pair][I]: the string Jb with <I|E_rs|Jb> != 0 or <I|E_sr|Jb> != 0 (at most one
//    of the two; both the diagonal for r = s) as Jb | sign << 15, or the column of zeros.
__global__ void __launch_bounds__(256) k_string_tables(SysDev S, SectorTables T, const uint32_t* __restrict__ binom,
                                                       int spin) {
  __shared__ uint8_t occ[4][64], vir[4][64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t dim = spin ? T.ndb : T.nda, I = blockIdx.x * 4 + wid;
  const int n = S.n, k = spin ? S.nb : S.na, v = n - k;
  const bool live = I < dim;
  const uint64_t s = string_unrank(binom, n, k, live ? I : 0u);
  if (lane < n) {
    const int c = __popcll(s & ((1ull << lane) - 1ull));
    if (s >> lane & 1) occ[wid][c] = (uint8_t)lane;
    else vir[wid][lane - c] = (uint8_t)lane;
  }
  __syncthreads();
  if (!live) return;
  if (lane == 0) {
    uint64_t m = s;
    if (spin == 0) {
      m = 0;
      for (int i = 0; i < k; ++i) m ^= (1ull << occ[wid][i]) - 1ull;
    }
    (spin ? T.mask_b : T.mask_a)[I] = m;
  }
  const uint32_t nsg = (uint32_t)(k * v), npo = (uint32_t)(k * (k - 1) / 2), npv = (uint32_t)(v * (v - 1) / 2);
  const uint32_t ne = 1u + nsg + npo * npv;
  const size_t ld = spin ? T.ldb_h : T.lda_h;
  uint32_t* col = (spin ? T.col_b : T.col_a) + (size_t)I * ld;
  double* val = (spin ? T.val_b : T.val_a) + (size_t)I * ld;
  for (uint32_t e = lane; e < ld; e += 64) {
    uint64_t t = s;
    double x = 0.0;
    if (e == 0) {
      double two = 0.0;
      for (int i = 0; i < k; ++i) {
        const int p = occ[wid][i];
        x += S.h1e[p * n + p];
        for (int j = 0; j < k; ++j) two += S.J2[p * n + occ[wid][j]] - S.K2[p * n + occ[wid][j]];
      }
      x += 0.5 * two;
    } else if (e < 1u + nsg) {
      const int i = occ[wid][(e - 1) / v], a = vir[wid][(e - 1) % v];
      const size_t at = (size_t)(a * n + i);
      x = S.h1e[at];
      for (int j = 0; j < k; ++j) x += S.J3[at * n + occ[wid][j]] - S.K3[at * n + occ[wid][j]];
      int neg = parity_under(t, i);
      t ^= 1ull << i;
      neg ^= parity_under(t, a);
      t ^= 1ull << a;
      x = neg ? -x : x;
    } else if (e < ne) {
      const uint32_t u = e - 1u - nsg, uo = u / npv, uv = u - uo * npv;
      int i, j, a, b;
      // pairs i < j are the strict ones of pair_of's order: (r, s + 1)
      pair_of(uo, i, j);
      pair_of(uv, a, b);
      i = occ[wid][i]; j = occ[wid][j + 1]; a = vir[wid][a]; b = vir[wid][b + 1];
      const size_t ab = (size_t)(a * n + b), nn = (size_t)(n * n);
      x = S.S[(size_t)(i * n + j) * nn + ab] - S.S[(size_t)(j * n + i) * nn + ab];
      int neg = parity_under(t, i);
      t ^= 1ull << i;
      neg ^= parity_under(t, j);
      t ^= 1ull << j;
      neg ^= parity_under(t, b);
      t ^= 1ull << b;
      neg ^= parity_under(t, a);
      t ^= 1ull << a;
      x = neg ? -x : x;
    }
    col[e] = e < ne ? string_rank(binom, t) : I;   // the row's padding: 0 times the diagonal's element
    val[e] = x;
  }
  if (spin == 0) {
    // <I|E_pq|Ja>: p is in I, q in Ja = I - p + q
    for (uint32_t e = lane; e < T.K; e += 64) {
      uint2 o = make_uint2(I, e == nsg ? T.npair + I : T.npair + T.nda);
      if (e < nsg) {
        const int p = occ[wid][e / v], q = vir[wid][e % v];
        uint64_t t = s;
        int neg = parity_under(t, p);
        t ^= 1ull << p;
        neg ^= parity_under(t, q);
        t ^= 1ull << q;
        o = make_uint2(string_rank(binom, t), pair_index(p, q) | (uint32_t)neg << 31);
      }
      T.one[(size_t)I * T.K + e] = o;
    }
    for (uint32_t e = lane; e < T.ldp; e += 64) {
      double x = 0.0;
      if (e < T.npair) {
        int r, q;
        pair_of(e, r, q);
        for (int i = 0; i < k; ++i) {
          const int p = occ[wid][i];
          x += S.S[(uint32_t)(((p * n + r) * n + p) * n + q)];
        }
      }
      T.two[(size_t)(T.npair + I) * T.ldp + e] = x;
    }
  } else {
    for (uint32_t e = lane; e < T.ldp; e += 64) {
      int r, q;
      pair_of(e, r, q);
      if (e >= T.npair) {
        T.hop[(size_t)e * T.ndb + I] = (uint16_t)couple_zero(T.ndb);
        continue;
      }
      const int br = (int)(s >> r & 1), bq = (int)(s >> q & 1);
      uint16_t h = (uint16_t)couple_zero(T.ndb);
      if (r == q ? br : br != bq) {
        uint64_t t = s;
        const int from = br ? r : q, to = r == q ? r : br ? q : r;
        int neg = parity_under(t, from);
        t ^= 1ull << from;
        neg ^= parity_under(t, to);
        t ^= 1ull << to;
        h = (uint16_t)(string_rank(binom, t) | (uint32_t)neg << 15);
      }
      T.hop[(size_t)e * T.ndb + I] = h;
    }
  }
}

// Vectors: out = V in the order alpha first (sign), and its transpose. 32 x 32 tiles through
// LDS, so that both sides are read and written along their rows.
__global__ void __launch_bounds__(256) k_sector_turn(SectorTables T, const double* __restrict__ v, int sign,
                                                     double* __restrict__ out, double* __restrict__ outT) {
  __shared__ double t[32][33];
  const uint32_t a0 = blockIdx.y * 32, b0 = blockIdx.x * 32;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
  for (int i = y; i < 32; i += 8) {
    const uint32_t a = a0 + i, b = b0 + x;
    if (a >= T.nda || b >= T.ndb) continue;
    double e = v[(size_t)a * T.ndb + b];
    if (sign && (__popcll(T.mask_a[a] & T.mask_b[b]) & 1)) e = -e;
    if (out) out[(size_t)a * T.ndb + b] = e;
    t[i][x] = e;
  }
  __syncthreads();
  for (int i = y; i < 32; i += 8) {
    const uint32_t b = b0 + i, a = a0 + x;
    if (a < T.nda && b < T.ndb) outT[(size_t)b * T.nda + a] = t[x][i];
  }
}

// Y = H X for one spin's string matrix, X with `nc` columns: a wave per row and 64 columns.
// The row's entries are wave-uniform (scalar loads) and the rows of X whole lines; a panel of
// 64 columns stays with one XCD (blocks go to the XCDs in turn), whose L2 then holds it. Bound
// by the 512 B per entry that a CU reads from there: 115 us for 924 strings either way round,
// 16 TB/s; twice the columns per wave and entries handed out by lanes instead of scalar loads
// took 125, twice the entries in flight 119.
constexpr int kRowBatch = 8;   // entries in flight (rows of the tables are padded to 16)
__global__ void __launch_bounds__(256) k_string_rows(const uint32_t* __restrict__ col, const double* __restrict__ val,
                                                     uint32_t ld, uint32_t rows, uint32_t nc,
                                                     const double* __restrict__ X, double* __restrict__ Y) {
  const int lane = threadIdx.x & 63;
  const uint32_t rb = (rows + 3) / 4, slot = blockIdx.x >> 3;
  const uint32_t panel = (blockIdx.x & 7) + 8 * (slot / rb);
  const uint32_t I = (uint32_t)__builtin_amdgcn_readfirstlane((int)((slot % rb) * 4 + (threadIdx.x >> 6)));
  if (I >= rows || panel * 64 >= nc) return;
  const uint32_t c = panel * 64 + lane, cc = min(c, nc - 1);
  const uint32_t* pc = col + (size_t)I * ld;
  const double* pv = val + (size_t)I * ld;
  double acc = 0.0;
  for (uint32_t e = 0; e < ld; e += kRowBatch) {
    double x[kRowBatch];
#pragma unroll
    for (int k = 0; k < kRowBatch; ++k) x[k] = X[(size_t)pc[e + k] * nc + cc];
#pragma unroll
    for (int k = 0; k < kRowBatch; ++k) acc += pv[e + k] * x[k];
  }
  if (c < nc) Y[(size_t)I * nc + c] = acc;
}

typedef double f64x4 __attribute__((ext_vector_type(4)));

// One Ia per block (W fills the CU's LDS: products and gathers take turns): W in chunks of 16 pairs rs (the rows of one matrix instruction) in LDS,
// each gathered by every Ib before the next; then y = ch (H V) + cv v + cz z and the block's
// partial sums of y.y and y.v. v, z and y are the caller's: with `sign` they are in the
// library's order, V is not. 179 us at 924 x 924 strings; with every integral gathered from
// S[p][r][q][s] (64 lines a load), conditional gathers and an instruction per diagonal
// excitation, 347 us.
constexpr int kCoupleThreads = 1024;
// STEPS: k-steps (of 4 excitations) of one pass over W; with ONE they are all of a string's.
template <int J, int STEPS, bool ONE>   // J: strings Ib per thread
__global__ void __launch_bounds__(kCoupleThreads) k_sector_couple(SectorTables T, double ch, double cv,
                                                                  const double* __restrict__ v, double cz,
                                                                  const double* __restrict__ z, int sign,
                                                                  const double* __restrict__ V,
                                                                  const double* __restrict__ Ya,
                                                                  const double* __restrict__ YbT,
                                                                  double* __restrict__ y,
                                                                  double* __restrict__ partial) {
  extern __shared__ __attribute__((aligned(16))) double W[];
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int g = lane >> 4, r16 = lane & 15;
  // neighbouring strings, which reach many of the same rows, on one XCD (blocks go to the
  // XCDs in turn)
  const uint32_t Ia = (blockIdx.x & 7) * ((T.nda + 7) / 8) + (blockIdx.x >> 3);
  if (Ia >= T.nda) return;
  const uint32_t ndb = T.ndb, tiles = (ndb + 15) / 16, ldw = couple_ldw(ndb);
  const uint32_t K = T.K;
  const uint2* one = T.one + (size_t)Ia * K + g;
  for (uint32_t i = threadIdx.x; i < 16; i += kCoupleThreads) W[i * ldw + couple_zero(ndb)] = 0.0;
  uint32_t row[STEPS], arow[STEPS];   // byte offsets; bit 0 of arow: the sign
  auto load_one = [&](uint32_t k0) {
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
      const uint2 o = one[k0 + 4 * k];
      row[k] = (o.x * ndb + r16) * 8u;   // (vectors of less than 4 GiB)
      arow[k] = ((o.y & 0x7FFFFFFFu) * T.ldp + r16) * 8u | o.y >> 31;
    }
  };
  if constexpr (ONE) load_one(0);
  double acc[J];
#pragma unroll
  for (int j = 0; j < J; ++j) acc[j] = 0.0;
  for (uint32_t c0 = 0; c0 < T.npair; c0 += 16) {
    __syncthreads();   // the last chunk of W has been read
    for (uint32_t k0 = 0; k0 < K; k0 += 4 * STEPS) {
      if constexpr (!ONE) load_one(k0);
      const char* tw = (const char*)(T.two + c0);
      double a[STEPS];
#pragma unroll
      for (int k = 0; k < STEPS; ++k) {
        const double x = *(const double*)(tw + (arow[k] & ~7u));
        a[k] = __hiloint2double(__double2hiint(x) ^ (int)(arow[k] << 31), __double2loint(x));
      }
      for (uint32_t t = wid; t < tiles; t += kCoupleThreads / 64) {
        // past the last column: the next row's, or what follows V in its workspace (columns of
        // W that no string gathers)
        const char* vt = (const char*)(V + 16 * t);
        double b[STEPS];
#pragma unroll
        for (int k = 0; k < STEPS; ++k) b[k] = *(const double*)(vt + row[k]);
        double* w = W + 16 * t + r16;
        f64x4 d = {0.0, 0.0, 0.0, 0.0};
        if (!ONE && k0 > 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) d[i] = w[(4 * i + g) * ldw];
        }
#pragma unroll
        for (int k = 0; k < STEPS; ++k) d = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k], b[k], d, 0, 0, 0);
        // the instruction returns row 4 i + lane / 16 in register i
#pragma unroll
        for (int i = 0; i < 4; ++i) w[(4 * i + g) * ldw] = d[i];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const uint32_t Ib = threadIdx.x + kCoupleThreads * j;
      if (Ib >= ndb) continue;
      const uint16_t* hop = T.hop + (size_t)c0 * ndb + Ib;
      uint32_t h[16];
      double x[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) h[i] = hop[(uint32_t)i * ndb];
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = W[(uint32_t)i * ldw + (h[i] & 0x7FFFu)];
#pragma unroll
      for (int i = 0; i < 16; ++i)
        acc[j] += __hiloint2double(__double2hiint(x[i]) ^ (int)((h[i] & 0x8000u) << 16), __double2loint(x[i]));
    }
  }
  const uint64_t ma = T.mask_a[Ia];
  double yy = 0.0, yv = 0.0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const uint32_t Ib = threadIdx.x + kCoupleThreads * j;
    if (Ib >= ndb) continue;
    const size_t at = (size_t)Ia * ndb + Ib;
    double h = acc[j] + Ya[at] + YbT[(size_t)Ib * T.nda + Ia];
    if (sign && (__popcll(ma & T.mask_b[Ib]) & 1)) h = -h;
    const double vr = v[at];
    double yr = ch * h + cv * vr;
    if (z) yr += cz * z[at];
    y[at] = yr;
    yy += yr * yr;
    yv += yr * vr;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    yy += __shfl_xor(yy, off);
    yv += __shfl_xor(yv, off);
  }
  __syncthreads();   // W is free: the waves' sums
  if (lane == 0) {
    W[2 * wid] = yy;
    W[2 * wid + 1] = yv;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    yy = yv = 0.0;
    for (int i = 0; i < kCoupleThreads / 64; ++i) {
      yy += W[2 * i];
      yv += W[2 * i + 1];
    }
    partial[2 * Ia] = yy;
    partial[2 * Ia + 1] = yv;
  }
}

// ----------------------------------------------------------------------------- launchers
// Excitations of an alpha string, padded to what a kernel takes: with the diagonal, 16, 32, 40
// or a multiple of 48. (17 to 24 take 32 and not a size of their own: products of zeros in sectors of
// few strings, whose calls are launches and gathers, 11 orbitals, 2 and 5 electrons 89 us.)
uint32_t sector_couple_k(uint32_t singles, uint32_t ndb) {
  const uint32_t k = singles + 1;
  if (ndb <= (uint32_t)kCoupleThreads)
    for (uint32_t f : {16u, 32u, 40u})
      if (k <= f) return f;
  return (k + 47) / 48 * 48;
}

size_t sector_couple_lds(uint32_t ndb) { return (size_t)couple_ldw(ndb) * 16 * sizeof(double); }

hipError_t launch_sector_tables(const SysDev& S, const SectorTables& T, const uint32_t* binom, hipStream_t st) {
  hipLaunchKernelGGL(k_pair_integrals, dim3((T.npair * T.ldp + 255) / 256), dim3(256), 0, st, S, T);
  hipLaunchKernelGGL(k_string_tables, dim3((T.nda + 3) / 4), dim3(256), 0, st, S, T, binom, 0);
  hipLaunchKernelGGL(k_string_tables, dim3((T.ndb + 3) / 4), dim3(256), 0, st, S, T, binom, 1);
  return hipGetLastError();
}

hipError_t launch_sector_turn(const SectorTables& T, const double* v, int sign, double* out, double* outT,
                              hipStream_t st) {
  hipLaunchKernelGGL(k_sector_turn, dim3((T.ndb + 31) / 32, (T.nda + 31) / 32), dim3(256), 0, st, T, v, sign, out,
                     outT);
  return hipGetLastError();
}

hipError_t launch_sector_product(const SectorTables& T, double ch, double cv, const double* v,
                                 double cz, const double* z, int sign, const double* V, const double* VT, double* Ya,
                                 double* YbT, double* y, double* partial, hipStream_t st) {
  auto panels = [](uint32_t nc) { return (nc + 511) / 512 * 8; };
  hipLaunchKernelGGL(k_string_rows, dim3(panels(T.ndb) * ((T.nda + 3) / 4)), dim3(256), 0, st, T.col_a, T.val_a,
                     T.lda_h, T.nda, T.ndb, V, Ya);
  hipLaunchKernelGGL(k_string_rows, dim3(panels(T.nda) * ((T.ndb + 3) / 4)), dim3(256), 0, st, T.col_b, T.val_b,
                     T.ldb_h, T.ndb, T.nda, VT, YbT);
  const size_t lds = std::max<size_t>(sector_couple_lds(T.ndb), 512);
  auto kern = T.ndb > kCoupleThreads ? k_sector_couple<2, 12, false>
              : T.K == 16            ? k_sector_couple<1, 4, true>
              : T.K == 32            ? k_sector_couple<1, 8, true>
              : T.K == 40            ? k_sector_couple<1, 10, true>
              : T.K == 48            ? k_sector_couple<1, 12, true>
                                     : k_sector_couple<1, 12, false>;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((T.nda + 7) / 8 * 8), dim3(kCoupleThreads), lds, st, T, ch, cv, v, cz, z, sign, V, Ya, YbT, y,
                     partial);
  return hipGetLastError();
}

}  // namespace elocal
