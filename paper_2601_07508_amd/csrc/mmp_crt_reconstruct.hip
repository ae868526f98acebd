// Chinese remainder reconstruction of integer products from their residues
// (Section 5.2: the multimodular product recovered by the CRT, exact once the
// moduli's product M exceeds the entries, eq. CRT2).
//
// Up to about 48 moduli, as a contraction on the INT8 matrix cores
// (crt_contract_kernel): with g_t = r_t (M / p_t)^{-1} mod p_t,
//   X = sum_t g_t (M / p_t) - h M,   h = floor(sum_t g_t / p_t).
// The bytes of every g_t multiply the bytes of the constants M / p_t and M in
// one exact int32 product per entry and output byte, and a carry chain makes
// the limbs: O(s) binary64 steps an entry instead of Garner's O(s^2).
//
// Beyond that, per entry on the device (crt_reconstruct_kernel):
//   1. Garner's mixed-radix digits: X = v_0 + p_0 (v_1 + p_1 (v_2 + ...)),
//      0 <= v_j < p_j, with v_j = (r_j - X_{j-1}) (p_0 ... p_{j-1})^{-1} mod p_j
//      and X_{j-1} mod p_j evaluated by Horner over v_{j-1} ... v_0.  Every
//      step is binary64 modular arithmetic: Alg. 2 for the products, Alg. 1
//      for the reductions, all factors below the modulus and p <= 2^52 / 3
//      (Prop. Joris's range, x y <= 2^(t-1) p / 3).
//   2. The digits into 64-bit limbs by Horner from the top, acc = acc p_i +
//      v_i with 64 x 64 -> 128-bit limb products.
// The inverses (p_0 ... p_{j-1})^{-1} mod p_j and the limb count of M come
// from the host; p_i mod p_j is tabulated in LDS per workgroup.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstring>
#include <type_traits>
#include <vector>

#include "mmp_internal.h"

namespace mmp {
namespace {

constexpr int kMaxModuli = 64;
constexpr uint64_t kRecPMax = (1ull << 52) / 3;  // Alg. 2 with both factors below p

struct RecArgs {
  const double* C[kMaxModuli];
  double p[kMaxModuli], q[kMaxModuli], inv[kMaxModuli];
  int act[kMaxModuli];  // limbs of p_i p_{i+1} ... p_{s-1}, for Horner step i
  int64_t ldc, m, n, ldo;
  uint64_t* out;
  int s, limbs;
};

// Alg. 1: x mod p for integer 0 <= x < 2^53.
__device__ __forceinline__ double rec_fmod(double x, double p, double q) {
  const double c = floor(x * q);
  double d = fma(-c, p, x);
  d = (d >= p) ? d - p : d;
  d = (d < 0.0) ? d + p : d;
  return d;
}

// Alg. 2: x y mod p for 0 <= x, y < p <= 2^52 / 3.
__device__ __forceinline__ double rec_mulmod(double x, double y, double p, double q) {
  const double h = x * y;
  const double l = fma(x, y, -h);
  const double c = floor(h * q);
  const double d = fma(-c, p, h);
  double e = d + l;
  e = (e >= p) ? e - p : e;
  e = (e < 0.0) ? e + p : e;
  return e;
}

// (t c + v) mod p for 0 <= t, c < p <= 2^52 / 3 and 0 <= v < 2^52: Alg. 2
// without its corrections leaves e = t c - b p in [-p, 2p), so
// e + v + p lies in [0, 2^53) and one Alg. 1 finishes.
__device__ __forceinline__ double rec_muladd(double t, double c, double v, double p, double q) {
  const double h = t * c;
  const double l = fma(t, c, -h);
  const double b = floor(h * q);
  const double d = fma(-b, p, h);
  const double e = d + l;
  return rec_fmod((e + p) + v, p, q);
}

// NT threads per workgroup; LDS holds the p_i mod p_j table and NT columns of
// s digits.
template <int LMAX, int NT>
__global__ __launch_bounds__(NT) void crt_reconstruct_kernel(const RecArgs a) {
  constexpr int kRecThreads = NT;
  extern __shared__ double lds[];
  const int s = a.s;
  double* pm = lds;                   // [s][s]: p_i mod p_j at i * s + j
  double* vcol = lds + s * s;         // [s][kRecThreads]: this thread's digits
  const int tid = threadIdx.x;
  for (int x = tid; x < s * s; x += kRecThreads) {
    const int i = x / s, j = x - i * s;
    pm[x] = rec_fmod(a.p[i], a.p[j], a.q[j]);
  }
  __syncthreads();
  const int64_t total = a.m * a.n;
  for (int64_t e = (int64_t)blockIdx.x * kRecThreads + tid; e < total; e += (int64_t)gridDim.x * kRecThreads) {
    const int64_t row = e / a.n, col = e - row * a.n;
    const int64_t off = row * a.ldc + col;
    // all residues first (independent loads), then Garner in place:
    // v_0 = r_0; v_j from r_j and X_{j-1} mod p_j
    for (int j = 0; j < s; j++) vcol[j * kRecThreads + tid] = a.C[j][off];
    for (int j = 1; j < s; j++) {
      const double pj = a.p[j], qj = a.q[j];
      double t = rec_fmod(vcol[(j - 1) * kRecThreads + tid], pj, qj);
      for (int i = j - 2; i >= 0; i--) t = rec_muladd(t, pm[i * s + j], vcol[i * kRecThreads + tid], pj, qj);
      double d = vcol[j * kRecThreads + tid] - t;
      d = (d < 0.0) ? d + pj : d;
      vcol[j * kRecThreads + tid] = rec_mulmod(d, a.inv[j], pj, qj);
    }
    // limbs: acc = v_{s-1}, then acc = acc p_i + v_i for i = s-2 .. 0
    uint64_t acc[LMAX];
#pragma unroll
    for (int w = 0; w < LMAX; w++) acc[w] = 0;
    acc[0] = (uint64_t)vcol[(s - 1) * kRecThreads + tid];
    for (int i = s - 2; i >= 0; i--) {
      const uint64_t pi = (uint64_t)a.p[i];
      uint64_t carry = (uint64_t)vcol[i * kRecThreads + tid];
      const int act = a.act[i];  // limbs that can be nonzero after this step
#pragma unroll
      for (int w = 0; w < LMAX; w++) {
        if (w < act) {
          const unsigned __int128 t = (unsigned __int128)acc[w] * pi + carry;
          acc[w] = (uint64_t)t;
          carry = (uint64_t)(t >> 64);
        }
      }
    }
#pragma unroll
    for (int w = 0; w < LMAX; w++)
      if (w < a.limbs) a.out[((int64_t)w * a.m + row) * a.ldo + col] = acc[w];
    for (int w = LMAX; w < a.limbs; w++) a.out[((int64_t)w * a.m + row) * a.ldo + col] = 0;
  }
}

// ---------------------------------------------------------------- contraction

typedef int int4v __attribute__((ext_vector_type(4)));

// From five moduli: a k-step holds eight, and with four Garner's few steps are as
// fast (2048^2 entries: 48 us either way with 4, 64 against 73 us with 5; with 3,
// 57 against 37).
constexpr int kConMinModuli = 5;
constexpr int kConMaxModuli = 48;     // six 64-byte k-steps of eight moduli
constexpr int kConDigitBytes = 12288; // the constants' digits, in the kernel arguments
constexpr int kConWaves = 8;
constexpr int64_t kConLdsMax = 160 * 1024;
constexpr int kConRow = 80;           // scratch bytes per entry: 16 sums, padded

// Bytes of the digits of 8 KS + 1 constants, each of at most 51 KS + 1 (a modulus
// has 50.5 bits), or all that the arguments leave room for.  Sized by the k-steps:
// with the largest table in every launch, 14 KB of arguments, calls of 5 and 6 moduli
// and up to 2^19 entries took 15.3 and 16.3 us, more than Garner's kernel (14.8 and
// 16.0), with their own 14.5 and 15.5.
constexpr int con_digit_bytes(int ksteps) {
  const int all = (8 * ksteps + 1) * (51 * ksteps + 1);
  return ((all < kConDigitBytes ? all : kConDigitBytes) + 15) / 16 * 16;
}

template <int KS>
struct ConArgs {
  const double* C[8 * KS];
  double p[8 * KS], q[8 * KS], inv[8 * KS];
  int64_t ldc, m, n, ldo;
  uint64_t* out;
  int s, limbs;
  int digits;     // signed base-256 digits of M and of each M / p_t
  int col_tiles;  // 16 output bytes each: the digits' products and M's limbs
  int8_t dig[con_digit_bytes(KS)];  // [s + 1][digits]: the M / p_t, then M
};

static_assert(sizeof(ConArgs<1>) < 1024 && sizeof(ConArgs<6>) < 16384, "as little as a launch has to carry");

// LDS: the constants as MFMA operands, [column tile][k-step][1 KB]; each
// wave's sums, 64 entries of 16; the moduli's p, q, inverse.
inline size_t con_lds(int ksteps, int col_tiles) {
  return (size_t)col_tiles * ksteps * 1024 + kConWaves * 64 * kConRow + (size_t)ksteps * 8 * 3 * sizeof(double);
}

// What bounds it: reading s residues and writing the limbs.  2048^2 entries from
// 32 moduli (1.74 GB) take 368 us, 4.7 TB/s, a large copy's rate, where Garner's
// kernel took 2914; from 48 of them 627 against 14886.  A wave takes 64
// entries.  Lane 16 q + r works on entry r of each 16-entry group and on moduli
// 8 ks + 2 q, + 1, whose g digits are the 16 k-bytes (2 moduli of 8 bytes) that
// the 16x16x64 MFMA takes from that lane: no exchange between lanes.
//   g: Alg. 2 with the quotient rounded to nearest and no correction, |g| <
//     0.7 p < 2^50, seven signed digits; the eighth byte multiplies zeros, except
//     modulus 0's, which holds -h and multiplies M's digits.
//   h: |sum g / p| <= 34 is summed with an error below 2^-40, so h = floor(sum +
//     2^-36) puts X in [-2^-35 M, M).  A negative X (its true value next to M)
//     is found by the last carry; those entries repeat with h - 1.
//   sums: |sum| <= 8 48 2^14 < 2^22.6, so two neighbouring bytes' sums combine
//     in int32, and 32 bits of a limb take one 64-bit addition with the carry.
template <int KS>
__global__ __launch_bounds__(64 * kConWaves, 2) void crt_contract_kernel(const ConArgs<KS> a) {
  extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63, q4 = lane >> 4, r16 = lane & 15;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int CT = a.col_tiles, s = a.s, D = a.digits;
  int8_t* const table = smem;
  int8_t* const sums = smem + CT * KS * 1024 + wv * 64 * kConRow;
  double* const pq = (double*)(smem + CT * KS * 1024 + kConWaves * 64 * kConRow);  // [8 KS][3]
  {
    // the digits through the scratch, then each operand's 16 bytes
    int8_t* const dig = smem + CT * KS * 1024;
    for (int i = tid; i < (s + 1) * D; i += 64 * kConWaves) dig[i] = a.dig[i];
    for (int t = tid; t < 8 * KS; t += 64 * kConWaves) {
      pq[3 * t] = t < s ? a.p[t] : 1.0;
      pq[3 * t + 1] = t < s ? a.q[t] : 1.0;
      pq[3 * t + 2] = t < s ? a.inv[t] : 0.0;
    }
    __syncthreads();
    for (int f = tid; f < CT * KS * 64; f += 64 * kConWaves) {
      const int l = f & 63, ks = (f >> 6) % KS, c = (f >> 6) / KS;
      const int w = 16 * c + (l & 15);
      uint32_t word[4];
#pragma unroll
      for (int b = 0; b < 16; b++) {
        const int t = 8 * ks + 2 * (l >> 4) + (b >> 3), i = b & 7;
        int v = 0;
        if (i < 7 && t < s && w >= i && w - i < D) v = dig[t * D + w - i];
        if (i == 7 && t == 0 && w < D) v = dig[s * D + w];
        if (b % 4 == 0) word[b / 4] = 0;
        word[b / 4] |= (uint32_t)(uint8_t)v << (8 * (b % 4));
      }
      *(int4v*)(table + f * 16) = (int4v){(int)word[0], (int)word[1], (int)word[2], (int)word[3]};
    }
    __syncthreads();
  }
  const int64_t total = a.m * a.n;
  const bool packed_in = a.ldc == a.n;
  for (int64_t unit = (int64_t)blockIdx.x * kConWaves + wv; unit * 64 < total;
       unit += (int64_t)gridDim.x * kConWaves) {
    const int64_t e0 = unit * 64;
    int64_t off[4];
#pragma unroll
    for (int x = 0; x < 4; x++) {
      const int64_t e = min(e0 + 16 * x + r16, total - 1);
      const int64_t row = packed_in ? 0 : e / a.n;
      off[x] = packed_in ? e : row * a.ldc + (e - row * a.n);
    }
    // all residues first, so that every load is in flight at once
    double g[KS][2][4];
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int h = 0; h < 2; h++) {
        const int t = 8 * ks + 2 * q4 + h;
        const double* C = a.C[t < s ? t : 0];
#pragma unroll
        for (int x = 0; x < 4; x++) g[ks][h][x] = __builtin_nontemporal_load(C + off[x]);
      }
    double S[4] = {0.0, 0.0, 0.0, 0.0};
    int4v A[4][KS];
#pragma unroll
    for (int ks = 0; ks < KS; ks++)
#pragma unroll
      for (int h = 0; h < 2; h++) {
        const double* c3 = pq + 3 * (8 * ks + 2 * q4 + h);
        const double p = c3[0], q = c3[1], y = c3[2];
#pragma unroll
        for (int x = 0; x < 4; x++) {
          const double u = g[ks][h][x] * y;
          const double l = fma(g[ks][h][x], y, -u);
          const double e = fma(-rint(u * q), p, u) + l;
          S[x] = fma(e, q, S[x]);
          // e + 1.5 2^52 holds e in its low bits; digits are the bytes of e + 0x80..80, less 128
          const uint64_t b = (uint64_t)__double_as_longlong(e + 6755399441055744.0) +
                             (0x0080808080808080ull - 0x4338000000000000ull);
          A[x][ks][2 * h] = (int)((uint32_t)b ^ 0x80808080u);
          A[x][ks][2 * h + 1] = (int)((uint32_t)(b >> 32) ^ 0x00808080u);
        }
      }
    int h[4];
#pragma unroll
    for (int x = 0; x < 4; x++) {
      double t = S[x];
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);
      h[x] = (int)floor(t + 0x1p-36);
    }
    const int64_t e = e0 + lane;
    const bool live = e < total;
    const int64_t row = e / a.n;
    uint64_t* const out = a.out + row * a.ldo + (e - row * a.n);
    const int64_t plane = a.m * a.ldo;
    // at most two rounds: h, then h - 1 where the first gave a negative X
    for (int round = 0; round < 2; round++) {
      if (q4 == 0) {
#pragma unroll
        for (int x = 0; x < 4; x++)
          A[x][0][1] = (int)(((uint32_t)A[x][0][1] & 0x00ffffffu) | ((uint32_t)-h[x] << 24));
      }
      int carry = 0;
      for (int c = 0; c < CT; c++) {
        int4v B[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ks++) B[ks] = *(const int4v*)(table + (c * KS + ks) * 1024 + lane * 16);
#pragma unroll
        for (int x = 0; x < 4; x++) {
          int4v acc = {0, 0, 0, 0};
#pragma unroll
          for (int ks = 0; ks < KS; ks++) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(B[ks], A[x][ks], acc, 0, 0, 0);
          // lane 16 q + r: bytes 4 q .. 4 q + 3 of entry r
          *(int4v*)(sums + (16 * x + r16) * kConRow + q4 * 16) = acc;
        }
        __builtin_amdgcn_wave_barrier();
        int4v v[4];
#pragma unroll
        for (int i = 0; i < 4; i++) v[i] = *(const int4v*)(sums + lane * kConRow + i * 16);
        __builtin_amdgcn_wave_barrier();
        uint32_t w32[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const int lo = v[i][0] + (v[i][1] << 8), hi = v[i][2] + (v[i][3] << 8);
          const int64_t t = (int64_t)carry + lo + ((int64_t)hi << 16);
          w32[i] = (uint32_t)t;
          carry = (int)(t >> 32);
        }
#pragma unroll
        for (int i = 0; i < 2; i++)
          if (live && 2 * c + i < a.limbs)
            __builtin_nontemporal_store((uint64_t)w32[2 * i] | (uint64_t)w32[2 * i + 1] << 32, out + (2 * c + i) * plane);
      }
      const int neg = carry < 0 ? 1 : 0;
      if (!__any(neg)) break;  // uniform per wave
#pragma unroll
      for (int x = 0; x < 4; x++) h[x] -= __shfl(neg, 16 * x + r16);
    }
    if (live)
      for (int w = 2 * CT; w < a.limbs; w++) out[w * plane] = 0;
  }
}

// x y mod p for x, y < p < 2^52: the quotient from 64-bit long double
// significands is within one, the remainder comes from the low 64 bits.
uint64_t mulmod(uint64_t x, uint64_t y, uint64_t p, long double pinv) {
  const uint64_t c = (uint64_t)((long double)x * (long double)y * pinv);
  int64_t r = (int64_t)(x * y - c * p);
  if (r < 0) r += (int64_t)p;
  if (r >= (int64_t)p) r -= (int64_t)p;
  return (uint64_t)r;
}

// x^{-1} mod p, 0 <= x < p (extended Euclid); false when gcd(x, p) != 1.
bool inv_mod(uint64_t x, uint64_t p, uint64_t* inv) {
  int64_t r0 = (int64_t)p, r1 = (int64_t)x, t0 = 0, t1 = 1;  // |t| <= p < 2^52
  while (r1 != 0) {
    const int64_t qq = r0 / r1;
    int64_t tmp = r0 - qq * r1;
    r0 = r1;
    r1 = tmp;
    tmp = t0 - qq * t1;
    t0 = t1;
    t1 = tmp;
  }
  if (r0 != 1) return false;
  *inv = (uint64_t)(t0 < 0 ? t0 + (int64_t)p : t0);
  return true;
}

// Little-endian products of moduli: at most 64 moduli below 2^50.5, 51 limbs.
struct Big {
  uint64_t w[52];
  int n = 1;
  Big() { w[0] = 1; }
  void mul(uint64_t x) {
    unsigned __int128 carry = 0;
    for (int i = 0; i < n; i++) {
      const unsigned __int128 t = (unsigned __int128)w[i] * x + carry;
      w[i] = (uint64_t)t;
      carry = t >> 64;
    }
    if (carry) w[n++] = (uint64_t)carry;
  }
  int bits() const { return 64 * n - __builtin_clzll(w[n - 1]); }
};

// x y, at most 52 limbs
Big product(const Big& x, const Big& y) {
  Big r;
  std::memset(r.w, 0, sizeof(r.w));
  for (int i = 0; i < x.n; i++) {
    unsigned __int128 carry = 0;
    for (int j = 0; j < y.n; j++) {
      const unsigned __int128 t = (unsigned __int128)x.w[i] * y.w[j] + r.w[i + j] + carry;
      r.w[i + j] = (uint64_t)t;
      carry = t >> 64;
    }
    if (i + y.n < 52) r.w[i + y.n] = (uint64_t)carry;
  }
  r.n = x.n + y.n;
  while (r.n > 1 && (r.n > 52 || r.w[r.n - 1] == 0)) r.n--;
  return r;
}

// D signed base-256 digits of x < 2^(8 D - 2): the bytes of x + 0x80..80, less 128
void signed_digits(const Big& x, int D, int8_t* out) {
  int carry = 0;
  for (int i = 0; i < D; i++) {
    const int byte = i / 8 < x.n ? (int)(x.w[i / 8] >> (8 * (i % 8)) & 0xff) : 0;
    const int v = byte + 0x80 + carry;
    out[i] = (int8_t)((v & 0xff) ^ 0x80);
    carry = v >> 8;
  }
}

// Number of 64-bit limbs of prod(p[lo..hi)).
int limbs_of_product(const uint64_t* p, int lo, int hi) {
  std::vector<uint64_t> x(1, 1);
  for (int i = lo; i < hi; i++) {
    unsigned __int128 carry = 0;
    for (auto& w : x) {
      const unsigned __int128 t = (unsigned __int128)w * p[i] + carry;
      w = (uint64_t)t;
      carry = t >> 64;
    }
    if (carry) x.push_back((uint64_t)carry);
  }
  int n = (int)x.size();
  while (n > 1 && x[n - 1] == 0) n--;
  return n;
}

template <int KS>
int launch_contract(const ConArgs<KS>& a, void* stream) {
  const int64_t units = (a.m * a.n + 63) / 64;
  const size_t shmem = con_lds(KS, a.col_tiles);
  static std::atomic<int> ready[64];  // per device: the LDS limit is raised
  int dev = 0;
  if (int e = (int)hipGetDevice(&dev)) return e;
  if (dev >= 64 || !ready[dev].load()) {
    if (int e = (int)hipFuncSetAttribute((const void*)crt_contract_kernel<KS>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, kConLdsMax))
      return e;
    if (dev < 64) ready[dev].store(1);
  }
  // persistent: the constants' operands are made once per workgroup
  const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(2, kConLdsMax / (int64_t)shmem));
  const int64_t blocks = std::min<int64_t>((units + kConWaves - 1) / kConWaves, 256 * per_cu);
  TimerTok* t = timer_begin("crt_reconstruct");
  hipExtLaunchKernelGGL((crt_contract_kernel<KS>), dim3((unsigned)blocks), dim3(64 * kConWaves), shmem,
                        (hipStream_t)stream, timer_start(t), timer_stop(t), 0, a);
  const int e = (int)hipGetLastError();
  timer_commit(t, e);
  return e;
}

// 128 threads up to 32 moduli (at most 40 KB of LDS), 64 beyond (at most 64 KB).
template <int LMAX>
int launch_rec(const RecArgs& a, void* stream) {
  const int64_t total = a.m * a.n;
  const int nt = a.s <= 32 ? 128 : 64;
  const int64_t blocks = std::min<int64_t>((total + nt - 1) / nt, 16384);
  const size_t shmem = sizeof(double) * ((size_t)a.s * a.s + (size_t)a.s * nt);
  if (nt == 128)
    hipLaunchKernelGGL((crt_reconstruct_kernel<LMAX, 128>), dim3((unsigned)blocks), dim3(128), shmem,
                       (hipStream_t)stream, a);
  else
    hipLaunchKernelGGL((crt_reconstruct_kernel<LMAX, 64>), dim3((unsigned)blocks), dim3(64), shmem,
                       (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

}  // namespace
}  // namespace mmp

using namespace mmp;

extern "C" int mmp_crt_reconstruct(const double* const* C, int64_t ldc, const uint64_t* moduli, int nmoduli,
                                   int64_t m, int64_t n, uint64_t* out, int64_t ldo, int limbs, void* stream) {
  try {
    if (m < 0 || n < 0 || nmoduli < 1 || nmoduli > kMaxModuli || !moduli || !C) return MMP_EINVAL;
    for (int i = 0; i < nmoduli; i++)
      if (moduli[i] < 2 || moduli[i] > kRecPMax) return MMP_EINVAL;
    // pairwise coprime: each modulus prime to the product of the others
    uint64_t rest_inv[kMaxModuli];  // (M / p_j)^{-1} mod p_j
    for (int j = 0; j < nmoduli; j++) {
      const uint64_t p = moduli[j];
      const long double pinv = 1.0L / (long double)p;
      uint64_t prod = 1;
      for (int i = 0; i < nmoduli; i++)
        if (i != j) prod = mulmod(prod, moduli[i] >= p ? moduli[i] % p : moduli[i], p, pinv);
      if (!inv_mod(prod, p, &rest_inv[j])) return MMP_EINVAL;
    }
    Big M;
    for (int i = 0; i < nmoduli; i++) M.mul(moduli[i]);
    // limbs that hold M - 1 (M itself may be a power of 2^64 only if one limb more)
    const int lm = limbs_of_product(moduli, 0, nmoduli);
    if (limbs < lm) return MMP_EINVAL;  // some X below M would not fit
    if (m == 0 || n == 0) return MMP_OK;
    if (!out || ldc < n || ldo < n) return MMP_EINVAL;
    for (int i = 0; i < nmoduli; i++) {
      if (!C[i]) return MMP_EINVAL;
      if (ranges_overlap(out, span_bytes((int64_t)limbs * m, n, ldo), C[i], span_bytes(m, n, ldc))) return MMP_EINVAL;
    }
    // the contraction, where its constants fit the kernel arguments and LDS
    const int D = (M.bits() + 1) / 8 + 1;
    const int ksteps = (nmoduli + 7) / 8, col_tiles = (std::max(D + 6, 8 * lm) + 15) / 16;
    if (nmoduli >= kConMinModuli && nmoduli <= kConMaxModuli && (nmoduli + 1) * D <= con_digit_bytes(ksteps) &&
        (int64_t)con_lds(ksteps, col_tiles) <= kConLdsMax) {
      auto run = [&](auto steps) {
        constexpr int KS = decltype(steps)::value;
        ConArgs<KS> a;
        std::memset(&a, 0, offsetof(ConArgs<KS>, dig));
        a.s = nmoduli;
        a.limbs = limbs;
        a.ldc = ldc;
        a.m = m;
        a.n = n;
        a.ldo = ldo;
        a.out = out;
        a.digits = D;
        a.col_tiles = col_tiles;
        std::vector<Big> after(nmoduli + 1);  // p_t ... p_{s-1}
        for (int t = nmoduli - 1; t >= 0; t--) {
          after[t] = after[t + 1];
          after[t].mul(moduli[t]);
        }
        Big before;
        for (int t = 0; t < nmoduli; t++) {
          const uint64_t p = moduli[t], inv = rest_inv[t];
          a.C[t] = C[t];
          a.p[t] = (double)p;
          a.q[t] = 1.0 / (double)p;
          a.inv[t] = 2 * inv > p ? (double)((int64_t)inv - (int64_t)p) : (double)inv;
          signed_digits(product(before, after[t + 1]), D, a.dig + t * D);
          before.mul(p);
        }
        signed_digits(M, D, a.dig + nmoduli * D);
        return launch_contract<KS>(a, stream);
      };
      int e;
      switch (ksteps) {
        case 1: e = run(std::integral_constant<int, 1>{}); break;
        case 2: e = run(std::integral_constant<int, 2>{}); break;
        case 3: e = run(std::integral_constant<int, 3>{}); break;
        case 4: e = run(std::integral_constant<int, 4>{}); break;
        case 5: e = run(std::integral_constant<int, 5>{}); break;
        default: e = run(std::integral_constant<int, 6>{}); break;
      }
      return hip_status(e);
    }
    RecArgs a;
    std::memset(&a, 0, sizeof(a));
    a.s = nmoduli;
    a.limbs = limbs;
    a.ldc = ldc;
    a.m = m;
    a.n = n;
    a.ldo = ldo;
    a.out = out;
    for (int j = 0; j < nmoduli; j++) {
      a.C[j] = C[j];
      a.p[j] = (double)moduli[j];
      a.q[j] = 1.0 / (double)moduli[j];
      // (p_0 ... p_{j-1})^{-1} mod p_j, the inverse of M / p_j times what follows j
      const long double pinv = 1.0L / (long double)moduli[j];
      uint64_t inv = rest_inv[j];
      for (int i = j + 1; i < nmoduli; i++) inv = mulmod(inv, moduli[i] % moduli[j], moduli[j], pinv);
      a.inv[j] = (double)inv;
      a.act[j] = limbs_of_product(moduli, j, nmoduli);
    }
    int e;
    if (lm <= 2)
      e = launch_rec<2>(a, stream);
    else if (lm <= 4)
      e = launch_rec<4>(a, stream);
    else if (lm <= 8)
      e = launch_rec<8>(a, stream);
    else if (lm <= 16)
      e = launch_rec<16>(a, stream);
    else if (lm <= 28)
      e = launch_rec<28>(a, stream);
    else
      e = launch_rec<56>(a, stream);
    return hip_status(e);
  } catch (...) {
    return MMP_ENOMEM;
  }
}
