// Residue form of the INT8 product: C = A B mod p from the integer product's
// residues modulo N pairwise coprime moduli m_t <= 256.
//
// The signed base-256 digit form spends D^2 INT8 digit products on D-digit
// entries.  The integer product X = sum_l a_l b_l of centered entries
// (|a|, |b| <= p / 2) has |X| <= k (p/2)^2, so it is determined by its
// residues modulo M = m_0 ... m_{N-1} > 2 |X|, and each modulus costs ONE
// INT8 product of residue matrices: N = 11 at 36 bits and k = 4096 (25 digit
// products), 15 at 50 bits and k = 8192 (49).  It is the multimodular product
// of Section 5.2 with moduli of one INT8 word each, the low-precision words of
// Section 6.  Three launches:
//   1. rns_convert_kernel: every entry's N residues in [-128, 127], one int8
//      plane per modulus;
//   2. rns_gemm_kernel: N independent INT8 products with int32 accumulation;
//      each output leaves as its residue, one byte;
//   3. rns_combine_kernel: the N bytes of an output into X mod p by the Chinese
//      remainder theorem in binary64, C written once.
// Every step is exact; the bounds stand beside each step.  Measured on one
// MI355X, digit form -> this form: 4096^3 at 36 bits 1167 -> 777 us, 6001 x 5003
// x 7013 at 50 bits 7691 -> 2925 us, 512 x 512 x 131072 at 52 bits 1515 -> 1208
// us.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "mmp_internal.h"

namespace mmp {
namespace rns {

typedef int int4v __attribute__((ext_vector_type(4)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));

// A residue plane of R rows (A) or columns (B) by kp k-bytes is stored in 1 KB
// blocks of 16 rows by 64 k-bytes, chunk-major inside: byte (r, c) of a block
// sits at (c / 16) 256 + r 16 + c % 16.  Lane 16 q + r of a wave then owns 16
// consecutive bytes, which is both the 16x16x64 INT8 MFMA operand layout (row
// r, k-bytes 16 q ..) and what one global-to-LDS copy instruction writes: the
// LDS image is the global image, and operand reads are lane-linear (no bank
// conflicts, no swizzle).  Rows past the matrix in the last block are zero.
__host__ __device__ inline int64_t row_blocks(int64_t rows) { return (rows + 15) / 16; }

// Per-modulus constants of the conversion.  With the entry's signed base-256
// digits d_i, y = sum_i d_i w_i, w_i = 256^i mod m in [-128, 127], is congruent
// to the entry and |y| <= 8 2^14 = 2^17.  Reduction without conversions: the
// integer `bits` = bit pattern of the binary32 number O, O a multiple of 256 m
// just above 2^23 + 2^17, plus y is the pattern of O + y (one ulp is 1 in
// [2^23, 2^24)); fma(O + y, inv, magic) with magic = 1.5 2^23 - O / m (exact)
// rounds (O + y) inv - O / m to an integer c in the low bits, and y - c m is
// the residue.  inv = fl(1 / m) moves the quotient by less than
// 2^24 2^-24 / m = 1 / m, so |y - c m| < m / 2 + 1 <= 127.5 for m <= 253; for
// m = 255, fl(1 / 255) > 1 / 255 moves it one way only, into [-128, 127]; for
// m = 256 the scaling is exact.  Only the low byte is kept, and O,
// 2^22 m and the pattern's exponent are 0 mod 256, so low byte (y - c m) =
// low byte (bits + y - (2^22 + c) m).
struct ConvConst {
  int32_t wlo, whi;  // w_0..w_3, w_4..w_7 as bytes
  uint32_t bits;
  float inv, magic;
  int32_t negm;
};
struct ConvArgs {
  int n;  // moduli
  ConvConst c[kRnsMaxModuli];
};

// Signed base-256 digits of v as bytes: byte i of v + 0x80..80, less 128.
// WIDE: up to 8 digits; else v lies in (-2^30, 2^30) and has 4.
template <bool WIDE>
struct Digits {
  uint32_t lo, hi;
  __device__ __forceinline__ void set(int64_t v) {
    if constexpr (WIDE) {
      const uint64_t b = (uint64_t)v + 0x8080808080808080ull;
      lo = (uint32_t)b ^ 0x80808080u;
      hi = (uint32_t)(b >> 32) ^ 0x80808080u;
    } else {
      lo = ((uint32_t)(int32_t)v + 0x80808080u) ^ 0x80808080u;
      hi = 0;
    }
  }
};

template <bool WIDE>
__device__ __forceinline__ uint32_t residue_bits(const Digits<WIDE>& d, const ConvConst& c) {
  int y = (int)c.bits;
  if constexpr (WIDE) y = __builtin_amdgcn_sdot4((int)d.hi, c.whi, y, false);
  y = __builtin_amdgcn_sdot4((int)d.lo, c.wlo, y, false);
  const float t = fmaf(__builtin_bit_cast(float, y), c.inv, c.magic);
  return (uint32_t)(__mul24(__builtin_bit_cast(int, t), c.negm) + y);
}

// low bytes of a, b, c, d packed, a lowest
__device__ __forceinline__ uint32_t pack4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400), cd = __builtin_amdgcn_perm(d, c, 0x0c0c0400);
  return __builtin_amdgcn_perm(cd, ab, 0x05040100);
}

// Residues mod p as centered integers: x in [0, p) -> x or x - p (x > p / 2).
struct CenteredIn {
  const double* X;
  int64_t p, half;  // floor(p / 2)
  static constexpr bool kInteger = false;
  __device__ __forceinline__ int64_t operator()(double x) const {
    // x < 2^52 is an integer: x + 2^52 is exact and its significand is x
    const int64_t v = __double_as_longlong(x + 4503599627370496.0) - 0x4330000000000000ll;
    return v > half ? v - p : v;
  }
};
// Integers in [0, 2^62) taken as they are.
struct IntegerIn {
  const uint64_t* X;
  static constexpr bool kInteger = true;
  __device__ __forceinline__ int64_t operator()(uint64_t x) const { return (int64_t)x; }
};

// One wave's 16 x 64 block of A's planes (row-major source): coalesced 512-byte
// row reads, through wave-private LDS (rows of 66 entries: the 16 rows one
// 16-byte read pass touches fall in distinct banks), so that lane 16 q + r
// holds the 16 entries (r, 16 q ..) it stores as one 16-byte word per plane.
constexpr int kConvRow = 66;
template <class In, bool WIDE>
__device__ __forceinline__ void convert_rows(const In& in, const ConvArgs& ca, int64_t rows, int64_t cols, int64_t ld,
                                             int64_t kp, int8_t* out, int64_t blk, int64_t kblk, int t0, int t1, uint64_t* lds) {
  const int lane = threadIdx.x & 63;
  const int64_t k0 = kblk * 64, r0 = blk * 16;
  auto* X = in.X;
  decltype(+*X) x[16];
  const bool kin = k0 + lane < cols;
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = (kin && r0 + i < rows) ? X[(r0 + i) * ld + k0 + lane] : 0;
#pragma unroll
  for (int i = 0; i < 16; i++) lds[i * kConvRow + lane] = (uint64_t)in(x[i]);
  __builtin_amdgcn_wave_barrier();
  Digits<WIDE> d[16];
  const uint64_t* row = lds + (lane & 15) * kConvRow + (lane >> 4) * 16;
#pragma unroll
  for (int i = 0; i < 16; i++) d[i].set((int64_t)row[i]);
  const int64_t plane = row_blocks(rows) * 16 * kp;
  int8_t* dst = out + blk * 16 * kp + kblk * 1024 + lane * 16;
  for (int t = t0; t < t1; t++) {
    const ConvConst c = ca.c[t];
    int4v w;
#pragma unroll
    for (int g = 0; g < 4; g++)
      w[g] = (int)pack4(residue_bits(d[4 * g], c), residue_bits(d[4 * g + 1], c), residue_bits(d[4 * g + 2], c),
                        residue_bits(d[4 * g + 3], c));
    *(int4v*)(dst + t * plane) = w;
  }
}

// One wave's 64 columns by 16 k-rows of B's planes: lane n reads column n0 + n
// of 16 k-rows (512-byte rows, coalesced) and holds exactly one 16-byte word.
template <class In, bool WIDE>
__device__ __forceinline__ void convert_cols(const In& in, const ConvArgs& ca, int64_t krows, int64_t cols, int64_t ld,
                                             int64_t kp, int8_t* out, int64_t cblk, int64_t kblk, int q, int t0, int t1) {
  const int lane = threadIdx.x & 63;
  const int64_t k0 = kblk * 64 + q * 16, col = cblk * 64 + lane;
  auto* X = in.X;
  decltype(+*X) x[16];
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = (k0 + i < krows && col < cols) ? X[(k0 + i) * ld + col] : 0;
  Digits<WIDE> d[16];
#pragma unroll
  for (int i = 0; i < 16; i++) d[i].set(in(x[i]));
  if (col >= row_blocks(cols) * 16) return;
  const int64_t plane = row_blocks(cols) * 16 * kp;
  int8_t* dst = out + (col >> 4) * 16 * kp + kblk * 1024 + q * 256 + (lane & 15) * 16;
  for (int t = t0; t < t1; t++) {
    const ConvConst c = ca.c[t];
    int4v w;
#pragma unroll
    for (int g = 0; g < 4; g++)
      w[g] = (int)pack4(residue_bits(d[4 * g], c), residue_bits(d[4 * g + 1], c), residue_bits(d[4 * g + 2], c),
                        residue_bits(d[4 * g + 3], c));
    *(int4v*)(dst + t * plane) = w;
  }
}

// Both operands in one launch.  Bound by memory: 8 bytes read and N written an
// entry, 3.9 to 4.6 TB/s measured at 4096^3 (N = 11) and 512 x 512 x 131072
// (N = 16) where a large copy reaches 4.8.  Workgroups below `na` take four consecutive
// k-blocks of a 16-row group of A each, the rest one 64-column by 64-k part of
// B each.  gridDim.y shares the moduli out (each part reads the entries again)
// where the operands alone give too few workgroups to hide the chain of one
// modulus after another.
template <class In, bool WIDE>
__global__ __launch_bounds__(256) void rns_convert_kernel(const ConvArgs ca, In A, int64_t m, int64_t lda, In B,
                                                          int64_t n, int64_t ldb, int64_t k, int64_t kp,
                                                          int8_t* outA, int8_t* outB, int64_t na) {
  __shared__ uint64_t lds[4][16 * kConvRow];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int share = (ca.n + (int)gridDim.y - 1) / (int)gridDim.y;
  const int t0 = (int)blockIdx.y * share, t1 = min(t0 + share, ca.n);
  int64_t b = blockIdx.x;
  if (b < na) {
    const int64_t per_row = (kp + 255) / 256;  // groups of four k-blocks
    const int64_t kblk = (b % per_row) * 4 + wave;
    if (kblk * 64 < kp) convert_rows<In, WIDE>(A, ca, m, k, lda, kp, outA, b / per_row, kblk, t0, t1, lds[wave]);
  } else {
    b -= na;
    const int64_t cb = (n + 63) / 64;
    convert_cols<In, WIDE>(B, ca, k, n, ldb, kp, outB, b % cb, b / cb, wave, t0, t1);
  }
}

// The operands of many products in one launch.
struct ConvJob {
  const double *A, *B;
  int64_t p, m, n, k, lda, ldb, kp;
  int8_t *outA, *outB;
  int nmod, start, na;  // first workgroup, and how many of them take A
};
constexpr int kRnsBatch = 64;  // products of a launch
struct ConvBatch {
  ConvArgs ca;  // every modulus; a product takes the first nmod
  int njobs;
  ConvJob job[kRnsBatch];
};

// the last product whose start is at most w (w and the starts uniform)
template <class Jobs, class F>
__device__ __forceinline__ int find_start(const Jobs& jobs, int njobs, int w, F start) {
  int lo = 0, hi = njobs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) / 2;
    if (start(jobs[mid]) <= w)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

template <bool WIDE>
__device__ __forceinline__ void convert_job(const ConvBatch& b, const ConvJob& j, int64_t w, int wave, uint64_t* lds) {
  const CenteredIn A{j.A, j.p, j.p / 2}, B{j.B, j.p, j.p / 2};
  if (w < j.na) {
    const int64_t per_row = (j.kp + 255) / 256, kblk = (w % per_row) * 4 + wave;
    if (kblk * 64 < j.kp)
      convert_rows<CenteredIn, WIDE>(A, b.ca, j.m, j.k, j.lda, j.kp, j.outA, w / per_row, kblk, 0, j.nmod, lds);
  } else {
    const int64_t cb = (j.n + 63) / 64;
    convert_cols<CenteredIn, WIDE>(B, b.ca, j.k, j.n, j.ldb, j.kp, j.outB, (w - j.na) % cb, (w - j.na) / cb, wave, 0,
                                   j.nmod);
  }
}

__global__ __launch_bounds__(256) void rns_convert_batch_kernel(const ConvBatch b) {
  __shared__ uint64_t lds[4][16 * kConvRow];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const ConvJob& j = b.job[find_start(b.job, b.njobs, (int)blockIdx.x, [](const ConvJob& x) { return x.start; })];
  if (j.p >> 31)
    convert_job<true>(b, j, (int)blockIdx.x - j.start, wave, lds[wave]);
  else
    convert_job<false>(b, j, (int)blockIdx.x - j.start, wave, lds[wave]);
}

// ---------------------------------------------------------------- products

struct GemmConst {
  uint32_t mul;   // 2^16 mod m in the high half, 1 in the low half
  uint32_t bits;  // bit pattern of O = the first multiple of 256 m from 2^23 on
  float inv, magic;
  int32_t negm;
  int32_t bias;   // accumulator start: the largest multiple of m up to 2^30
};
struct GemmJob {
  const int8_t* Ad;
  const int8_t* Bd;
  int8_t* res;
  int64_t kp;
  int ablk, bblk;         // 16-row blocks of A, 16-column blocks of B
  int tiles_m, tiles_n;
  int n, splits;
  int stages, per_split;  // 64-k stages in all, and per k-range
  int start;              // first item
};
// One product, or JOBS of one tile shape whose items follow one another.
template <int JOBS>
struct RnsGemmArgs {
  int njobs, total;  // total: items
  GemmConst c[kRnsMaxModuli];
  GemmJob job[JOBS];
};

template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// dword 3 of a raw buffer resource
constexpr int kBufferWord3 = 0x00020000;

// workgroup barrier that leaves copies in flight; the empty asm statements keep
// the compiler from moving LDS accesses or copies across it
__device__ __forceinline__ void lds_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Workgroup tile: WM x WN waves of XB x 4 MFMA tiles of 16 x 16 outputs.
//   large: 2 x 4 waves of 8 x 4 (256 x 256 outputs, 512 threads, one per CU);
//   small: 2 x 2 waves of 4 x 4 (128 x 128, 256 threads, two per CU).
// What bounds it: power.  A stage of the large tile copies 32 KB for 256 MFMAs
// of 16 cycles on 4 SIMDs (32 bytes a cycle and CU from L2; 128 x 128 tiles take
// twice that, the L1's whole rate, so they serve only products with too few
// large tiles).  8192^3 with 15 moduli takes 5.9 ms, 2.8e15 operations a second,
// on uniform residues and 4.6 ms on zeros, the clock falling from 2.4 to about
// 1.9 GHz.  What it measured on the way (uniform / zeros): copies issued together
// ahead of the MFMAs 6.4 to 6.6 / 5.4 ms; two halves of the workgroup taking turns at
// reads and MFMAs 6.65 / 5.2; four waves of 128 x 128 outputs in 512 registers
// with the copies among the MFMAs 5.9 / 4.8; 32x32x32 MFMAs 6.9 / 4.9.
template <int WM_, int WN_, int XB_, int YB_, int RING_>
struct RnsShape {
  static constexpr int WM = WM_, WN = WN_, XB = XB_, YB = YB_;
  static constexpr int PER = (XB + YB + XB - 1) / XB;  // operand reads per group of YB MFMAs
  static constexpr int NW = WM * WN, THREADS = 64 * NW;
  static constexpr int MB = WM * XB, NB = WN * YB;  // 16-row / 16-column blocks
  static constexpr int BM = 16 * MB, BN = 16 * NB;
  static constexpr int CA = MB / NW, CB = NB / NW;  // copies per wave and stage
  static constexpr int RING = RING_, AHEAD = RING_ - 1;
  static constexpr int STAGE = (MB + NB) * 1024;
  static constexpr int GROUPS = 160 * 1024 / (RING * STAGE);  // per CU, by LDS
  static constexpr int64_t TILE_BYTES = (int64_t)BM * BN;
  static_assert(CA * NW == MB && CB * NW == NB, "whole copies per wave");
};
using RnsLarge = RnsShape<2, 4, 8, 4, 4>;
using RnsSmall = RnsShape<2, 2, 4, 4, 4>;

// A persistent grid over (modulus, k-range, tile) items.  The four-stage copy
// ring runs across items: three stages are always in flight, also through an
// item's epilogue, so no item waits out a copy latency at its start.
template <class S, int JOBS>
__global__ __launch_bounds__(S::THREADS, S::THREADS *S::GROUPS / 256) void rns_gemm_kernel(const RnsGemmArgs<JOBS> a) {
  constexpr int XB = S::XB, YB = S::YB, CA = S::CA, CB = S::CB;
  constexpr int PER = S::PER;
  __shared__ __attribute__((aligned(1024))) int8_t lds[S::RING][S::STAGE];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wv / S::WN, wn = wv % S::WN;
  const int total = a.total;
  const int G = (int)gridDim.x;
  // workgroups are dispatched round-robin over the 8 XCDs: give each XCD a
  // contiguous run of every round's items, so that neighbours share panels in L2
  int first;
  {
    const int per = G / 8, rem = G % 8, xcd = (int)blockIdx.x % 8, loc = (int)blockIdx.x / 8;
    first = (xcd < rem) ? xcd * (per + 1) + loc : rem * (per + 1) + (xcd - rem) * per + loc;
  }
  struct Item {
    int j, t, s, tile, tm, tn, st0, nst;
  };
  auto div = [](int x, int y) { return __builtin_amdgcn_readfirstlane(x / y); };  // both uniform
  auto item_of = [&](int it) {
    Item x;
    x.j = JOBS == 1 ? 0 : __builtin_amdgcn_readfirstlane(
                              find_start(a.job, a.njobs, it, [](const GemmJob& g) { return g.start; }));
    const GemmJob& g = a.job[x.j];
    const int tiles = g.tiles_m * g.tiles_n, local = it - g.start;
    const int ts = div(local, tiles);
    x.tile = local - ts * tiles;
    x.t = div(ts, g.splits);
    x.s = ts - x.t * g.splits;
    // groups of 8 tile rows, column by column
    const int group = 8 * g.tiles_n, gid = div(x.tile, group), f = gid * 8;
    const int gm = min(g.tiles_m - f, 8), in = x.tile - gid * group;
    x.tn = div(in, gm);
    x.tm = f + in - x.tn * gm;
    x.st0 = x.s * g.per_split;
    x.nst = min(g.per_split, g.stages - x.st0);
    return x;
  };

  // Copy cursor: where the next stage's copies come from.  Buffer copies with
  // one resource per operand and item and a scalar offset per copy: with
  // global_load_lds the compiler drains every outstanding LDS read at each
  // wait for one (it takes the copy for a flat access to LDS), which undid the
  // read-ahead below.
  __amdgpu_buffer_rsrc_t ra, rb;
  uint32_t off[CA + CB];
  int c_item = first, c_left = 0;
  auto aim = [&](int it) {
    const Item x = item_of(it);
    const GemmJob& g = a.job[x.j];
    const int64_t row = g.kp * 16, planeA = (int64_t)g.ablk * row, planeB = (int64_t)g.bblk * row;
    c_left = x.nst;
    ra = __builtin_amdgcn_make_buffer_rsrc((void*)(g.Ad + x.t * planeA), (short)0, (int)(uint32_t)planeA, kBufferWord3);
    rb = __builtin_amdgcn_make_buffer_rsrc((void*)(g.Bd + x.t * planeB), (short)0, (int)(uint32_t)planeB, kBufferWord3);
#pragma unroll
    for (int e = 0; e < CA; e++)
      off[e] = (uint32_t)(min(x.tm * S::MB + wv * CA + e, g.ablk - 1) * row) + (uint32_t)x.st0 * 1024u;
#pragma unroll
    for (int e = 0; e < CB; e++)
      off[CA + e] = (uint32_t)(min(x.tn * S::NB + wv * CB + e, g.bblk - 1) * row) + (uint32_t)x.st0 * 1024u;
  };
  // the cursor's stage, one step on: called once before each stage's copies
  auto advance = [&]() {
    if (c_left == 0) {
      c_item += G;
      if (c_item < total)
        aim(c_item);
      else
        c_left = 0x7fffffff;  // past the last item: copies of bytes that nothing reads
      // its scalar loads are done here, so that waits for operand reads in the
      // stage loop count LDS reads alone and need not drain them all
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    }
    c_left--;
  };
  auto copy = [&](int e, int buf) {
    const int blk = e < CA ? wv * CA + e : S::MB + wv * CB + (e - CA);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(e < CA ? ra : rb,
                                             (__attribute__((address_space(3))) void*)&lds[buf][blk * 1024], 16,
                                             lane * 16, (int)off[e], 0, 0);
    off[e] += 1024;
  };

  if (first >= total) return;  // uniform
  aim(first);
#pragma unroll
  for (int i = 0; i < S::AHEAD; i++) {
    advance();
#pragma unroll
    for (int e = 0; e < CA + CB; e++) copy(e, i);
  }

  const int8_t* const la = &lds[0][(wm * XB) * 1024 + lane * 16];
  const int8_t* const lb = &lds[0][(S::MB + wn * YB) * 1024 + lane * 16];
  int buf = 0, after = 0;  // after: stages since an epilogue whose stores may still be counted
  int4v acc[XB][YB];
  // One stage.  b0, a0: its B fragments and its first two A fragments, read
  // ahead; b1, a1: the next stage's.
  auto stage = [&](const int4v (&b0)[YB], const int4v (&a0)[2], int4v (&b1)[YB], int4v (&a1)[2]) {
    advance();
    // This wave's copies of the NEXT stage are complete once at most the
    // later stages' copies (and the stores of an epilogue that ran since)
    // are outstanding: vector memory operations retire in issue order.  The
    // barrier extends that to every wave and ends the reads of the buffer
    // that the next copies overwrite.
    if (after > 0)
      wait_vm<(S::RING - 3) * (CA + CB) + XB * YB / 4>();
    else
      wait_vm<(S::RING - 3) * (CA + CB)>();
    after--;
    lds_fence();
    const int fill = buf == 0 ? S::AHEAD : buf - 1;
    const int next = buf + 1 == S::RING ? 0 : buf + 1;
    const int8_t* const sa = la + buf * S::STAGE;
    const int8_t* const na = la + next * S::STAGE;
    const int8_t* const nb = lb + next * S::STAGE;
    int4v af[XB];
    af[0] = a0[0];
    af[1] = a0[1];
#pragma unroll
    for (int i = 0; i < XB; i++) {
#pragma unroll
      for (int h = i * PER; h < (i + 1) * PER; h++) {
        if (h < XB - 2)
          af[h + 2] = *(const int4v*)(sa + (h + 2) * 1024);
        else if (h < XB - 2 + YB)
          b1[h - (XB - 2)] = *(const int4v*)(nb + (h - (XB - 2)) * 1024);
        else if (h < XB + YB)
          a1[h - (XB + YB - 2)] = *(const int4v*)(na + (h - (XB + YB - 2)) * 1024);
      }
#pragma unroll
      for (int e = i * (CA + CB) / XB; e < (i + 1) * (CA + CB) / XB; e++) copy(e, fill);
      // output layout: a lane holds four consecutive rows of column lane & 15
#pragma unroll
      for (int j = 0; j < YB; j++)
        acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af[i], b0[j], acc[i][j], 0, 0, 0);
    }
    // keep that order: a group's reads and copies between its MFMAs
#pragma unroll
    for (int i = 0; i < XB; i++) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, YB / 2 - 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, PER - 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, YB / 4, 0);
      __builtin_amdgcn_sched_group_barrier(0x010, (CA + CB) / XB, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, YB / 4, 0);
    }
    buf = next;
  };
  int4v bp[YB], ap[2], bq[YB], aq[2];
  wait_vm<0>();
  lds_fence();
#pragma unroll
  for (int j = 0; j < YB; j++) bp[j] = *(const int4v*)(lb + j * 1024);
  ap[0] = *(const int4v*)la;
  ap[1] = *(const int4v*)(la + 1024);
  for (int it = first; it < total; it += G) {
    const Item x = item_of(it);
    const GemmConst c = a.c[x.t];
#pragma unroll
    for (int i = 0; i < XB; i++)
#pragma unroll
      for (int j = 0; j < YB; j++) acc[i][j] = (int4v){c.bias, c.bias, c.bias, c.bias};
    int st = 0;
    for (; st + 1 < x.nst; st += 2) {
      stage(bp, ap, bq, aq);
      stage(bq, aq, bp, ap);
    }
    if (st < x.nst) {
      stage(bp, ap, bq, aq);
#pragma unroll
      for (int j = 0; j < YB; j++) bp[j] = bq[j];
      ap[0] = aq[0];
      ap[1] = aq[1];
    }
    // Each output's residue.  An item has at most 1024 stages, so its sum lies
    // within 2^30 of zero and the biased accumulator in [0, 2^31]:
    // y = hi (2^16 mod m) + lo <= 2^15 225 + 2^16 < 2^23 - 2^16 is congruent to
    // it, and is reduced as in the conversion, from O just above 2^23.
    const GemmJob& g = a.job[x.j];
    int8_t* dst = g.res + ((int64_t)(x.t * g.splits + x.s) * (g.tiles_m * g.tiles_n) + x.tile) * S::TILE_BYTES + wv * XB * YB * 256 + lane * 16;
#pragma unroll
    for (int i = 0; i < XB * YB / 4; i++) {
      int4v w;
#pragma unroll
      for (int j = 0; j < 4; j++) {
        uint32_t r[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const uint32_t y = __builtin_amdgcn_udot2(__builtin_bit_cast(us2, (uint32_t)acc[i / (YB / 4)][i % (YB / 4) * 4 + j][e]),
                                                    __builtin_bit_cast(us2, c.mul), c.bits, false);
          const float f = fmaf(__builtin_bit_cast(float, y), c.inv, c.magic);
          r[e] = (uint32_t)(__mul24(__builtin_bit_cast(int, f), c.negm) + (int)y);
        }
        w[j] = (int)pack4(r[0], r[1], r[2], r[3]);
      }
      *(int4v*)(dst + i * 1024) = w;
    }
    after = S::RING - 2;
  }
  wait_vm<0>();  // no copy may land in LDS after the workgroup has left it
}

// ---------------------------------------------------------------- recombination

// Where a wave's outputs lie: unit u of a tile is 16 rows by 64 columns, 1 KB of
// residue bytes per modulus and k-range.  Lane 16 g + c holds, in word y, rows
// 4 g .. 4 g + 3 of column 16 y + c: a store over the lanes writes whole 128-byte
// pieces of four rows.
struct RnsOut {
  const int8_t* res;
  int64_t m, n, ldc;
  int tiles_m, tiles_n, nmod, splits;
};
struct Unit {
  const int8_t* src;
  int64_t step;  // to the next (modulus, k-range)
  int64_t row, col;
  bool any;      // part of the unit lies inside the output
};
template <class S>
__device__ __forceinline__ Unit unit_of(const RnsOut& a, int64_t unit, int lane) {
  constexpr int UNITS = S::NW * S::XB * S::YB / 4;
  const int tiles = a.tiles_m * a.tiles_n;
  const int tile = (int)(unit / UNITS), u = (int)(unit % UNITS);
  const int group = 8 * a.tiles_n, gid = tile / group, first = gid * 8;
  const int gm = min(a.tiles_m - first, 8), in = tile - gid * group;
  const int tm = first + in % gm, tn = in / gm;
  const int w = u / (S::XB * S::YB / 4), x = u % (S::XB * S::YB / 4) / (S::YB / 4), y4 = u % (S::YB / 4);
  const int64_t row0 = (int64_t)tm * S::BM + ((w / S::WN) * S::XB + x) * 16;
  const int64_t col0 = (int64_t)tn * S::BN + (w % S::WN) * S::YB * 16 + y4 * 64;
  Unit r;
  r.src = a.res + (int64_t)tile * S::TILE_BYTES + u * 1024 + lane * 16;
  r.step = (int64_t)tiles * S::TILE_BYTES;
  r.row = row0 + (lane >> 4) * 4;
  r.col = col0 + (lane & 15);
  r.any = row0 < a.m && col0 < a.n;  // uniform
  return r;
}

// Feeds add(r, t) the residues mod m_t of this lane's 4 W outputs (summed over
// the k-ranges), W words a (modulus, k-range) pair from `src` on, with kLoads
// pairs in flight.
template <int W, class Add>
__device__ __forceinline__ void each_modulus(const int8_t* src, int64_t step, int nmod, int splits, Add add) {
  typedef int words __attribute__((ext_vector_type(W)));
  constexpr int kLoads = 8;
  const int total = nmod * splits;
  words v[kLoads];
#pragma unroll
  for (int i = 0; i < kLoads; i++) v[i] = __builtin_nontemporal_load((const words*)(src + min(i, total - 1) * step));
  int sum[4 * W];
  int t = 0, s = 0;
  for (int j = 0; j < total; j += kLoads) {
    words w[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; i++) w[i] = v[i];
    if (j + kLoads < total) {
#pragma unroll
      for (int i = 0; i < kLoads; i++)
        v[i] = __builtin_nontemporal_load((const words*)(src + min(j + kLoads + i, total - 1) * step));
    }
#pragma unroll
    for (int h = 0; h < kLoads; h++) {
      if (j + h >= total) break;  // uniform
      int r[4 * W];
#pragma unroll
      for (int i = 0; i < 4 * W; i++) r[i] = (int)(int8_t)(w[h][i / 4] >> (8 * (i % 4)));
      if (splits == 1) {
        add(r, j + h);
        continue;
      }
#pragma unroll
      for (int i = 0; i < 4 * W; i++) sum[i] = s == 0 ? r[i] : sum[i] + r[i];
      if (++s == splits) {
        add(sum, t++);
        s = 0;
      }
    }
  }
}

struct CombineArgs {
  RnsOut o;
  double* C;
  double p, q;
  double mhi, mlo;  // M mod p as mhi 2^26 + mlo
  double whi[kRnsMaxModuli], wlo[kRnsMaxModuli];  // W_t mod p as whi 2^26 + wlo
  double f[kRnsMaxModuli];                        // W_t / M mod 1
};

__device__ __forceinline__ double reduce_near(double x, double p, double q) {
  return fma(-floor(fma(x, q, 0.5)), p, x);
}

// With inv_t = (M / m_t)^-1 mod m_t (|inv_t| <= m_t / 2) and W_t = inv_t M / m_t,
// X = sum_t r_t W_t - h M for the one integer h that puts X in (-M/2, M/2):
// h = round(sum_t r_t inv_t / m_t).  The planner keeps |X| <= M 2^-1.05, so the
// sum lies at least 0.017 from a rounding boundary; its binary64 error is below
// 2^-30.  With residues summed over at most 64 k-ranges, |r_t| <= 2^13:
//   hi = sum_t r_t whi_t - h mhi, |hi| <= 20 2^13 2^25 + 2^17 2^25 < 2^44,
//   lo = sum_t r_t wlo_t - h mlo, |lo| < 2^45,
// all exact, and X = 2^26 hi + lo mod p.  hi is reduced to p/2 + 1 of zero,
// 2^26 times that is exact (a power of two) and its quotient is below 2^26.1,
// so it reduces to p/2 + 1 of zero again; adding lo stays below 2^53 and one
// complete Alg. 1 ends it.  Bound by memory: N bytes read and 8 written an output,
// 5.1 TB/s at 8192^2 outputs and 15 moduli.
constexpr int kOutRow = 66;
template <class S>
__device__ __forceinline__ void combine_unit(const CombineArgs& a, int64_t unit, double (&lds)[4][16 * kOutRow]) {
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Unit u = unit_of<S>(a.o, unit + wv, lane);
  if (!u.any) return;
  double hi[16], lo[16], g[16];
#pragma unroll
  for (int i = 0; i < 16; i++) hi[i] = lo[i] = g[i] = 0.0;
  each_modulus<4>(u.src, u.step, a.o.nmod, a.o.splits, [&](const int (&r)[16], int t) {
    const double wh = a.whi[t], wl = a.wlo[t], f = a.f[t];
#pragma unroll
    for (int i = 0; i < 16; i++) {
      const double d = (double)r[i];
      hi[i] = fma(d, wh, hi[i]);
      lo[i] = fma(d, wl, lo[i]);
      g[i] = fma(d, f, g[i]);
    }
  });
  const double p = a.p, q = a.q;
#pragma unroll
  for (int y = 0; y < 4; y++)
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int i = 4 * y + e;
      const double h = rint(g[i]);
      const double H = fma(-h, a.mhi, hi[i]), L = fma(-h, a.mlo, lo[i]);
      const double t = reduce_near(67108864.0 * reduce_near(H, p, q), p, q) + L;
      double d = fma(-floor(t * q), p, t);
      d = (d >= p) ? d - p : d;
      d = (d < 0.0) ? d + p : d;
      lds[wv][((lane >> 4) * 4 + e) * kOutRow + 16 * y + (lane & 15)] = d + 0.0;  // +0.0: canonical zero
    }
  __builtin_amdgcn_wave_barrier();
  // whole rows of 64 columns, 512 contiguous bytes a store (stores of the lanes'
  // own values, four pieces of 128 bytes, took 74 us at 4096^2 outputs against
  // 62).  Streaming ones or not is within 10% either way, on rows that start on
  // cache lines as on others: 15 moduli, streaming against not, 4096^2 outputs 87
  // and 88 us, 4096 x 4104 74 and 78, 8192^2 291 and 280, 6001 x 5003 155 and 142.
  const int64_t row0 = u.row - (lane >> 4) * 4, col = u.col - (lane & 15) + lane;
  const int rows = (int)min((int64_t)16, a.o.m - row0);
  double* const out = a.C + row0 * a.o.ldc + col;
  if (col < a.o.n)
    for (int r = 0; r < rows; r++) __builtin_nontemporal_store(lds[wv][r * kOutRow + lane], out + r * a.o.ldc);
}

template <class S>
__global__ __launch_bounds__(256) void rns_combine_kernel(const CombineArgs a) {
  __shared__ double lds[4][16 * kOutRow];
  combine_unit<S>(a, (int64_t)blockIdx.x * 4, lds);
}

// Several products of one tile shape.
constexpr int kCombineBatch = 16;
struct CombineBatch {
  int njobs;
  int start[kCombineBatch];  // first workgroup
  CombineArgs job[kCombineBatch];
};
template <class S>
__global__ __launch_bounds__(256) void rns_combine_batch_kernel(const CombineBatch b) {
  __shared__ double lds[4][16 * kOutRow];
  const int j = find_start(b.start, b.njobs, (int)blockIdx.x, [](int x) { return x; });
  combine_unit<S>(b.job[j], (int64_t)((int)blockIdx.x - b.start[j]) * 4, lds);
}

// The multi-modular product's recombination: the same residues, of products of
// integers in [0, 2^62), into X itself as NG limbs of base 2^b, and each of up
// to 64 primes reduces those.
constexpr int kCrtLimbs = 6;
struct CrtCombineArgs {
  RnsOut o;
  int nprimes;
  int lines;           // every C's rows start on 128-byte lines
  double base, rbase;  // 2^b, 2^-b
  double f[kRnsMaxModuli], w[kRnsMaxModuli][kCrtLimbs], M[kCrtLimbs];
  double p[kMaxPrimesCrt], q[kMaxPrimesCrt];
  double* C[kMaxPrimesCrt];
};

// Limb j of X is sum_t r_t W_t,j - h M_j (the top limb of W_t signed, the others
// in [0, 2^b)), below 20 64 2^7 2^b + 2^17 2^b; the launcher keeps that below
// 2^53.  Carries rounded to nearest leave |limb| <= 2^(b-1) + 1, the top one
// below 2^b.  Per prime, Horner's rule with the base 2^b over the limbs as they
// are: |t| <= p + 2^b at every step and the quotient argument 2^b (1 + 2^b / p)
// stays below 2^50 (launcher), so its error is below 1/4, the reduced value lies
// within 3/4 p + 1 of zero and every step is exact; the last reduction's quotient
// is below 2^26, which leaves it within p/2 + 1 of zero, and adding p to a
// negative one ends it.  Bound by the primes' outputs: 32 of them at 2048^2 are
// 1.07 GB.
constexpr int kCrtRow = 34;
template <class S, int NG>
__global__ __launch_bounds__(256) void rns_crt_combine_kernel(const CrtCombineArgs a) {
  __shared__ double lds[4][16 * kCrtRow];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // a wave takes half a unit, two of the four words: its limbs then leave
  // registers for two waves a SIMD and more
  const int64_t id = (int64_t)blockIdx.x * 4 + wv;
  const int half = (int)(id & 1);
  const Unit u = unit_of<S>(a.o, id >> 1, lane);
  const int64_t col = u.col + 32 * half;
  if (!u.any || col - (lane & 15) >= a.o.n) return;
  double g[8], G[8][NG];
#pragma unroll
  for (int i = 0; i < 8; i++) {
    g[i] = 0.0;
#pragma unroll
    for (int j = 0; j < NG; j++) G[i][j] = 0.0;
  }
  each_modulus<2>(u.src + 8 * half, u.step, a.o.nmod, a.o.splits, [&](const int (&r)[8], int t) {
    const double f = a.f[t];
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const double d = (double)r[i];
      g[i] = fma(d, f, g[i]);
#pragma unroll
      for (int j = 0; j < NG; j++) G[i][j] = fma(d, a.w[t][j], G[i][j]);
    }
  });
  const double base = a.base, rbase = a.rbase;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const double h = rint(g[i]);
#pragma unroll
    for (int j = 0; j < NG; j++) G[i][j] = fma(-h, a.M[j], G[i][j]);
#pragma unroll
    for (int j = 0; j + 1 < NG; j++) {
      const double c = rint(G[i][j] * rbase);
      G[i][j] = fma(-c, base, G[i][j]);
      G[i][j + 1] += c;
    }
  }
  // whole rows through LDS as in rns_combine_kernel, two of 32 columns a store
  const int64_t row0 = u.row - (lane >> 4) * 4 + (lane >> 5), col0 = col - (lane & 15) + (lane & 31);
  const int rows = col0 < a.o.n ? (int)min((int64_t)16, a.o.m - row0) : 0;
  const int64_t off = row0 * a.o.ldc + col0;
  for (int pi = 0; pi < a.nprimes; pi++) {
    const double p = a.p[pi], q = a.q[pi];
    double* const out = a.C[pi] + off;
#pragma unroll
    for (int y = 0; y < 2; y++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int i = 4 * y + e;
        double t = G[i][NG - 1];
#pragma unroll
        for (int j = NG - 2; j >= 0; j--) t = reduce_near(base * t, p, q) + G[i][j];
        const double d = reduce_near(t, p, q);
        lds[wv][((lane >> 4) * 4 + e) * kCrtRow + 16 * y + (lane & 15)] = (d < 0.0 ? d + p : d) + 0.0;
      }
    __builtin_amdgcn_wave_barrier();
    double v[8];
#pragma unroll
    for (int r = 0; r < 8; r++) v[r] = lds[wv][(2 * r + (lane >> 5)) * kCrtRow + (lane & 31)];
    // streaming stores where rows start on cache lines (32 primes at 2048^2: 231 us
    // against 244); on others they write parts of lines to memory (2521 x 2750, 5
    // primes: 131 us against 97)
    if (a.lines) {
#pragma unroll
      for (int r = 0; r < 8; r++)
        if (2 * r < rows) __builtin_nontemporal_store(v[r], out + 2 * r * a.o.ldc);
    } else {
#pragma unroll
      for (int r = 0; r < 8; r++)
        if (2 * r < rows) out[2 * r * a.o.ldc] = v[r];
    }
    __builtin_amdgcn_wave_barrier();
  }
}

}  // namespace rns
}  // namespace mmp
