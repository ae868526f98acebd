// Residue form of the INT8 product (rns_kernel.h): moduli, constants, the
// choice of tile and k-ranges, and the three launches.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <type_traits>
#include <vector>

#include "rns_kernel.h"

namespace mmp {

namespace {

// The largest pairwise coprime integers up to 256, greedily.
const int kModuli[kRnsMaxModuli] = {256, 255, 253, 251, 247, 241, 239, 233, 229, 227,
                                    223, 217, 211, 199, 197, 193, 191, 181, 179, 173};

int inv_mod_small(int x, int m) {
  x %= m;
  for (int i = 1; i < m; i++)
    if ((int64_t)x * i % m == 1) return i;
  return 0;
}

uint32_t float_bits(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  return u;
}

// O = the first multiple of 256 m at or above `from`, as a binary32 pattern,
// and the constants that reduce O + y (rns_kernel.h, ConvConst).
void reduction(int m, int64_t from, uint32_t* bits, float* inv, float* magic) {
  const int64_t step = 256 * (int64_t)m, O = (from + step - 1) / step * step;
  *bits = float_bits((float)O);
  *inv = 1.0f / (float)m;
  *magic = (float)(12582912 - O / m);
}

// Everything that depends on the moduli alone, made once.
struct Tables {
  rns::ConvConst conv[kRnsMaxModuli];
  rns::GemmConst gemm[kRnsMaxModuli];
  int inv[kRnsMaxModuli + 1][kRnsMaxModuli];  // [n][t]: (M / m_t)^-1 mod m_t for M = m_0 .. m_(n-1), within m_t / 2
  double log2M[kRnsMaxModuli + 1];
  Tables() {
    log2M[0] = 0.0;
    for (int t = 0; t < kRnsMaxModuli; t++) {
      const int m = kModuli[t];
      log2M[t + 1] = log2M[t] + std::log2((double)m);
      rns::ConvConst& c = conv[t];
      uint32_t w[2] = {0, 0};
      int64_t pw = 1;
      for (int i = 0; i < 8; i++) {
        int s = (int)(pw % m);
        if (s > 127) s -= m;
        w[i / 4] |= (uint32_t)(uint8_t)s << (8 * (i % 4));
        pw = pw * 256 % m;
      }
      c.wlo = (int32_t)w[0];
      c.whi = (int32_t)w[1];
      c.negm = -m;
      reduction(m, (1 << 23) + (1 << 17), &c.bits, &c.inv, &c.magic);
      rns::GemmConst& g = gemm[t];
      g.mul = (uint32_t)(65536 % m) << 16 | 1u;
      g.negm = -m;
      g.bias = (1 << 30) / m * m;
      reduction(m, 1 << 23, &g.bits, &g.inv, &g.magic);
    }
    for (int n = 0; n <= kRnsMaxModuli; n++)
      for (int t = 0; t < n; t++) {
        const int m = kModuli[t];
        int x = 1;
        for (int j = 0; j < n; j++)
          if (j != t) x = x * (kModuli[j] % m) % m;
        const int i = inv_mod_small(x, m);
        inv[n][t] = 2 * i > m ? i - m : i;
      }
  }
};
const Tables& tables() {
  static const Tables t;
  return t;
}

uint64_t mulmod_u64(uint64_t x, uint64_t y, uint64_t p) { return (uint64_t)((unsigned __int128)x * y % p); }

void split26(uint64_t w, uint64_t p, double* hi, double* lo) {
  // the representative within p / 2 of zero, as hi 2^26 + lo, 0 <= lo < 2^26
  const int64_t s = w > p / 2 ? (int64_t)w - (int64_t)p : (int64_t)w;
  const int64_t h = s >> 26;
  *hi = (double)h;
  *lo = (double)(s - h * (1 << 26));
}

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

int current_cus() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) dev = 0;
  if (dev < 64 && cache[dev].load(std::memory_order_relaxed) > 0) return cache[dev].load(std::memory_order_relaxed);
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
  if (dev < 64) cache[dev].store(cus, std::memory_order_relaxed);
  return cus;
}

// Residue planes of both operands.  WIDE: entries of more than 4 digits.
template <class In, bool WIDE>
int launch_convert(const RnsPlan& r, const In& A, int64_t m, int64_t lda, const In& B, int64_t n, int64_t ldb,
                   int64_t k, int8_t* planes, hipStream_t s) {
  using namespace rns;
  ConvArgs ca;
  ca.n = r.n;
  std::memcpy(ca.c, tables().conv, sizeof(ca.c));
  const int64_t kp = cdiv(k, 64) * 64;
  const int64_t na = row_blocks(m) * cdiv(kp, 256), nb = cdiv(n, 64) * (kp / 64);
  // moduli in up to four parts while the grid is under four workgroups a CU
  unsigned parts = 1;
  while (parts < 4 && (na + nb) * parts < 1024) parts *= 2;
  TimerTok* t = timer_begin("rns_convert");
  hipExtLaunchKernelGGL((rns_convert_kernel<In, WIDE>), dim3((unsigned)(na + nb), parts), dim3(256), 0, s,
                        timer_start(t), timer_stop(t), 0, ca, A, m, lda, B, n, ldb, k, kp, planes, planes + r.bytes_a,
                        na);
  const int e = (int)hipGetLastError();
  timer_commit(t, e);
  return e;
}

// One product's entry of the GEMM's table (its items from `start` on; returns
// how many), and where its residues lie.
template <class S>
int64_t gemm_job(const RnsPlan& r, int64_t m, int64_t n, int64_t k, int8_t* planes, int64_t start, rns::GemmJob* g,
                 rns::RnsOut* o) {
  using namespace rns;
  g->Ad = planes;
  g->Bd = planes + r.bytes_a;
  g->res = planes + r.bytes_a + r.bytes_b;
  g->kp = cdiv(k, 64) * 64;
  g->ablk = (int)row_blocks(m);
  g->bblk = (int)row_blocks(n);
  g->tiles_m = (int)cdiv(m, S::BM);
  g->tiles_n = (int)cdiv(n, S::BN);
  g->n = r.n;
  g->splits = r.splits;
  g->stages = (int)(g->kp / 64);
  g->per_split = (int)cdiv(g->stages, r.splits);
  g->start = (int)start;
  o->res = g->res;
  o->m = m;
  o->n = n;
  o->tiles_m = g->tiles_m;
  o->tiles_n = g->tiles_n;
  o->nmod = r.n;
  o->splits = r.splits;
  return (int64_t)g->tiles_m * g->tiles_n * r.n * r.splits;
}

template <class S, int JOBS>
int launch_gemm(rns::RnsGemmArgs<JOBS>& a, hipStream_t s) {
  std::memcpy(a.c, tables().gemm, sizeof(a.c));
  const int64_t grid = std::min<int64_t>(a.total, (int64_t)current_cus() * S::GROUPS);
  TimerTok* t = timer_begin(JOBS == 1 ? "rns_gemm" : "rns_batch_gemm");
  hipExtLaunchKernelGGL((rns::rns_gemm_kernel<S, JOBS>), dim3((unsigned)grid), dim3(S::THREADS), 0, s, timer_start(t),
                        timer_stop(t), 0, a);
  const int e = (int)hipGetLastError();
  timer_commit(t, e);
  return e;
}

// The INT8 products of one product.
template <class S>
int launch_products(const RnsPlan& r, int64_t m, int64_t n, int64_t k, int8_t* planes, hipStream_t s, rns::RnsOut* o) {
  rns::RnsGemmArgs<1> a;
  std::memset(&a, 0, sizeof(a));
  a.njobs = 1;
  a.total = (int)gemm_job<S>(r, m, n, k, planes, 0, &a.job[0], o);
  return launch_gemm<S, 1>(a, s);
}

template <class S>
int64_t units_of(const rns::RnsOut& o) {
  return (int64_t)o.tiles_m * o.tiles_n * S::NW * S::XB * S::YB / 4;
}

// The recombination's constants mod p.
void combine_args(const RnsPlan& r, const Int8Args& g, rns::CombineArgs* b) {
  b->o.ldc = g.ldc;
  b->C = g.C;
  b->p = (double)g.p;
  b->q = g.q;
  // M / m_t mod p as the product of the moduli before t and those after it
  uint64_t after[kRnsMaxModuli + 1], before = 1;
  after[r.n] = 1;
  for (int i = r.n - 1; i >= 0; i--) after[i] = mulmod_u64(after[i + 1], (uint64_t)kModuli[i], g.p);
  split26(after[0] % g.p, g.p, &b->mhi, &b->mlo);
  for (int i = 0; i < r.n; i++) {
    const int inv = tables().inv[r.n][i];
    const uint64_t iv = (uint64_t)(inv < 0 ? inv + (int64_t)g.p : inv);  // p >= 2^16
    split26(mulmod_u64(mulmod_u64(before, after[i + 1], g.p), iv, g.p), g.p, &b->whi[i], &b->wlo[i]);
    b->f[i] = (double)inv / (double)kModuli[i];
    before = mulmod_u64(before, (uint64_t)kModuli[i], g.p);
  }
}

template <class S>
int launch_mod_p(const RnsPlan& r, const Int8Args& g, int8_t* planes, hipStream_t s) {
  using namespace rns;
  CombineArgs b;
  std::memset(&b, 0, sizeof(b));
  if (int e = launch_products<S>(r, g.m, g.n, g.k, planes, s, &b.o)) return e;
  combine_args(r, g, &b);
  TimerTok* t = timer_begin("rns_combine");
  hipExtLaunchKernelGGL((rns_combine_kernel<S>), dim3((unsigned)cdiv(units_of<S>(b.o), 4)), dim3(256), 0, s,
                        timer_start(t), timer_stop(t), 0, b);
  const int e = (int)hipGetLastError();
  timer_commit(t, e);
  return e;
}

// Products of one tile shape (`pick`, in table order): their INT8 products in one
// launch, their recombinations 16 a launch.
template <class S>
int launch_shape_batch(const RnsBatchJob* jobs, const std::vector<int>& pick, hipStream_t s) {
  using namespace rns;
  if (pick.empty()) return 0;
  RnsGemmArgs<kRnsBatch> a;
  std::memset(&a, 0, sizeof(a));
  std::vector<CombineArgs> outs(pick.size());
  int64_t items = 0;
  for (size_t i = 0; i < pick.size(); i++) {
    const RnsBatchJob& j = jobs[pick[i]];
    std::memset(&outs[i], 0, sizeof(outs[i]));
    items += gemm_job<S>(j.plan, j.g.m, j.g.n, j.g.k, j.g.work, items, &a.job[i], &outs[i].o);
    combine_args(j.plan, j.g, &outs[i]);
  }
  if (items > 0x3fffffff) return (int)hipErrorInvalidValue;
  a.njobs = (int)pick.size();
  a.total = (int)items;
  if (int e = launch_gemm<S, kRnsBatch>(a, s)) return e;
  for (size_t c = 0; c < outs.size(); c += kCombineBatch) {
    CombineBatch b;
    std::memset(&b, 0, sizeof(b));
    b.njobs = (int)std::min<size_t>(kCombineBatch, outs.size() - c);
    int64_t groups = 0;
    for (int i = 0; i < b.njobs; i++) {
      b.start[i] = (int)groups;
      b.job[i] = outs[c + i];
      groups += cdiv(units_of<S>(outs[c + i].o), 4);
    }
    if (groups > 0x7fffffff) return (int)hipErrorInvalidValue;
    TimerTok* t = timer_begin("rns_batch_combine");
    hipExtLaunchKernelGGL((rns_combine_batch_kernel<S>), dim3((unsigned)groups), dim3(256), 0, s, timer_start(t),
                          timer_stop(t), 0, b);
    const int e = (int)hipGetLastError();
    timer_commit(t, e);
    if (e) return e;
  }
  return 0;
}

// Integers of up to 192 bits, two's complement, as 32-bit words: W_t and M.
struct Wide {
  static constexpr int kWords = 6;
  uint32_t w[kWords] = {1, 0, 0, 0, 0, 0};
  void mul(uint32_t x) {
    uint64_t c = 0;
    for (int i = 0; i < kWords; i++) {
      c += (uint64_t)w[i] * x;
      w[i] = (uint32_t)c;
      c >>= 32;
    }
  }
  void negate() {
    uint64_t c = 1;
    for (int i = 0; i < kWords; i++) {
      c += (uint32_t)~w[i];
      w[i] = (uint32_t)c;
      c >>= 32;
    }
  }
  // limbs of base 2^b, all but the top in [0, 2^b)
  void limbs(int b, int n, double* out) const {
    for (int j = 0; j < n; j++) {
      unsigned __int128 v = 0;
      const int bit = j * b;
      for (int i = bit / 32, s = -(bit % 32); i < kWords && s < 64; i++, s += 32)
        v |= s >= 0 ? (unsigned __int128)w[i] << s : (unsigned __int128)(w[i] >> -s);
      if (j + 1 < n) {
        out[j] = (double)(uint64_t)(v & (((uint64_t)1 << b) - 1));
      } else {  // sign-extended from 192 bits
        const int left = 32 * kWords - bit;
        int64_t x = (int64_t)(uint64_t)v;
        if (left < 64) x = (int64_t)((uint64_t)x << (64 - left)) >> (64 - left);
        out[j] = (double)x;
      }
    }
  }
};

template <class S, int NG>
int launch_primes(const rns::CrtCombineArgs& b, hipStream_t s) {
  TimerTok* t = timer_begin("rns_crt_combine");
  hipExtLaunchKernelGGL((rns::rns_crt_combine_kernel<S, NG>), dim3((unsigned)cdiv(2 * units_of<S>(b.o), 4)), dim3(256),
                        0, s, timer_start(t), timer_stop(t), 0, b);
  const int e = (int)hipGetLastError();
  timer_commit(t, e);
  return e;
}

template <class S>
int launch_crt_shape(const RnsCrt& c, const uint64_t* primes, int nprimes, double* const* C, int64_t ldc, int64_t m,
                     int64_t n, int64_t k, int8_t* planes, hipStream_t s) {
  using namespace rns;
  const RnsPlan& r = c.plan;
  CrtCombineArgs b;
  std::memset(&b, 0, sizeof(b));
  if (int e = launch_products<S>(r, m, n, k, planes, s, &b.o)) return e;
  b.o.ldc = ldc;
  b.base = std::ldexp(1.0, c.base_bits);
  b.rbase = std::ldexp(1.0, -c.base_bits);
  Wide M;
  for (int i = 0; i < r.n; i++) M.mul((uint32_t)kModuli[i]);
  M.limbs(c.base_bits, c.limbs, b.M);
  for (int i = 0; i < r.n; i++) {
    const int inv = tables().inv[r.n][i];
    Wide W;
    for (int j = 0; j < r.n; j++)
      if (j != i) W.mul((uint32_t)kModuli[j]);
    W.mul((uint32_t)std::abs(inv));
    if (inv < 0) W.negate();
    W.limbs(c.base_bits, c.limbs, b.w[i]);
    b.f[i] = (double)inv / (double)kModuli[i];
  }
  for (int i0 = 0; i0 < nprimes; i0 += kMaxPrimesCrt) {
    b.nprimes = std::min(kMaxPrimesCrt, nprimes - i0);
    b.lines = ldc % 16 == 0;
    for (int i = 0; i < b.nprimes; i++) {
      b.p[i] = (double)primes[i0 + i];
      b.q[i] = 1.0 / (double)primes[i0 + i];
      b.C[i] = C[i0 + i];
      if ((uintptr_t)b.C[i] % 128) b.lines = 0;
    }
    int e;
    switch (c.limbs) {
      case 1: e = launch_primes<S, 1>(b, s); break;
      case 2: e = launch_primes<S, 2>(b, s); break;
      case 3: e = launch_primes<S, 3>(b, s); break;
      case 4: e = launch_primes<S, 4>(b, s); break;
      case 5: e = launch_primes<S, 5>(b, s); break;
      default: e = launch_primes<S, 6>(b, s); break;
    }
    if (e) return e;
  }
  return 0;
}

}  // namespace

// Moduli whose product exceeds 2^1.05 bound (|X| <= bound), 0 if none: log2 M
// and log2 bound are binary64 sums of at most 21 logarithms, good to 1e-12.
int rns_moduli(double log2_bound) {
  for (int n = 1; n <= kRnsMaxModuli; n++)
    if (tables().log2M[n] >= log2_bound + 1.05) return n;
  return 0;
}

namespace {

// Estimates in microseconds, fitted (least relative squares) to 260 products
// with m, n, k log-uniform up to 12000 (k to 131072) and 18 to 52 bits, each
// timed in both forms on one MI355X: within 10% of the measured time for 80%
// of the products in the residue form and 18% in the digit form.  Choosing by
// them costs 0.8% over always choosing right.
//
// Digit form: a fixed part, the planes (8 bytes read and D written an entry),
// the digit products (by work, by rounds of workgroups and by the length of
// one workgroup's chain) and the outputs.
double digits_us(int64_t m, int64_t n, int64_t k, int D) {
  const int64_t st = cdiv(k, 64);
  const int s = choose_splits_fill(cdiv(m, 64) * cdiv(n, 64), st, 32);
  const int64_t items = cdiv(m, 64) * cdiv(n, n <= 32 ? 32 : 64) * s;
  const double chain = (double)cdiv(st, s), stage = (double)D * D * (n <= 32 ? 0.5 : 1.0);
  return 12.7 + 0.233e-6 * ((double)m + n) * k * (8 + D) + 0.0558 * (double)items * chain * stage / 512 +
         0.0162 * (double)cdiv(items, D <= 5 ? 512 : 256) * chain * stage + 0.0119 * chain * D * D + 0.22 * chain +
         2.4e-6 * (double)m * n * (s > 1 ? s + 1 : 1);
}

// Residue form: a fixed part, the planes (N written an entry, and read by the
// products), the products by rounds of workgroups, and the residue bytes
// (written, then read) with the outputs.
double residues_us(const RnsPlan& r, int64_t m, int64_t n, int64_t k, int64_t items, int64_t per) {
  const double entries = ((double)m + n) * k, rows = entries * r.n;
  const double out = 0.22e-6 * (double)m * n * (2.0 * r.n * r.splits + 8);
  if (r.large)
    return 15.1 + 0.233e-6 * entries * (8 + r.n) + 0.0575e-6 * rows + 0.65 * (double)(cdiv(items, 256) * per) + out +
           r.n * (0.11 + 0.256 * r.splits);
  return 14.0 + 0.209e-6 * entries * (8 + r.n) + 0.153e-6 * rows + 0.339 * (double)(cdiv(items, 512) * per) + out +
         r.n * (0.064 + 0.246 * r.splits);
}

// One tile shape's plan for nm moduli; false beyond the kernels' index ranges.
template <class S>
bool plan_shape(int nm, int64_t m, int64_t n, int64_t k, RnsPlan* r, bool alone = true) {
  using namespace rns;
  const int64_t stages = cdiv(k, 64), kp = stages * 64, tiles = cdiv(m, S::BM) * cdiv(n, S::BN);
  const int64_t slots = 256 * S::GROUPS;
  // k-ranges: at most 1024 stages each (the int32 bound), and while the items
  // do not fill the chip more, of at least 16 stages
  // (in a batch, others do): of at most 128, or the last would run on alone
  int64_t s = cdiv(stages, alone ? 1024 : 128);
  while (alone && tiles * nm * s < slots && stages / (s + 1) >= 16 && s < 64) s++;
  if (s > 64) return false;
  const int64_t per = cdiv(stages, s);
  r->n = nm;
  r->splits = (int)cdiv(stages, per);  // no empty range
  r->large = std::is_same<S, RnsLarge>::value;
  const int64_t items = tiles * nm * r->splits;
  const int64_t parts = row_blocks(m) * cdiv(kp, 256) + cdiv(n, 64) * stages;  // conversion workgroups
  if (items > 0x3fffffff || tiles * 64 > 0x7fffffff || parts > 0x7fffffff) return false;
  // copies address an operand's plane with 32-bit offsets
  if (row_blocks(std::max(m, n)) * 16 * kp >= ((int64_t)1 << 32)) return false;
  r->bytes_a = (size_t)nm * row_blocks(m) * 16 * kp;
  r->bytes_b = (size_t)nm * row_blocks(n) * 16 * kp;
  r->bytes = r->bytes_a + r->bytes_b + (size_t)items * S::TILE_BYTES;
  r->us = residues_us(*r, m, n, k, items, per);
  return true;
}

}  // namespace

bool rns_chosen(uint64_t p, int64_t m, int64_t n, int64_t k, const mmp_opts* opts, RnsPlan* r) {
  using namespace rns;
  // what asks for the digit form: MMP_FORM_INT8_WORDS by name, prepared planes, a
  // forced block or k-ranges.  From three digits on (one or two digits need at
  // most four products, and the recombination's bounds take p >= 2^16).
  if (opts && (opts->form != MMP_FORM_AUTO || opts->prepared_a || opts->prepared_b || opts->force_kblock ||
               opts->splits))
    return false;
  if (m <= 0 || n <= 0 || k <= 0 || p < (1u << 16)) return false;
  if (std::max(std::max(m, n), k) > 0x7fffffff) return false;
  const int nm = rns_moduli(std::log2((double)k) + 2.0 * std::log2((double)(p / 2)));
  if (nm == 0) return false;
  RnsPlan small;
  if (!plan_shape<RnsSmall>(nm, m, n, k, &small)) return false;
  *r = small;
  RnsPlan large;
  if (plan_shape<RnsLarge>(nm, m, n, k, &large) && large.us < small.us) *r = large;
  if (r->bytes > kInt8MaxBytes) return false;
  // Where a size is below 1024 the estimates err more, above all with a short k (957^3,
  // 42 bits: estimated 45 us against 53 on digits, took 55 against 49): the residue
  // form has to be 20% faster by them there, 10% with m or n below 1024.
  const double margin = k < 1024 ? 0.8 : std::min(m, n) < 1024 ? 0.9 : 1.0;
  return r->us < margin * digits_us(m, n, k, digits_for(p));
}

double int8_us(uint64_t p, int64_t m, int64_t n, int64_t k, const mmp_opts* opts, size_t* bytes) {
  RnsPlan r;
  const bool residues = rns_chosen(p, m, n, k, opts, &r);
  *bytes = residues ? r.bytes : 0;
  return residues ? r.us : digits_us(m, n, k, digits_for(p));
}

int launch_rns(const RnsPlan& r, const Int8Args& g, void* stream) {
  using namespace rns;
  hipStream_t s = (hipStream_t)stream;
  const CenteredIn A{g.A, (int64_t)g.p, (int64_t)(g.p / 2)}, B{g.B, (int64_t)g.p, (int64_t)(g.p / 2)};
  const int e = g.p >> 31 ? launch_convert<CenteredIn, true>(r, A, g.m, g.lda, B, g.n, g.ldb, g.k, g.work, s)
                          : launch_convert<CenteredIn, false>(r, A, g.m, g.lda, B, g.n, g.ldb, g.k, g.work, s);
  if (e) return e;
  return r.large ? launch_mod_p<RnsLarge>(r, g, g.work, s) : launch_mod_p<RnsSmall>(r, g, g.work, s);
}

bool rns_batch_chosen(uint64_t p, int64_t m, int64_t n, int64_t k, RnsPlan* r, Int8Share* share) {
  using namespace rns;
  *share = Int8Share{0.0, 0.0, 0.0};
  if (m <= 0 || n <= 0 || k <= 0 || std::max(std::max(m, n), k) > 0x7fffffff) return false;
  // the chip's time of this product on its digits, in the launch of the whole batch
  const int D = digits_for(p), bn = D <= 4 ? 64 : 32;
  const double entries = ((double)m + n) * k, tiles = (double)(cdiv(m, 64) * cdiv(n, bn)), st = (double)cdiv(k, 64);
  const double products = 0.064 / 512 * D * D * (bn / 64.0) * tiles * st, planes = 0.233e-6 * entries * (8 + D);
  share->digits_us = products + planes;
  share->us = products + planes + 0.636 / 512 * D * tiles + 1.96e-6 * (double)m * n;
  share->chain_us = 0.014 * st * D * D + 0.33 * st;
  const int nm = p < (1u << 16) ? 0 : rns_moduli(std::log2((double)k) + 2.0 * std::log2((double)(p / 2)));
  if (nm == 0) return false;
  RnsPlan small, large;
  if (!plan_shape<RnsSmall>(nm, m, n, k, &small, false) || !plan_shape<RnsLarge>(nm, m, n, k, &large, false)) return false;
  // and by its residues: a large tile's stage takes 0.65 / 256 us, a small one's 0.339 / 512
  const double tl = 0.65 / 256 * st * nm * (double)cdiv(m, RnsLarge::BM) * cdiv(n, RnsLarge::BN);
  const double ts = 0.339 / 512 * st * nm * (double)cdiv(m, RnsSmall::BM) * cdiv(n, RnsSmall::BN);
  *r = tl < ts ? large : small;
  const double residues = std::min(tl, ts) + 0.233e-6 * entries * (8 + nm) + 0.22e-6 * (double)m * n * (2 * nm + 8);
  share->us = std::min(share->us, residues);
  // The digits' launch holds the code of every digit count, at 64 x 32 tiles from
  // five digits on, and its products run well below that estimate: batches of 32 and
  // 64 products with sizes 64 to 4096 took 1553 and 1112 us with every product on
  // its digits, 1154 and 953 with those whose residues take less than 1.3 times the
  // estimate, 1112 and 924 with 3 times, 1106 and 937 with all.  The planes run as
  // estimated in both forms, so that where they are most of the time, in products
  // with one narrow side, the digits' smaller ones win (6 of 8 x 4096 x 8192, 36
  // bits: 880 us against 1420), unless one workgroup's chain of digit products is
  // longer (4 of 325 x 3 x 32231, 43 bits: 446 us in the residue form, its k-ranges
  // side by side, 661 on digits).
  return residues < std::max(3.0 * products + planes, share->chain_us);
}

int launch_rns_batch(const RnsBatchJob* jobs, int njobs, void* stream) {
  using namespace rns;
  if (njobs < 1 || njobs > kRnsBatch) return (int)hipErrorInvalidValue;
  hipStream_t s = (hipStream_t)stream;
  ConvBatch b;
  std::memset(&b, 0, sizeof(b));
  b.ca.n = kRnsMaxModuli;
  std::memcpy(b.ca.c, tables().conv, sizeof(b.ca.c));
  b.njobs = njobs;
  int64_t groups = 0;
  std::vector<int> large, small;
  for (int i = 0; i < njobs; i++) {
    const Int8Args& g = jobs[i].g;
    ConvJob& c = b.job[i];
    c.A = g.A;
    c.B = g.B;
    c.p = (int64_t)g.p;
    c.m = g.m;
    c.n = g.n;
    c.k = g.k;
    c.lda = g.lda;
    c.ldb = g.ldb;
    c.kp = g.kp;
    c.outA = g.work;
    c.outB = g.work + jobs[i].plan.bytes_a;
    c.nmod = jobs[i].plan.n;
    c.start = (int)groups;
    const int64_t na = row_blocks(g.m) * cdiv(g.kp, 256);
    c.na = (int)na;
    groups += na + cdiv(g.n, 64) * (g.kp / 64);
    if (groups > 0x7fffffff) return (int)hipErrorInvalidValue;
    (jobs[i].plan.large ? large : small).push_back(i);
  }
  TimerTok* t = timer_begin("rns_batch_convert");
  hipExtLaunchKernelGGL(rns_convert_batch_kernel, dim3((unsigned)groups), dim3(256), 0, s, timer_start(t), timer_stop(t),
                        0, b);
  int e = (int)hipGetLastError();
  timer_commit(t, e);
  if (e) return e;
  // longest items first, so that the short ones fill the end
  auto longer = [&](int x, int y) {
    const RnsPlan &a = jobs[x].plan, &c = jobs[y].plan;
    return jobs[x].g.kp * c.splits > jobs[y].g.kp * a.splits;
  };
  std::stable_sort(large.begin(), large.end(), longer);
  std::stable_sort(small.begin(), small.end(), longer);
  e = launch_shape_batch<RnsLarge>(jobs, large, s);
  return e ? e : launch_shape_batch<RnsSmall>(jobs, small, s);
}

// The multi-modular product of integers below 2^entry_bits: 0 <= X <
// k 2^(2 entry_bits).
bool rns_crt_plan(int64_t m, int64_t n, int64_t k, int entry_bits, uint64_t smallest_prime, RnsCrt* c) {
  using namespace rns;
  if (m <= 0 || n <= 0 || k <= 0 || std::max(std::max(m, n), k) > 0x7fffffff) return false;
  const double bits = std::log2((double)k) + 2.0 * entry_bits;
  const int nm = rns_moduli(bits);
  if (nm == 0) return false;
  RnsPlan small, large;
  if (!plan_shape<RnsSmall>(nm, m, n, k, &small)) return false;
  c->plan = small;
  if (plan_shape<RnsLarge>(nm, m, n, k, &large) && large.us < small.us) c->plan = large;
  if (c->plan.bytes > kInt8MaxBytes) return false;
  // the base: 2^b (1 + 2^b / p) <= 2^50 for every prime, limbs below 2^53 before
  // their carries (20 moduli, 128, the k-ranges)
  int b = 24;
  while (b < 40 && std::ldexp(1.0, 2 * (b + 1)) / (double)smallest_prime + std::ldexp(1.0, b + 1) <= std::ldexp(1.0, 50) &&
         std::ldexp(1.0, b + 1) * 2 * 20 * 128 * c->plan.splits < std::ldexp(1.0, 53))
    b++;
  // the limbs hold M, and with it every W_t
  const double mbits = tables().log2M[nm] + 1.0;
  const int limbs = (int)std::ceil(mbits / b);
  if (limbs > kCrtLimbs) return false;
  c->base_bits = (int)std::ceil(mbits / limbs);  // no wider than it needs to be
  c->limbs = limbs;
  return true;
}

bool rns_crt_chosen(int64_t m, int64_t n, int64_t k, int entry_bits, const uint64_t* primes, int nprimes,
                    const mmp_opts* opts, RnsCrt* c) {
  if (opts && opts->form != MMP_FORM_AUTO) return false;
  if (!rns_crt_plan(m, n, k, entry_bits, *std::min_element(primes, primes + nprimes), c)) return false;
  // Beyond one int32 block the alternative is a product per prime.
  if (k > int8_bound_integers(entry_bits).kblock) return true;
  // Else the digit form's one kernel for the D^2 digit products and all primes.
  // Both in microseconds, fitted to 300 jobs with m, n log-uniform up to 3072,
  // k to 8192, 16 to 62 bits and 3 to 64 primes (within 18% for 80% of them;
  // choosing by it costs 5% over always choosing right, 1.2% without the margins below).  The residue form
  // won 214 of them (2048^3, 60 bits, 32 primes: 666 -> 445 us); short k with
  // few bits stays with the digits (2521 x 2750 x 263, 32 bits, 5 primes: 164
  // against 190).
  const int D = crt_digits(entry_bits);
  const double entries = ((double)m + n) * k, out = 8e-6 * (double)m * n * nprimes, chain = (double)cdiv(k, 64) * D * D;
  const int64_t tiles = cdiv(m, 64) * cdiv(n, 64), rounds = cdiv(tiles, D <= 5 ? 512 : 256);
  const double digits = 12.5 + 0.22e-6 * entries * (8 + D) + 0.0092 * (double)tiles * chain / 512 +
                        0.037 * (double)rounds * chain + 0.79 * (double)rounds * nprimes + 0.231 * out;
  const int64_t waves = 32 * cdiv(m, 128) * cdiv(n, 128);
  const double residues = 0.7 + 0.894 * c->plan.us + 0.139 * out + nprimes * (0.464 + 0.2 * (double)cdiv(waves, 1024));
  // Of those 300 jobs 11 ran 4 to 23% slower in the residue form than the estimates
  // said, 2 with these margins: from few digits, and where a size is small.
  const double margin = D <= 4 ? 0.78 : std::min(std::min(m, n), k) <= 700 ? 0.9 : 1.0;
  return residues < margin * digits;
}

int launch_rns_crt(const RnsCrt& c, const uint64_t* A, int64_t lda, const uint64_t* B, int64_t ldb, int64_t m, int64_t n,
                   int64_t k, const uint64_t* primes, int nprimes, double* const* C, int64_t ldc, void* work,
                   void* stream) {
  using namespace rns;
  hipStream_t s = (hipStream_t)stream;
  int8_t* planes = (int8_t*)work;
  if (int e = launch_convert<IntegerIn, true>(c.plan, IntegerIn{A}, m, lda, IntegerIn{B}, n, ldb, k, planes, s)) return e;
  return c.plan.large ? launch_crt_shape<RnsLarge>(c, primes, nprimes, C, ldc, m, n, k, planes, s)
                      : launch_crt_shape<RnsSmall>(c, primes, nprimes, C, ldc, m, n, k, planes, s);
}

}  // namespace mmp
