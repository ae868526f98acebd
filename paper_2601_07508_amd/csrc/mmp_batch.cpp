// Batched products and multi-modular (CRT) products.
//
// mm_modp_batched: every product is planned on its own; those of an AUTO batch may
// then move to INT8 words for launches that they share (move_to_int8), and on INT8
// words to the residue form.  FP64-word products of one configuration run together,
// up to kMaxBatch per launch, with the job table in the kernel arguments.  INT8
// products have one workspace for the whole batch: those in the residue form share a
// conversion, a product launch per tile size and their recombinations, the others
// one launch of digit planes and one of the digit GEMM for every 64 of them
// (batch_launch = 1: planes per product, one GEMM per digit count).  The batch is
// enqueued on one stream with no host synchronisation, so with a caller workspace it
// can be captured into a HIP graph and replayed.
//
// mm_modp_crt: one integer pair A, B against many moduli.  AUTO jobs run in the
// residue form where it is estimated faster, and for any k beyond one exact int32
// block.  Else, within one block, the integers are digitised once, one digit GEMM
// forms the digit-weight sums of A B, and each modulus reduces those sums in the
// epilogue; beyond it (opts->form set, or a workspace too small for the residue
// planes) A and B are reduced mod each p on the device and the products run one by
// one.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <tuple>
#include <vector>

#include "mmp_internal.h"

namespace {

using namespace mmp;

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Planned {
  const mmp_job* job;
  mmp_plan_t plan;
  size_t ws_offset;
  bool residues;  // in the residue form
  RnsPlan rns;
  Int8Share share;
};

// FP64-word products of one configuration run together
using Fp64Key = std::tuple<int, int, int, int>;
Fp64Key fp64_key(const mmp_plan_t& pl) {
  return std::make_tuple(pl.u, pl.v, pl.tile, fp64_class(pl.slots, pl.kblock, pl.lazy != 0));
}

// Products of a batch that their plans give to FP64 words and that are moved to INT8
// words (`may`: those that may be).  On INT8 words a product fills in beside others
// in launches that it shares with them, where each FP64 configuration is a launch of
// its own with the chip mostly idle (40 to 170 us each in a batch of 32 with sizes 64
// to 4096).  But products bound by reading one large operand pay for its planes (2 of
// 16384 x 8 x 32768, 25 bits: 2.06 ms on FP64 words, 4.64 on INT8), and small ones of
// one configuration need one launch instead of two (2 of 64^3: 17 us against 24).
// So each configuration's launches are compared with what its products take of the
// chip on INT8 words: all of them, or those that alone take less there.  Where no
// other product runs on INT8 words anyway, those launches are paid for as well.
// Over 15000 random batches (2 to 64 products, sizes 1 to 17000, 8 to 52 bits) the
// choice between all and none by these estimates costs 0.7% over always choosing
// right; always moving cost 17%, never 59%.
void move_to_int8(std::vector<Planned>& pj, const std::vector<char>& may, std::vector<char>* moved) {
  constexpr double kLaunchUs = 3.0;   // a further launch: its host time and the gap before it
  constexpr double kSharedUs = 24.0;  // the digits' two launches and a workspace
  std::map<Fp64Key, std::vector<int>> groups;
  bool others = false;
  double chain = 0.0, gain = 0.0;
  for (size_t i = 0; i < pj.size(); i++) {
    const mmp_job& j = *pj[i].job;
    if (j.m == 0 || j.n == 0 || j.k == 0) continue;
    if (pj[i].plan.form == MMP_FORM_FP64_WORDS)
      groups[fp64_key(pj[i].plan)].push_back((int)i);
    else
      others = true;
  }
  std::vector<Fp64Load> loads;
  auto launches_us = [&](const std::vector<int>& g, auto stays) {
    loads.clear();
    for (int i : g)
      if (stays(i)) loads.push_back(fp64_load(pj[i].plan, pj[i].job->m, pj[i].job->n, pj[i].job->k));
    double us = 0.0;
    for (size_t c = 0; c < loads.size(); c += kMaxBatch)
      us += kLaunchUs + fp64_launch_us(pj[g[0]].plan, loads.data() + c, (int)std::min<size_t>(kMaxBatch, loads.size() - c));
    return us;
  };
  for (const auto& kv : groups) {
    const std::vector<int>& g = kv.second;
    const double none = launches_us(g, [](int) { return true; });
    double best = none;
    int choice = 0;
    for (int which = 1; which <= 2; which++) {
      auto moves = [&](int i) {
        return may[i] && (which == 1 || pj[i].share.us <
                                            fp64_load(pj[i].plan, pj[i].job->m, pj[i].job->n, pj[i].job->k).share);
      };
      double us = launches_us(g, [&](int i) { return !moves(i); });
      for (int i : g)
        if (moves(i)) us += pj[i].share.us;
      if (us >= best) continue;
      best = us;
      choice = which;
      for (int i : g) (*moved)[i] = moves(i);
    }
    if (choice == 0) continue;
    gain += none - best;
    for (int i : g)
      if ((*moved)[i]) chain = std::max(chain, pj[i].share.chain_us);
  }
  if (!others && gain < kSharedUs + chain) moved->assign(pj.size(), 0);
}

// together: AUTO products of a batch of two or more are planned for the launches
// they share: on FP64 or INT8 words by move_to_int8, and each on INT8 words in the
// residue form where that is less of the chip's time.
int plan_batch(const mmp_job* jobs, int count, const mmp_opts* opts, bool together, std::vector<Planned>* out,
               size_t* ws_total) {
  if (count < 0 || (count > 0 && !jobs)) return MMP_EINVAL;
  // batched products run one k-range each (their many tiles fill the chip)
  mmp_opts o1;
  std::memset(&o1, 0, sizeof(o1));
  if (opts) o1 = *opts;
  o1.splits = 1;
  opts = &o1;
  together = together && count >= 2 && o1.form == MMP_FORM_AUTO && o1.batch_launch == 0 && !o1.tile &&
             !o1.force_kblock && !o1.extended_block && !o1.centered_words;
  out->clear();
  out->reserve(count);
  std::vector<char> may(count, 0), moved(count, 0);
  bool any = false;
  for (int i = 0; i < count; i++) {
    const mmp_job& j = jobs[i];
    if (int st = check_product_args(j.m, j.n, j.k, j.A, j.lda, j.B, j.ldb, j.C, j.ldc)) return st;
    Planned pj;
    pj.job = &j;
    if (int st = mmp::plan(j.p, j.u, j.v, j.m, j.n, j.k, opts, &pj.plan)) return st;
    if (!fp64_ld_ok(pj.plan, j.lda, j.ldb)) return MMP_EINVAL;
    pj.residues = false;
    pj.share = Int8Share{0.0, 0.0, 0.0};
    if (together && j.u == 0 && j.m > 0 && j.n > 0 && j.k > 0) {
      pj.residues = rns_batch_chosen(j.p, j.m, j.n, j.k, &pj.rns, &pj.share);
      TunedChoice tuned;  // a measured choice stands
      may[i] = pj.plan.form == MMP_FORM_FP64_WORDS && !o1.strict_fmod && !tune_lookup(j.p, j.m, j.n, j.k, 0, &tuned);
      any = any || may[i];
    }
    out->push_back(pj);
  }
  if (any) move_to_int8(*out, may, &moved);
  // Small batches stay whole on their digits, two launches instead of five (16
  // products with sizes 64 to 1000, 75 us of kernels: 87 us against 95).
  constexpr double kSmallBatchUs = 120.0;
  // Memory that no product's own plan calls for, at most in all: residue planes, and
  // any planes of products planned on FP64 words.  Beyond it each is as planned.
  constexpr size_t kMaxExtraBytes = (size_t)8 << 30;
  double digits_us = 0.0;
  for (int i = 0; i < count; i++) {
    Planned& pj = (*out)[i];
    if (!moved[i] && pj.plan.form != MMP_FORM_INT8_WORDS)
      pj.residues = false;
    else if (together && jobs[i].u == 0)
      digits_us += pj.share.digits_us;
  }
  size_t ws = 0, extra = 0;
  for (int i = 0; i < count; i++) {
    Planned& pj = (*out)[i];
    const mmp_job& j = jobs[i];
    if (pj.residues && (digits_us < kSmallBatchUs || extra + pj.rns.bytes > kMaxExtraBytes)) pj.residues = false;
    if (moved[i]) {
      mmp_opts o2 = o1;
      o2.form = MMP_FORM_INT8_WORDS;
      mmp_plan_t p8;
      if (int st = mmp::plan(j.p, 0, 0, j.m, j.n, j.k, &o2, &p8)) return st;
      if (pj.residues || extra + p8.workspace_bytes <= kMaxExtraBytes) pj.plan = p8;
    }
    pj.ws_offset = ws;
    if (pj.plan.form != MMP_FORM_INT8_WORDS || j.m == 0 || j.n == 0 || j.k == 0) continue;
    const size_t bytes = pj.residues ? pj.rns.bytes : pj.plan.workspace_bytes;
    if (pj.residues || moved[i]) extra += bytes;
    ws += align_up(bytes);
  }
  // outputs must not overlap each other
  for (int a = 0; a < count; a++)
    for (int b = a + 1; b < count; b++)
      if (ranges_overlap(jobs[a].C, span_bytes(jobs[a].m, jobs[a].n, jobs[a].ldc), jobs[b].C,
                         span_bytes(jobs[b].m, jobs[b].n, jobs[b].ldc)))
        return MMP_EINVAL;
  *ws_total = ws;
  return MMP_OK;
}

int run_batch(const std::vector<Planned>& pj, const mmp_opts* opts, size_t ws_total, void* stream) {
  const bool validate = opts && opts->validate_entries;
  // zero fills, validation
  for (const Planned& x : pj) {
    const mmp_job& j = *x.job;
    if (j.m == 0 || j.n == 0) continue;
    if (j.k == 0) {
      if (int e = launch_zero_fill(j.C, j.m, j.n, j.ldc, stream)) return hip_status(e);
      continue;
    }
    if (validate)
      if (int st = validate_product_entries(j.p, j.m, j.n, j.k, j.A, j.lda, j.B, j.ldb, stream)) return st;
  }
  // FP64-word products, grouped by kernel configuration
  std::map<Fp64Key, std::vector<const Planned*>> groups;
  for (const Planned& x : pj) {
    const mmp_job& j = *x.job;
    if (j.m == 0 || j.n == 0 || j.k == 0 || x.plan.form != MMP_FORM_FP64_WORDS) continue;
    groups[fp64_key(x.plan)].push_back(&x);
  }
  for (auto& kv : groups) {
    const auto& v = kv.second;
    for (size_t c = 0; c < v.size(); c += kMaxBatch) {
      Fp64Batch b;
      std::memset(&b, 0, sizeof(b));
      b.njobs = (int)std::min<size_t>(kMaxBatch, v.size() - c);
      for (int t = 0; t < b.njobs; t++) {
        const Planned& x = *v[c + t];
        const mmp_job& j = *x.job;
        b.job[t] = make_fp64_args(x.plan, j.m, j.n, j.k, j.A, j.lda, j.B, j.ldb, j.C, j.ldc);
      }
      if (int e = launch_fp64_words(std::get<0>(kv.first), std::get<1>(kv.first), std::get<2>(kv.first), b,
                                    stream))
        return hip_status(e);
    }
  }
  // INT8-digit products
  if (ws_total == 0) return MMP_OK;
  void* work = nullptr;
  bool owned = false;
  if (int st = acquire_workspace(ws_total, opts, stream, &work, &owned)) return st;
  int err = 0;
  // the one-launch form: planes of up to 64 products in one launch, their
  // digit GEMM in one persistent launch
  const int mode = opts ? opts->batch_launch : 0;
  std::vector<Int8Args> all;
  std::vector<int> all_digits;
  std::vector<RnsBatchJob> residues;
  for (const Planned& x : pj) {
    const mmp_job& j = *x.job;
    if (j.m == 0 || j.n == 0 || j.k == 0 || x.plan.form != MMP_FORM_INT8_WORDS) continue;
    const Int8Args g = make_int8_args(x.plan, j.m, j.n, j.k, j.A, j.lda, j.B, j.ldb, j.C, j.ldc,
                                      (int8_t*)work + x.ws_offset);
    if (x.residues) {
      residues.push_back({g, x.rns});
      continue;
    }
    all.push_back(g);
    all_digits.push_back(x.plan.digits_a);
  }
  for (size_t c = 0; c < residues.size() && !err; c += kMaxRnsBatch)
    err = launch_rns_batch(residues.data() + c, (int)std::min<size_t>(kMaxRnsBatch, residues.size() - c), stream);
  if (mode == 2 || (mode == 0 && (all.size() >= 2 || !residues.empty()))) {
    for (size_t c = 0; c < all.size() && !err; c += kMaxMixedBatch) {
      const int nj = (int)std::min<size_t>(kMaxMixedBatch, all.size() - c);
      err = launch_int8_batch(all.data() + c, all_digits.data() + c, nj, stream);
    }
    const int st = hip_status(err);
    const int st2 = release_workspace(work, owned, stream);
    return st ? st : st2;
  }
  std::map<int, std::vector<Int8Args>> by_digits;
  for (const Planned& x : pj) {
    const mmp_job& j = *x.job;
    if (j.m == 0 || j.n == 0 || j.k == 0 || x.plan.form != MMP_FORM_INT8_WORDS) continue;
    Int8Args g = make_int8_args(x.plan, j.m, j.n, j.k, j.A, j.lda, j.B, j.ldb, j.C, j.ldc,
                                (int8_t*)work + x.ws_offset);
    if (!err) err = launch_int8_digitize(x.plan.digits_a, g, stream);
    by_digits[x.plan.digits_a].push_back(g);
  }
  for (auto& kv : by_digits) {
    for (size_t c = 0; c < kv.second.size() && !err; c += kMaxBatch) {
      const int nj = (int)std::min<size_t>(kMaxBatch, kv.second.size() - c);
      err = launch_int8_gemm(kv.first, kv.second.data() + c, nj, stream);
    }
  }
  const int st = hip_status(err);
  const int st2 = release_workspace(work, owned, stream);
  return st ? st : st2;
}

// CRT: workspace for the fast path, or for the reduced copies of the
// fallback (two binary64 matrices per modulus plus their products' needs).
bool crt_fast(int64_t k, int entry_bits, int nprimes) {
  return k <= int8_bound_integers(entry_bits).kblock && nprimes >= 1;
}

// Without the residue form: the digit planes of one integer product, or beyond
// one int32 block the reduced copies.
size_t crt_digits_workspace(int64_t m, int64_t n, int64_t k, int entry_bits, int nprimes) {
  const int d = crt_digits(entry_bits);
  const size_t kp = (size_t)((k + 63) / 64 * 64);
  if (crt_fast(k, entry_bits, nprimes)) return digit_planes_bytes(d, m, kp) + digit_planes_bytes(d, n, kp);
  // fallback: per modulus, reduced A and B in binary64 (the products use the
  // planner's form; an INT8 product needs at most 7-digit planes of A and B)
  const size_t per = align_up(8 * (size_t)(m * k + k * n)) + align_up(int8_workspace_bytes(kMaxDigits, m, n, k));
  return per * (size_t)nprimes;
}

}  // namespace

extern "C" {

size_t mmp_workspace_batched(const mmp_job* jobs, int count, const mmp_opts* opts) {
  std::vector<Planned> pj;
  size_t ws = 0;
  if (plan_batch(jobs, count, opts, true, &pj, &ws) != MMP_OK) return 0;
  return ws;
}

int mm_modp_batched(const mmp_job* jobs, int count, const mmp_opts* opts, void* stream) {
  try {
    std::vector<Planned> pj;
    size_t ws = 0;
    // a capture without a workspace records no allocation that the products' own
    // plans do not call for
    const bool together = (opts && opts->workspace) || !capturing(stream);
    if (int st = plan_batch(jobs, count, opts, together, &pj, &ws)) return st;
    // a caller's workspace too small for that (or unaligned): each product as planned on its own
    if (opts && opts->workspace && (opts->workspace_bytes < ws || (uintptr_t)opts->workspace % 16))
      if (int st = plan_batch(jobs, count, opts, false, &pj, &ws)) return st;
    const int st = run_batch(pj, opts, ws, stream);
    if (st != MMP_ENOMEM || !together || (opts && opts->workspace)) return st;
    // no memory for the shared launches' planes: again with each product's own
    (void)hipGetLastError();
    if (int st2 = plan_batch(jobs, count, opts, false, &pj, &ws)) return st2;
    return run_batch(pj, opts, ws, stream);
  } catch (...) {
    return MMP_EINVAL;
  }
}

size_t mmp_workspace_crt(int64_t m, int64_t n, int64_t k, int entry_bits, int nprimes, const mmp_opts* opts) {
  (void)opts;
  if (m <= 0 || n <= 0 || k <= 0 || entry_bits < 1 || entry_bits > 62 || nprimes < 1) return 0;
  RnsCrt rc;  // its planes do not depend on the primes
  const size_t residues = rns_crt_plan(m, n, k, entry_bits, kPMax, &rc) ? rc.plan.bytes : 0;
  return std::max(residues, crt_digits_workspace(m, n, k, entry_bits, nprimes));
}

int mm_modp_crt(const mmp_opts* opts, const uint64_t* A, int64_t lda, const uint64_t* B, int64_t ldb, int64_t m,
                int64_t n, int64_t k, int entry_bits, const uint64_t* primes, int nprimes, double* const* C,
                int64_t ldc, void* stream) {
  try {
    if (m < 0 || n < 0 || k < 0 || entry_bits < 1 || entry_bits > 62) return MMP_EINVAL;
    if (nprimes < 1 || !primes || !C) return MMP_EINVAL;
    if (opts) {
      if (opts->batch_launch != 0) return MMP_EINVAL;
      if (opts->prepared_a || opts->prepared_b) return MMP_EINVAL;
    }
    for (int i = 0; i < nprimes; i++) {
      if (primes[i] < 5 || primes[i] >= kPMax) return MMP_EINVAL;
      if (m > 0 && n > 0 && !C[i]) return MMP_EINVAL;
    }
    if (m == 0 || n == 0) return MMP_OK;
    if (ldc < n) return MMP_EINVAL;
    if (k > 0 && (!A || !B || lda < k || ldb < n)) return MMP_EINVAL;
    for (int i = 0; i < nprimes; i++)
      for (int j = i + 1; j < nprimes; j++)
        if (ranges_overlap(C[i], span_bytes(m, n, ldc), C[j], span_bytes(m, n, ldc))) return MMP_EINVAL;
    if (k == 0) {
      for (int i = 0; i < nprimes; i++)
        if (int e = launch_zero_fill(C[i], m, n, ldc, stream)) return hip_status(e);
      return MMP_OK;
    }
    if (opts && opts->validate_entries)
      if (int st = validate_integer_entries(entry_bits, m, n, k, A, lda, B, ldb, stream)) return st;

    const int d = crt_digits(entry_bits);
    void* work = nullptr;
    bool owned = false;
    // the residue form where it is faster and its planes fit
    RnsCrt rc;
    if (rns_crt_chosen(m, n, k, entry_bits, primes, nprimes, opts, &rc) &&
        (!opts || ((uintptr_t)opts->workspace % 16) == 0)) {
      if (acquire_workspace(rc.plan.bytes, opts, stream, &work, &owned) == MMP_OK) {
        const int st = hip_status(launch_rns_crt(rc, A, lda, B, ldb, m, n, k, primes, nprimes, C, ldc, work, stream));
        const int st2 = release_workspace(work, owned, stream);
        return st ? st : st2;
      }
      if (!(opts && opts->workspace)) (void)hipGetLastError();  // the launches below report their own
    }
    const size_t ws = crt_digits_workspace(m, n, k, entry_bits, nprimes);
    if (int st = acquire_workspace(ws, opts, stream, &work, &owned)) return st;
    int st = MMP_OK;
    if (crt_fast(k, entry_bits, nprimes)) {
      CrtLaunch c;
      std::memset(&c, 0, sizeof(c));
      c.A = A;
      c.B = B;
      c.m = m;
      c.n = n;
      c.k = k;
      c.lda = lda;
      c.ldb = ldb;
      c.ldc = ldc;
      c.kp = (k + 63) / 64 * 64;
      c.work = (int8_t*)work;
      for (int i0 = 0; i0 < nprimes && st == MMP_OK; i0 += kMaxPrimesCrt) {
        c.nprimes = std::min(kMaxPrimesCrt, nprimes - i0);
        for (int i = 0; i < c.nprimes; i++) {
          c.p[i] = primes[i0 + i];
          c.C[i] = C[i0 + i];
        }
        st = hip_status(launch_crt(d, c, stream));
      }
    } else {
      // reduce mod each p on the device, then the products one by one
      const size_t per = align_up(8 * (size_t)(m * k + k * n)) + align_up(int8_workspace_bytes(kMaxDigits, m, n, k));
      std::vector<mmp_job> jobs(nprimes);
      for (int i = 0; i < nprimes && st == MMP_OK; i++) {
        double* Ar = (double*)((char*)work + per * i);
        double* Br = Ar + m * k;
        st = hip_status(launch_reduce_mod(A, m, k, lda, primes[i], Ar, k, stream));
        if (st == MMP_OK) st = hip_status(launch_reduce_mod(B, k, n, ldb, primes[i], Br, n, stream));
        mmp_job& j = jobs[i];
        std::memset(&j, 0, sizeof(j));
        j.p = primes[i];
        j.m = m;
        j.n = n;
        j.k = k;
        j.A = Ar;
        j.lda = k;
        j.B = Br;
        j.ldb = n;
        j.C = C[i];
        j.ldc = ldc;
      }
      // each product's digit planes go after its reduced copies
      for (int i = 0; i < nprimes && st == MMP_OK; i++) {
        mmp_opts o;
        std::memset(&o, 0, sizeof(o));
        if (opts) o.form = opts->form;
        o.splits = 1;
        o.workspace = (char*)work + per * i + align_up(8 * (size_t)(m * k + k * n));
        o.workspace_bytes = align_up(int8_workspace_bytes(kMaxDigits, m, n, k));
        st = mm_modp_async(&o, jobs[i].p, 0, 0, m, n, k, jobs[i].A, jobs[i].lda, jobs[i].B, jobs[i].ldb,
                           jobs[i].C, jobs[i].ldc, stream);
      }
    }
    const int st2 = release_workspace(work, owned, stream);
    return st ? st : st2;
  } catch (...) {
    return MMP_EINVAL;
  }
}

}  // extern "C"
