// Batched execution of many join-aggregate instances of uneven size in one
// persistent, graph-captured launch.
//
// Handled shape ("row union"): two annotated relations A(i, j) and E(j)
// or E(j, k) under the order i, j[, k] with output [i] or [i, k] -- the
// sparse matrix-vector and matrix-matrix products the paper expresses as
// join-aggregate queries (the order i, j, k is the relaxed order of section
// 4.1.2, whose last attribute is materialized by a GROUP BY on a key,
// section 5).  Every row i of every instance is a work item:
//  * vector rows (E(j)) are taken by eight lanes each, long ones by a block;
//  * light rows (few products) are taken by one wave, which sums exactly
//    into a private LDS hash keyed by k;
//  * heavy rows are taken by a whole block: a symbolic pass marks the k the
//    row produces in an LDS bitmap, whose popcount prefixes rank them; the
//    products are then summed exactly in LDS accumulators indexed by rank,
//    512 ranks at a time, each window's products cut out of the B rows by
//    binary search and spread evenly over the block, and emitted in k order;
//  * rows with many products relative to the size of E are taken by a
//    block in inner-product form: A's row becomes an LDS bitmap over j and
//    the entries of E transposed (built once per batch) are streamed
//    through it, matches adding to per-column LDS accumulators.
// Workers pull items from two device queues (heavy rows first, longest
// first), so one launch balances thousands of instances.  Plans that come
// a second time have the launch and its queue resets captured in a hipGraph
// and replayed from then on.  Sums are
// exact (the same accumulator as the single-plan path), so every instance's
// result is bit-identical to running its plan alone.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <filesystem>
#include <fstream>
#include <map>
#include <memory>
#include <mutex>
#include <sstream>
#include <string>

#include "device_common.h"
#include "engine.h"
#include "exact.h"

namespace lh {

namespace {

constexpr int B_NT = 256;
constexpr int B_NW = B_NT / WAVE;
constexpr uint32_t KW_MAX = 64 * 4 * B_NT;   // k values per heavy window (4 bitmap words per thread)
constexpr uint32_t EMPTY_KEY = 0xffffffffu;

struct BInst {
  uint32_t kind;             // 0: E(j) (vector), 1: E(j, k) (matrix)
  uint32_t n_rows;           // nodes of A's first level (the rows i)
  const uint32_t* a_i;       // A level 0 keys
  const uint32_t* a_off;     // A level 0 child offsets
  const uint32_t* a_j;       // A level 1 keys
  const uint32_t* a_run;     // A bag runs of level 1 (null: one row per node)
  const double* a_val;       // A annotation in trie order (null for COUNT)
  const uint32_t* e_j;       // E level 0 keys
  uint32_t e_n0;
  uint32_t e_dense;          // E's first-level keys are exactly 0 .. e_n0 - 1
  uint64_t e_bsw;            // E root set bitset word (UINT64_MAX: uint layout); both read
  uint32_t e_bsb;            //   from the trie's descriptors by k_inst_roots
  const uint64_t* e_bsw_of;
  const uint32_t* e_bsb_of;
  const uint64_t* e_pool;
  const uint32_t* e_off;     // matrix: E level 0 child offsets
  const uint32_t* e_k;       // matrix: E level 1 keys
  const uint32_t* e_run;     // bag runs of E's last level (null: one row per node)
  const double* e_val;
  int32_t lsb;
  uint32_t D;
  uint32_t sum;
  uint32_t n_k;              // matrix: largest k + 1
  uint64_t row_base;         // first batch row of this instance
  // matrix, inner-product rows: E transposed (levels k, j) and A's j range
  uint32_t n_j;              // largest j of A + 1
  uint32_t bt_n0;            // k nodes of E transposed
  const uint32_t* bt_k;      // their k values
  const uint32_t* bt_off;    // child offsets into bt_j
  const uint32_t* bt_j;      // j of each (k, j)
  const uint32_t* bt_run;    // bag runs of (k, j) into bt_val rows (null: one row each)
  const double* bt_val;      // E's annotation in transposed row order
  uint64_t nnz_e;            // (k, j) pairs of E
};

__device__ __forceinline__ bool find_j(const BInst& I, uint32_t j, uint32_t& pos) {
  if (I.e_dense) {  // E's first level holds every key 0 .. e_n0 - 1: j is its own position
    pos = j;
    return j < I.e_n0;
  }
  if (I.e_n0 == 0) return false;
  if (I.e_bsw != UINT64_MAX) {
    if (j < I.e_bsb || j > I.e_j[I.e_n0 - 1]) return false;
    const uint32_t d = j - I.e_bsb;
    if (!((I.e_pool[I.e_bsw + (d >> 6)] >> (d & 63u)) & 1ull)) return false;
  }
  const uint32_t q = lower_bound_u32(I.e_j, 0, I.e_n0, j);
  if (q < I.e_n0 && I.e_j[q] == j) {
    pos = q;
    return true;
  }
  return false;
}

__device__ __forceinline__ void rows_of(const uint32_t* run, uint32_t node, uint32_t& b, uint32_t& e) {
  if (run) {
    b = run[node];
    e = run[node + 1];
  } else {
    b = node;
    e = node + 1;
  }
}

// ---- setup: per-row product bounds and classes ----------------------------

__global__ void k_inst_roots(BInst* inst, uint32_t n) {
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
    BInst& I = inst[i];
    if (!I.e_n0) continue;
    I.e_bsw = *I.e_bsw_of;
    I.e_bsb = *I.e_bsb_of;
  }
}

// What entries of A's second level contribute to their row.
struct RowTotals {
  uint64_t prod = 0;  // products: pairs of a row of A and a row of E (bags may repeat a key pair on either side)
  uint64_t upd = 0;   // a matrix's scattered updates: rows of A times distinct keys of E (the classes go by these:
                      //   a key's repeated rows are summed where it was found)
};

__device__ __forceinline__ void add_entry(const BInst& I, uint32_t q, RowTotals& r) {
  uint32_t pe;
  if (!find_j(I, I.a_j[q], pe)) return;
  uint32_t ab, ae, eb, ee;
  rows_of(I.a_run, q, ab, ae);
  if (I.kind == 0) {
    rows_of(I.e_run, pe, eb, ee);
  } else {
    eb = I.e_off[pe];
    ee = I.e_off[pe + 1];
    r.upd += (uint64_t)(ae - ab) * (ee - eb);
    if (I.e_run) {
      eb = I.e_run[eb];
      ee = I.e_run[ee];
    }
  }
  r.prod += (uint64_t)(ae - ab) * (ee - eb);
}

// Every row's instance, products and output bound.  A thread walks a row of
// up to ROW_THREAD entries; longer ones are left to its wave, and those past
// ROW_WAVE to its block (a thread walking a power-law hub's row alone took
// 12.5 ms of a 16-instance setup; now 0.1 ms).
constexpr uint32_t ROW_THREAD = 16, ROW_WAVE = 2048;
__global__ __launch_bounds__(B_NT) void k_row_products(const BInst* inst, const uint64_t* inst_row0, uint32_t n_inst,
                                                       uint64_t R, uint32_t* row_inst, uint64_t* prod, uint64_t* upd,
                                                       uint32_t* ub) {
  __shared__ uint32_t s_long[B_NT];
  __shared__ uint32_t s_n;
  __shared__ uint64_t s_red[B_NW];
  const int lane = lane_id();
  for (uint64_t t0 = (uint64_t)blockIdx.x * B_NT; t0 < R; t0 += (uint64_t)gridDim.x * B_NT) {
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    const uint64_t t = t0 + threadIdx.x;
    uint32_t ii = 0, qb = 0, len = 0;
    if (t < R) {
      ii = (uint32_t)upper_bound_minus1<uint64_t>(inst_row0, 0, n_inst, t);
      const uint32_t p = (uint32_t)(t - inst_row0[ii]);
      qb = inst[ii].a_off[p];
      len = inst[ii].a_off[p + 1] - qb;
      row_inst[t] = ii;
    }
    RowTotals u;
    if (len <= ROW_THREAD) {
      for (uint32_t q = qb; q < qb + len; q++) add_entry(inst[ii], q, u);
    } else if (len > ROW_WAVE) {
      s_long[atomicAdd(&s_n, 1u)] = threadIdx.x;
    }
    for (uint64_t m = ballot(len > ROW_THREAD && len <= ROW_WAVE); m; m &= m - 1) {
      const int l = __builtin_ctzll(m);
      const BInst& I = inst[__shfl((int)ii, l, WAVE)];
      const uint32_t b = (uint32_t)__shfl((int)qb, l, WAVE), n = (uint32_t)__shfl((int)len, l, WAVE);
      RowTotals v;
      for (uint32_t k = lane; k < n; k += WAVE) add_entry(I, b + k, v);
      v.prod = wave_sum(v.prod);
      v.upd = wave_sum(v.upd);
      if (lane == l) u = v;
    }
    __syncthreads();
    for (uint32_t i = 0; i < s_n; i++) {  // uniform over the block
      const uint64_t tl = t0 + s_long[i];
      const uint32_t il = (uint32_t)upper_bound_minus1<uint64_t>(inst_row0, 0, n_inst, tl);
      const BInst& I = inst[il];
      const uint32_t p = (uint32_t)(tl - inst_row0[il]);
      const uint32_t b = I.a_off[p], e = I.a_off[p + 1];
      RowTotals v;
      for (uint32_t k = b + threadIdx.x; k < e; k += 4 * B_NT) {
#pragma unroll
        for (int j = 0; j < 4; j++)
          if (k + j * B_NT < e) add_entry(I, k + j * B_NT, v);
      }
      v.prod = block_sum<uint64_t, B_NT>(v.prod, s_red);
      v.upd = block_sum<uint64_t, B_NT>(v.upd, s_red);
      if (threadIdx.x == s_long[i]) u = v;
    }
    if (t < R) {
      prod[t] = u.prod;
      if (upd) upd[t] = u.upd;
      ub[t] = inst[ii].kind == 0 ? 1u : (uint32_t)min<uint64_t>(u.upd, inst[ii].n_k);
    }
    __syncthreads();  // s_long and s_n are free again
  }
}

// The class of every row, by its updates, under a tuning; n_inner[instance] is
// set where the instance has inner-product rows.
__global__ void k_row_classes(const BInst* inst, const uint32_t* row_inst, const uint64_t* upd, uint64_t R,
                              uint32_t light_max, uint32_t inner_ratio, uint32_t* is_heavy, uint32_t* is_light,
                              uint32_t* is_inner, uint32_t* n_inner) {
  for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < R; t += (uint64_t)gridDim.x * blockDim.x) {
    const BInst& I = inst[row_inst[t]];
    const uint64_t u = upd[t];
    const bool heavy = I.kind == 1 && u > light_max;
    // inner-product form when walking all of E costs less than inner_ratio
    // scattered updates per product
    const bool inner = heavy && I.n_j <= KW_MAX && u * inner_ratio >= I.nnz_e;
    is_heavy[t] = heavy && !inner ? 1u : 0u;
    is_light[t] = I.kind == 1 && !heavy ? 1u : 0u;
    is_inner[t] = inner ? 1u : 0u;
    if (inner) n_inner[row_inst[t]] = 1u;
  }
}

// Heavy rows longest first: keys that ascend as products fall.
constexpr uint32_t HEAVY_KEY_BITS = 40;
__global__ void k_heavy_keys(const uint32_t* rows, uint64_t n, const uint64_t* prod, uint64_t* key) {
  constexpr uint64_t top = (1ull << HEAVY_KEY_BITS) - 1;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    key[i] = top - min(prod[rows[i]], top);
}

__global__ void k_fill_u32_dev(uint32_t* p, uint32_t v, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) p[i] = v;
}

// ---- the persistent kernel -------------------------------------------------------

struct BatchArgs {
  const BInst* inst;
  const uint32_t* row_inst;
  const uint64_t* inst_row0;
  const uint64_t* ub_off;    // per batch row: first upper-bound output slot
  const uint32_t* heavy;     // heavy rows, longest first
  uint64_t n_heavy;
  const uint32_t* light;     // light rows
  uint64_t n_light;
  const uint32_t* inner;     // inner-product rows, grouped by instance
  uint64_t n_inner;
  uint32_t* qhead;           // [0] heavy queue, [1] light queue, [2] inner queue, [3] long vector rows
  uint32_t* row_nnz;         // outputs per row
  uint32_t* ub_k;
  uint64_t* ub_cnt;
  double* ub_sum;
  uint32_t* err;
  const uint64_t* prod;      // per batch row: its number of products
  uint32_t kw;                      // k values per heavy window (multiple of 64, <= KW_MAX)
};

// LDS accumulators of the heavy and inner kernels sit DSTRIDE 8-byte slots
// apart: with 9 (72 bytes), the same digit of different accumulators falls
// in different LDS banks (at 8, 64 bytes apart, every accumulator's digit k
// shared two banks and the atomics of a wave serialized on them).
constexpr int DSTRIDE = EXACT_MAXD + 1;

// A row with fewer products than this keeps its LDS accumulators in signed
// slots: a product adds two terms, each at most one word below 2^32 to any
// slot, so no slot can leave int64 (2 * 2^30 * 2^32 = 2^63).
constexpr uint64_t BOUNDED_PRODUCTS = SIGNED_TERMS;

// Exact sum held in the LDS slots (digits) of one accumulator: add v.
// bounded (the row has fewer than BOUNDED_PRODUCTS products): signed slots,
// plain atomic adds whose returned values nobody waits for.  Otherwise the
// shared slot form, which carries every wrap, so any number of terms is
// exact.  A row uses one form for all of its accumulators.
__device__ __forceinline__ bool lds_add_term(long long* slots, double v, int32_t lsb, uint32_t D, bool bounded) {
  return bounded ? signed_add_term((int64_t*)slots, v, lsb, D, 1) : atomic_add_term((int64_t*)slots, v, lsb, D, 1);
}

// The correctly rounded value of an LDS accumulator in the form lds_add_term
// used: signed slots are carried into digits first (a normalized value is
// also a shared-form value).
__device__ __forceinline__ double lds_round(const long long* slots, uint32_t D, int32_t lsb, bool bounded,
                                            uint32_t* err) {
  if (!bounded) return exact_round((const int64_t*)slots, D, lsb, err);
  RegAcc r;
  r.load_signed((const int64_t*)slots, D);
  return exact_round(r.s, D, lsb, err);
}

// Heavy rows: one block per row.  A symbolic pass marks every k the row
// produces in an LDS bitmap (per window of kw values of k); per-word
// popcount prefixes give each k its rank, which is also its place in the
// row's sorted output.  The ranks are then taken HC at a time: the k range
// of the rank window is found from the bitmap, every B row is cut to that
// range by two binary searches, and the products in it add their exact
// digits to LDS accumulators indexed by rank - r0, which are emitted in
// order and cleared.  No global atomics.  In both passes the products of
// B_NT entries of A's row at a time are numbered by a block scan and dealt
// out evenly to the threads.  A row of at most CUR_MAX entries whose
// outputs take several rank windows keeps, per entry of A, a cursor into
// its E row in LDS: windows are taken in increasing k, so each window's
// products of an entry start at its cursor and end where a short gallop
// finds the window's upper k; neither j's lookup nor the two binary
// searches are repeated per window.
constexpr uint32_t HC = 512;
constexpr uint32_t CUR_MAX = 2048;

// First position in [b, e) of the sorted a holding a value >= x, found by
// galloping from b (most windows take few products of one entry).
__device__ __forceinline__ uint32_t gallop_lower_bound(const uint32_t* a, uint32_t b, uint32_t e, uint32_t x) {
  if (b >= e || a[b] >= x) return b;
  uint32_t lo = b, step = 1;   // a[lo] < x
  while (lo + step < e && a[lo + step] < x) {
    lo += step;
    step <<= 1;
  }
  return lower_bound_u32(a, lo + 1, min(lo + step, e), x);
}

__device__ __forceinline__ uint32_t rank_select(const unsigned long long* bm, const uint32_t* pre, uint32_t nwords,
                                                uint32_t r) {
  // the k whose rank is r: the word holding the r-th set bit, then the bit
  uint32_t w = 0, n = nwords;
  while (n > 1) {
    const uint32_t half = n >> 1;
    w = (pre[w + half] <= r) ? w + half : w;
    n -= half;
  }
  uint64_t word = bm[w];
  for (uint32_t i = pre[w]; i < r; i++) word &= word - 1;
  return w * 64 + (uint32_t)__builtin_ctzll(word);
}

__global__ __launch_bounds__(B_NT) void k_batch_heavy(BatchArgs a) {
  __shared__ unsigned long long bm[KW_MAX / 64];   // k the row touches in the window
  __shared__ uint32_t pre[KW_MAX / 64];            // set bits before each word
  __shared__ uint32_t sk[HC];
  __shared__ unsigned long long scnt[HC];
  __shared__ long long sdig[HC * DSTRIDE];
  __shared__ uint32_t s_item, s_klo, s_khi;
  __shared__ uint32_t s_wsum[B_NW];
  // products of a batch of B_NT entries of A's row, numbered by a block
  // scan so that every thread takes an equal share (E's rows have skewed
  // lengths, and one thread per entry would wait on the longest)
  __shared__ uint32_t s_off[B_NT], s_kb[B_NT], s_ab[B_NT], s_ae[B_NT];
  __shared__ uint32_t s_cur[CUR_MAX], s_cend[CUR_MAX];   // per entry of A: its E row, from the next window on
  const int tid = threadIdx.x;
  uint32_t bad = 0;
  // owner of product idx: the last entry whose first product is <= idx
  auto owner = [&](uint32_t idx) {
    uint32_t lo = 0, n = B_NT;
    while (n > 1) {
      const uint32_t half = n >> 1;
      lo = (s_off[lo + half] <= idx) ? lo + half : lo;
      n -= half;
    }
    return lo;
  };
  for (uint32_t sl = tid; sl < HC; sl += B_NT) {
    scnt[sl] = 0;
#pragma unroll
    for (int d = 0; d < EXACT_MAXD; d++) sdig[sl * DSTRIDE + d] = 0;
  }
  for (;;) {
    if (tid == 0) s_item = atomicAdd(&a.qhead[0], 1u);
    __syncthreads();
    // uniform across the block: the row's descriptor goes to scalar registers
    const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
    __syncthreads();
    if (item >= a.n_heavy) break;
    const uint32_t t = __builtin_amdgcn_readfirstlane(a.heavy[item]);
    const BInst I = a.inst[a.row_inst[t]];
    const uint32_t p = t - (uint32_t)a.inst_row0[a.row_inst[t]];
    const uint32_t qb = I.a_off[p], qe = I.a_off[p + 1];
    const uint64_t out = a.ub_off[t];
    const bool bounded = a.prod[t] < BOUNDED_PRODUCTS;
    uint32_t nnz = 0;
    for (uint32_t w0 = 0; w0 < I.n_k; w0 += a.kw) {
      const uint32_t wend = min(w0 + a.kw, I.n_k);
      const uint32_t nwords = (wend - w0 + 63) / 64;
      for (uint32_t sl = tid; sl < nwords; sl += B_NT) bm[sl] = 0;
      __syncthreads();
      for (uint32_t qs = qb; qs < qe; qs += B_NT) {
        const uint32_t q = qs + tid;
        uint32_t cnt = 0, kb = 0;
        uint32_t pe;
        if (q < qe && find_j(I, I.a_j[q], pe)) {
          kb = I.e_off[pe];
          uint32_t kend = I.e_off[pe + 1];
          if (I.n_k > a.kw) {
            kb = lower_bound_u32(I.e_k, kb, kend, w0);
            kend = lower_bound_u32(I.e_k, kb, kend, wend);
          }
          cnt = kend - kb;
        }
        uint32_t tot;
        const uint32_t off = block_excl_scan<uint32_t, B_NT>(cnt, s_wsum, tot);
        s_off[tid] = off;
        s_kb[tid] = kb;
        __syncthreads();
        for (uint32_t idx = tid; idx < tot; idx += B_NT) {
          const uint32_t o = owner(idx);
          const uint32_t k = I.e_k[s_kb[o] + (idx - s_off[o])] - w0;
          atomicOr(&bm[k >> 6], 1ull << (k & 63u));
        }
        __syncthreads();
      }
      uint32_t m;
      {
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const uint32_t wi = 4 * tid + i;
          c += wi < nwords ? (uint32_t)__popcll(bm[wi]) : 0u;
        }
        uint32_t r = block_excl_scan<uint32_t, B_NT>(c, s_wsum, m);
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const uint32_t wi = 4 * tid + i;
          if (wi < nwords) {
            pre[wi] = r;
            r += (uint32_t)__popcll(bm[wi]);
          }
        }
      }
      // cursors: several rank windows over one k window, few enough entries
      const bool cursors = m > HC && I.n_k <= a.kw && qe - qb <= CUR_MAX;
      if (cursors) {
        for (uint32_t q = qb + tid; q < qe; q += B_NT) {
          uint32_t pe, b = 0, e = 0;
          if (find_j(I, I.a_j[q], pe)) {
            b = I.e_off[pe];
            e = I.e_off[pe + 1];
          }
          s_cur[q - qb] = b;
          s_cend[q - qb] = e;
        }
      }
      __syncthreads();
      for (uint32_t r0 = 0; r0 < m; r0 += HC) {
        if (tid == 0) {
          s_klo = rank_select(bm, pre, nwords, r0);
          s_khi = r0 + HC < m ? rank_select(bm, pre, nwords, r0 + HC) : wend - w0;
        }
        __syncthreads();
        const uint32_t klo = s_klo + w0, khi = s_khi + w0;
        for (uint32_t qs = qb; qs < qe; qs += B_NT) {
          const uint32_t q = qs + tid;
          uint32_t cnt = 0, kb = 0, ab = 0, ae = 0;
          uint32_t pe;
          if (cursors) {
            if (q < qe) {
              // this thread alone reads and advances entry q's cursor
              kb = s_cur[q - qb];
              const uint32_t kend = gallop_lower_bound(I.e_k, kb, s_cend[q - qb], khi);
              s_cur[q - qb] = kend;
              cnt = kend - kb;
              if (cnt) rows_of(I.a_run, q, ab, ae);
            }
          } else if (q < qe && find_j(I, I.a_j[q], pe)) {
            rows_of(I.a_run, q, ab, ae);
            kb = I.e_off[pe];
            uint32_t kend = I.e_off[pe + 1];
            if (m > HC || I.n_k > a.kw) {
              kb = lower_bound_u32(I.e_k, kb, kend, klo);
              kend = lower_bound_u32(I.e_k, kb, kend, khi);
            }
            cnt = kend - kb;
          }
          uint32_t tot;
          const uint32_t off = block_excl_scan<uint32_t, B_NT>(cnt, s_wsum, tot);
          s_off[tid] = off;
          s_kb[tid] = kb;
          s_ab[tid] = ab;
          s_ae[tid] = ae;
          __syncthreads();
          for (uint32_t idx = tid; idx < tot; idx += B_NT) {
            const uint32_t own = owner(idx);
            const uint32_t kp = s_kb[own] + (idx - s_off[own]);
            const uint32_t ab = s_ab[own], ae = s_ae[own];
            const uint32_t k = I.e_k[kp] - w0;
            const uint64_t word = bm[k >> 6];
            const uint32_t sl = pre[k >> 6] + (uint32_t)__popcll(word & ((1ull << (k & 63u)) - 1ull)) - r0;
            sk[sl] = k + w0;
            uint32_t eb, ee;
            rows_of(I.e_run, kp, eb, ee);
            atomicAdd(&scnt[sl], (unsigned long long)(ae - ab) * (ee - eb));
            if (I.sum)
              for (uint32_t ra = ab; ra < ae; ra++)
                for (uint32_t re = eb; re < ee; re++) {
                  double hi, lo;
                  two_prod(I.a_val[ra], I.e_val[re], hi, lo);
                  bool ok = lds_add_term(sdig + sl * DSTRIDE, hi, I.lsb, I.D, bounded);
                  ok = lds_add_term(sdig + sl * DSTRIDE, lo, I.lsb, I.D, bounded) && ok;
                  if (!ok) bad = 1;
                }
          }
          __syncthreads();
        }
        __syncthreads();
        const uint32_t nw = min(HC, m - r0);
        for (uint32_t sl = tid; sl < nw; sl += B_NT) {
          const uint64_t o = out + nnz + r0 + sl;
          a.ub_k[o] = sk[sl];
          a.ub_cnt[o] = scnt[sl];
          if (I.sum) a.ub_sum[o] = lds_round(sdig + sl * DSTRIDE, I.D, I.lsb, bounded, a.err);
          scnt[sl] = 0;
#pragma unroll
          for (int d = 0; d < EXACT_MAXD; d++) sdig[sl * DSTRIDE + d] = 0;
        }
        __syncthreads();
      }
      nnz += m;
    }
    if (tid == 0) a.row_nnz[t] = nnz;
  }
  if (bad) atomicOr(a.err, 1u);
}

// The products of one matched entry e (with j) of an inner-product row into
// its column's LDS accumulator.
__device__ __forceinline__ void inner_product(const BInst& I, uint32_t e, uint32_t j,
                                              const unsigned long long* bm,
                                              const uint32_t* pre, const uint32_t* soff, uint32_t nk, uint32_t qb,
                                              unsigned long long* ccnt, long long* cdig, bool bounded, uint32_t& bad) {
  // column of entry e: the last c with soff[c] <= e
  uint32_t c = 0, n = nk;
  while (n > 1) {
    const uint32_t half = n >> 1;
    c = (soff[c + half] <= e) ? c + half : c;
    n -= half;
  }
  const uint64_t word = bm[j >> 6];
  const uint32_t q = qb + pre[j >> 6] + (uint32_t)__popcll(word & ((1ull << (j & 63u)) - 1ull));
  uint32_t ab, ae, eb, ee;
  rows_of(I.a_run, q, ab, ae);
  rows_of(I.bt_run, e, eb, ee);
  atomicAdd(&ccnt[c], (unsigned long long)(ae - ab) * (ee - eb));
  if (!I.sum) return;
  for (uint32_t ra = ab; ra < ae; ra++)
    for (uint32_t re = eb; re < ee; re++) {
      double hi, lo;
      two_prod(I.a_val[ra], I.bt_val[re], hi, lo);
      bool ok = lds_add_term(cdig + c * DSTRIDE, hi, I.lsb, I.D, bounded);
      ok = lds_add_term(cdig + c * DSTRIDE, lo, I.lsb, I.D, bounded) && ok;
      if (!ok) bad = 1;
    }
}

// Inner-product rows: one block per row.  A's row is marked in an LDS
// bitmap over j with per-word rank prefixes (the position of j in the row).
// E transposed is then streamed chunk by chunk (I_NT columns k at a time):
// the block's threads take the chunk's (k, j) entries in order, coalesced
// and independent, probe j in the bitmap and queue the matching entries;
// full waves of them then add each product's exact digits to its column's
// LDS accumulator (the column found by bisecting the chunk's offsets); the
// columns are then emitted in k order and their accumulators cleared.
// Threads of a block, columns of a chunk: a row is one block's, and its
// stream of E's entries is a chain of load latencies, so a block is large.
constexpr int I_NT = 1024;
constexpr int I_NW = I_NT / WAVE;
constexpr int I_WPT = (int)(KW_MAX / 64) / I_NT;  // bitmap words per thread
static_assert(I_WPT >= 1 && I_WPT * I_NT == (int)(KW_MAX / 64), "bitmap words per thread");
__global__ __launch_bounds__(I_NT) void k_batch_inner(BatchArgs a) {
  __shared__ unsigned long long bm[KW_MAX / 64];
  __shared__ uint32_t pre[KW_MAX / 64];
  __shared__ uint32_t soff[I_NT + 1];                 // the chunk's column offsets
  __shared__ unsigned long long ccnt[I_NT];           // per column of the chunk
  __shared__ long long cdig[I_NT * DSTRIDE];
  __shared__ uint32_t s_qe[I_NW][2 * WAVE], s_qj[I_NW][2 * WAVE];  // matched entries waiting, per wave
  __shared__ uint32_t s_item;
  __shared__ uint32_t s_wsum[I_NW];
  const int tid = threadIdx.x, w = tid / WAVE, lane = lane_id();
  uint32_t bad = 0;
  ccnt[tid] = 0;
#pragma unroll
  for (int d = 0; d < EXACT_MAXD; d++) cdig[tid * DSTRIDE + d] = 0;
  for (;;) {
    if (tid == 0) s_item = atomicAdd(&a.qhead[2], 1u);
    __syncthreads();
    const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
    __syncthreads();
    if (item >= a.n_inner) break;
    const uint32_t t = __builtin_amdgcn_readfirstlane(a.inner[item]);
    const BInst I = a.inst[a.row_inst[t]];
    const uint32_t p = t - (uint32_t)a.inst_row0[a.row_inst[t]];
    const uint32_t qb = I.a_off[p], qe = I.a_off[p + 1];
    const bool bounded = a.prod[t] < BOUNDED_PRODUCTS;
    const uint32_t nwords = (I.n_j + 63) / 64;
    for (uint32_t s = tid; s < nwords; s += I_NT) bm[s] = 0;
    __syncthreads();
    for (uint32_t q = qb + tid; q < qe; q += I_NT) {
      const uint32_t j = I.a_j[q];
      atomicOr(&bm[j >> 6], 1ull << (j & 63u));
    }
    __syncthreads();
    {
      uint32_t c = 0;
#pragma unroll
      for (int i = 0; i < I_WPT; i++) {
        const uint32_t wi = I_WPT * tid + i;
        c += wi < nwords ? (uint32_t)__popcll(bm[wi]) : 0u;
      }
      uint32_t tot;
      uint32_t r = block_excl_scan<uint32_t, I_NT>(c, s_wsum, tot);
#pragma unroll
      for (int i = 0; i < I_WPT; i++) {
        const uint32_t wi = I_WPT * tid + i;
        if (wi < nwords) {
          pre[wi] = r;
          r += (uint32_t)__popcll(bm[wi]);
        }
      }
    }
    const uint64_t out = a.ub_off[t];
    uint32_t nnz = 0;
    for (uint32_t kb0 = 0; kb0 < I.bt_n0; kb0 += I_NT) {
      const uint32_t nk = min((uint32_t)I_NT, I.bt_n0 - kb0);
      soff[tid] = I.bt_off[kb0 + min((uint32_t)tid, nk)];
      if (tid == 0) soff[I_NT] = I.bt_off[kb0 + nk];
      __syncthreads();
      const uint32_t e0 = soff[0], e1 = soff[nk];
      // Four entries per thread per round: their loads are independent and
      // in flight together.  Entries whose j the row holds (2 to 30% of
      // them) are queued per wave in LDS and worked on 64 at a time: worked
      // on where they were found, nearly every wave ran the whole product
      // path for one or two lanes (6.1 ms of a 16-instance batch).
      // With blocks of 1024 threads for 256: 2.1 ms.
      constexpr uint32_t UNR = 4;
      uint32_t qn = 0;  // queued entries (uniform over the wave)
      for (uint32_t eb = e0 + tid; eb - lane < e1; eb += UNR * I_NT) {
        uint32_t jv[UNR];
#pragma unroll
        for (uint32_t u = 0; u < UNR; u++) {
          const uint32_t e = eb + u * I_NT;
          jv[u] = e < e1 ? I.bt_j[e] : UINT32_MAX;
        }
#pragma unroll
        for (uint32_t u = 0; u < UNR; u++) {
          const uint32_t j = jv[u];
          const bool hit = j < I.n_j && ((bm[j >> 6] >> (j & 63u)) & 1ull);
          const uint64_t hits = ballot(hit);
          if (hit) {
            const uint32_t at = qn + lanes_below(hits);
            s_qe[w][at] = eb + u * I_NT;
            s_qj[w][at] = j;
          }
          qn += (uint32_t)__popcll(hits);
          if (qn >= WAVE) {
            wave_lds_sync();
            inner_product(I, s_qe[w][lane], s_qj[w][lane], bm, pre, soff, nk, qb, ccnt, cdig, bounded, bad);
            qn -= WAVE;
            wave_lds_sync();
            if (lane < (int)qn) {
              s_qe[w][lane] = s_qe[w][WAVE + lane];
              s_qj[w][lane] = s_qj[w][WAVE + lane];
            }
            wave_lds_sync();
          }
        }
      }
      wave_lds_sync();
      if (lane < (int)qn) inner_product(I, s_qe[w][lane], s_qj[w][lane], bm, pre, soff, nk, qb, ccnt, cdig, bounded, bad);
      __syncthreads();
      const uint64_t cnt = (uint32_t)tid < nk ? ccnt[tid] : 0ull;
      uint32_t tot;
      const uint32_t r = block_excl_scan<uint32_t, I_NT>(cnt ? 1u : 0u, s_wsum, tot);
      if (cnt) {
        const uint64_t o = out + nnz + r;
        a.ub_k[o] = I.bt_k[kb0 + tid];
        a.ub_cnt[o] = cnt;
        if (I.sum) a.ub_sum[o] = lds_round(cdig + tid * DSTRIDE, I.D, I.lsb, bounded, a.err);
      }
      ccnt[tid] = 0;
#pragma unroll
      for (int d = 0; d < EXACT_MAXD; d++) cdig[tid * DSTRIDE + d] = 0;
      nnz += tot;
      __syncthreads();
    }
    if (tid == 0) a.row_nnz[t] = nnz;
    __syncthreads();
  }
  if (bad) atomicOr(a.err, 1u);
}

constexpr uint32_t LIGHT_GRAB = 32;

// Light rows: one wave per row, private LDS hash of HS slots.
template <int HS>
__global__ __launch_bounds__(B_NT) void k_batch_light(BatchArgs a) {
  constexpr int SLOT_BYTES = 4 + 8 + 8 * EXACT_MAXD + 2;
  constexpr uint32_t HS_SHIFT = HS == 128 ? 25 : 24;  // top bits of the multiplicative hash
  static_assert(HS == 128 || HS == 256, "hash size");
  __shared__ __align__(16) unsigned char lds[B_NW * HS * SLOT_BYTES];
  const int tid = threadIdx.x, w = tid / WAVE, lane = lane_id();
  uint32_t bad = 0;
  uint32_t* hk = (uint32_t*)(lds + w * HS * SLOT_BYTES);
  unsigned long long* hc = (unsigned long long*)(hk + HS);
  long long* hd = (long long*)(hc + HS);
  uint16_t* hl = (uint16_t*)(hd + HS * EXACT_MAXD);
  // Light rows are claimed LIGHT_GRAB at a time: one atomic on the queue
  // head per claim (a head taken once per row serializes millions of rows).
  uint32_t item = 0, item_end = 0;
  for (;;) {
    if (item == item_end) {
      uint32_t g = 0;
      if (lane == 0) g = atomicAdd(&a.qhead[1], LIGHT_GRAB);
      item = __builtin_amdgcn_readfirstlane(__shfl(g, 0, WAVE));
      item_end = (uint32_t)min<uint64_t>((uint64_t)item + LIGHT_GRAB, a.n_light);
    }
    if (item >= a.n_light) break;
    const uint32_t t = __builtin_amdgcn_readfirstlane(a.light[item]);
    item++;
    const BInst I = a.inst[a.row_inst[t]];
    const uint32_t p = t - (uint32_t)a.inst_row0[a.row_inst[t]];
    const uint32_t qb = I.a_off[p], qe = I.a_off[p + 1];
    const uint64_t out = a.ub_off[t];
    // matrix: hash the row's products by k
    const bool bounded = a.prod[t] < BOUNDED_PRODUCTS;
    for (int s = lane; s < HS; s += WAVE) {
      hk[s] = EMPTY_KEY;
      hc[s] = 0;
#pragma unroll
      for (int d = 0; d < EXACT_MAXD; d++) hd[s * EXACT_MAXD + d] = 0;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // The row's products are spread over the lanes: per chunk of 64 A
    // entries, a scan of their B-row lengths numbers the products, and
    // each lane takes products f, f + 64, ... (finding its A entry by
    // bisecting the scan across lanes), so all loads are independent.
    for (uint32_t c0 = qb; c0 < qe; c0 += WAVE) {
      const uint32_t q = c0 + lane;
      uint32_t pe = 0, len = 0, kb = 0;
      if (q < qe && find_j(I, I.a_j[q], pe)) {
        kb = I.e_off[pe];
        len = I.e_off[pe + 1] - kb;
      }
      const uint32_t incl = wave_incl_scan(len);
      const uint32_t start = incl - len;
      const uint32_t total = (uint32_t)__shfl((int)incl, WAVE - 1, WAVE);
      for (uint32_t f0 = 0; f0 < total; f0 += WAVE) {   // uniform: every lane takes part in the shuffles
        const uint32_t f = f0 + lane;
        // owner: the last lane whose start <= f (lanes with len 0 share a start)
        uint32_t src = 0, n = WAVE;
#pragma unroll
        for (int step = 0; step < 6; step++) {
          const uint32_t half = n >> 1;
          const uint32_t st = (uint32_t)__shfl((int)start, (int)(src + half), WAVE);
          src = st <= f ? src + half : src;
          n -= half;
        }
        const uint32_t kbs = (uint32_t)__shfl((int)kb, (int)src, WAVE);
        const uint32_t sts = (uint32_t)__shfl((int)start, (int)src, WAVE);
        if (f >= total) continue;
        const uint32_t qq = c0 + src;
        const uint32_t kp = kbs + (f - sts);
        uint32_t ab, ae;
        rows_of(I.a_run, qq, ab, ae);
        const uint32_t k = I.e_k[kp];
        uint32_t slot = (k * 2654435761u) >> HS_SHIFT;
        for (;;) {
          const uint32_t prev = atomicCAS(&hk[slot], EMPTY_KEY, k);
          if (prev == EMPTY_KEY || prev == k) break;
          slot = (slot + 1) & (HS - 1);
        }
        uint32_t eb, ee;
        rows_of(I.e_run, kp, eb, ee);
        atomicAdd(&hc[slot], (unsigned long long)(ae - ab) * (ee - eb));
        if (I.sum)
          for (uint32_t ra = ab; ra < ae; ra++)
            for (uint32_t re = eb; re < ee; re++) {
              double hi, lo;
              two_prod(I.a_val[ra], I.e_val[re], hi, lo);
              bool ok = lds_add_term(hd + slot * EXACT_MAXD, hi, I.lsb, I.D, bounded);
              ok = lds_add_term(hd + slot * EXACT_MAXD, lo, I.lsb, I.D, bounded) && ok;
              if (!ok) bad = 1;
            }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // list the occupied slots, then place each by its rank in k order
    uint32_t m = 0;
    for (int s0 = 0; s0 < HS; s0 += WAVE) {
      const bool occ = hk[s0 + lane] != EMPTY_KEY;
      const uint64_t bal = ballot(occ);
      if (occ) hl[m + lanes_below(bal)] = (uint16_t)(s0 + lane);
      m += (uint32_t)__popcll(bal);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // rank of each listed key among the listed keys: lane holds entries
    // lane + 64 c in registers; every key is broadcast once by a shuffle
    constexpr int NC = HS / WAVE;
    uint32_t kk[NC], ss[NC], rk[NC];
#pragma unroll
    for (int c = 0; c < NC; c++) {
      const uint32_t f = c * WAVE + lane;
      ss[c] = f < m ? hl[f] : 0u;
      kk[c] = f < m ? hk[ss[c]] : EMPTY_KEY;
      rk[c] = 0;
    }
#pragma unroll
    for (int c2 = 0; c2 < NC; c2++) {
      if ((uint32_t)c2 * WAVE >= m) break;
      const uint32_t n2 = min((uint32_t)WAVE, m - (uint32_t)c2 * WAVE);
      for (uint32_t j = 0; j < n2; j++) {
        const uint32_t kf = (uint32_t)__shfl((int)kk[c2], (int)j, WAVE);
#pragma unroll
        for (int c = 0; c < NC; c++) rk[c] += kf < kk[c] ? 1u : 0u;
      }
    }
#pragma unroll
    for (int c = 0; c < NC; c++) {
      if ((uint32_t)c * WAVE + lane >= m) continue;
      const uint32_t s = ss[c];
      const uint64_t o = out + rk[c];
      a.ub_k[o] = kk[c];
      a.ub_cnt[o] = hc[s];
      if (I.sum) a.ub_sum[o] = lds_round(hd + s * EXACT_MAXD, I.D, I.lsb, bounded, a.err);
    }
    if (lane == 0) a.row_nnz[t] = m;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  if (bad) atomicOr(a.err, 1u);
}

// ---- vector rows ------------------------------------------------------------

// Products of A's entries qb + from, qb + from + step, ... below qe.
__device__ __forceinline__ void vector_products(const BInst& I, uint32_t qb, uint32_t qe, uint32_t from, uint32_t step,
                                                uint64_t& cnt, RegAcc& acc, uint32_t& bad) {
  for (uint32_t q = qb + from; q < qe; q += step) {
    uint32_t pe;
    if (!find_j(I, I.a_j[q], pe)) continue;
    uint32_t ab, ae, eb, ee;
    rows_of(I.a_run, q, ab, ae);
    rows_of(I.e_run, pe, eb, ee);
    cnt += (uint64_t)(ae - ab) * (ee - eb);
    if (!I.sum) continue;
    for (uint32_t ra = ab; ra < ae; ra++)
      for (uint32_t re = eb; re < ee; re++) {
        double hi, lo;
        two_prod(I.a_val[ra], I.e_val[re], hi, lo);
        bool ok = acc.add(hi, I.lsb, I.D, 1);
        ok = acc.add(lo, I.lsb, I.D, 1) && ok;
        if (!ok) bad = 1;
      }
  }
}

// A vector row's single output, by the thread that holds its sums.
__device__ __forceinline__ void vector_output(const BatchArgs& a, const BInst& I, uint64_t t, uint64_t cnt,
                                              const int64_t* digits) {
  if (cnt) {
    const uint64_t out = a.ub_off[t];
    a.ub_k[out] = 0;
    a.ub_cnt[out] = cnt;
    if (I.sum) a.ub_sum[out] = exact_round(digits, I.D, I.lsb, a.err);
  }
  a.row_nnz[t] = cnt ? 1u : 0u;
}

// Rows of vector instances: eight lanes take a row of up to VEC_SHORT
// entries (most rows of a power-law matrix hold one to three, and a wave
// each spent itself on reducing them); longer rows are listed.
constexpr uint32_t VEC_SHORT = 128;
__global__ __launch_bounds__(B_NT) void k_batch_vec(BatchArgs a, uint64_t R, uint32_t* longs) {
  constexpr int LPR = 8;
  const int l = lane_id() % LPR;
  uint32_t bad = 0;
  for (uint64_t t = ((uint64_t)blockIdx.x * B_NT + threadIdx.x) / LPR; t < R;
       t += (uint64_t)gridDim.x * (B_NT / LPR)) {  // (a row's lanes stay together)
    const uint32_t ii = a.row_inst[t];
    const BInst& I = a.inst[ii];
    if (I.kind != 0) continue;
    const uint32_t p = (uint32_t)(t - a.inst_row0[ii]);
    const uint32_t qb = I.a_off[p], qe = I.a_off[p + 1];
    if (qe - qb > VEC_SHORT) {
      if (l == 0) longs[atomicAdd(&a.qhead[3], 1u)] = (uint32_t)t;
      continue;
    }
    RegAcc acc;
    acc.clear();
    uint64_t cnt = 0;
    vector_products(I, qb, qe, (uint32_t)l, LPR, cnt, acc, bad);
    cnt = unit_sum<LPR>(cnt);
    if (I.sum) {
      acc.normalize(I.D);
#pragma unroll
      for (int i = 0; i < EXACT_MAXD; i++) acc.s[i] = unit_sum<LPR>(acc.s[i]);
    }
    // (sums of normalized digits: below 2^35, a valid shared-form value)
    if (l == 0) vector_output(a, I, t, cnt, acc.s);
  }
  if (bad) atomicOr(a.err, 1u);
}

// The listed long rows, a block each.
__global__ __launch_bounds__(B_NT) void k_batch_vec_long(BatchArgs a, const uint32_t* longs) {
  __shared__ int64_t s_red[B_NW];
  const uint32_t n = a.qhead[3];
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const uint32_t t = longs[i];
    const uint32_t ii = a.row_inst[t];
    const BInst& I = a.inst[ii];
    const uint32_t p = t - (uint32_t)a.inst_row0[ii];
    RegAcc acc;
    acc.clear();
    uint64_t cnt = 0;
    uint32_t bad = 0;
    vector_products(I, I.a_off[p], I.a_off[p + 1], threadIdx.x, B_NT, cnt, acc, bad);
    if (bad) atomicOr(a.err, 1u);
    cnt = (uint64_t)block_sum<int64_t, B_NT>((int64_t)cnt, s_red);
    acc.normalize(I.D);
#pragma unroll
    for (int q = 0; q < EXACT_MAXD; q++) acc.s[q] = block_sum<int64_t, B_NT>(acc.s[q], s_red);
    if (threadIdx.x == 0) vector_output(a, I, t, cnt, acc.s);
  }
}

// Copy each row's outputs from its upper-bound slots to the packed result.
struct PackArgs2 {
  const BInst* inst;
  const uint32_t* row_inst;
  const uint64_t* inst_row0;
  const uint64_t* ub_off;
  const uint64_t* out_off;   // exclusive scan of row_nnz
  const uint32_t* ub_k;
  const uint64_t* ub_cnt;
  const double* ub_sum;
  uint32_t* out_i;
  uint32_t* out_k;
  uint64_t* out_cnt;
  double* out_sum;
  uint64_t R;
};

// A wave takes PACK_SPAN consecutive outputs (rows may hold none or tens of
// thousands: a wave per 64 rows waited for its hub rows).  It finds its first
// output's row by bisection; 64 outputs at a time, the offsets of the 64
// rows from the current one are loaded by the lanes and each lane finds its
// output's row among them by bisecting across the lanes.  Rows without
// outputs leave the row further on: PACK_WINDOWS windows are looked at, then
// each lane bisects the offsets itself (3150 outputs of two 2 M-row matrices:
// 31.5 ms a call walking every window, 0.86 with the bisection, 5.2 with a
// wave per 64 rows).
constexpr uint32_t PACK_SPAN = 2048;
constexpr int PACK_WINDOWS = 4;
__global__ __launch_bounds__(B_NT) void k_pack_rows(PackArgs2 a, uint64_t total) {
  const int lane = lane_id();
  const uint64_t wave = ((uint64_t)blockIdx.x * B_NT + threadIdx.x) / WAVE;
  const uint64_t base = wave * PACK_SPAN;
  if (base >= total) return;
  const uint64_t end = min<uint64_t>(total, base + PACK_SPAN);
  uint64_t r0 = upper_bound_minus1<uint64_t>(a.out_off, 0, a.R, base);
  for (uint64_t e0 = base; e0 < end; e0 += WAVE) {   // uniform: every lane takes part in the shuffles
    const uint64_t e = min<uint64_t>(e0 + lane, end - 1);
    uint64_t row = 0;
    bool found = false;
    uint64_t rw = r0;
    for (int win = 0; win < PACK_WINDOWS && !__all(found); win++, rw += WAVE) {
      // offsets of rows rw .. rw + 63 (past the last row: the end), and the
      // next window's first
      const uint64_t off = a.out_off[min<uint64_t>(rw + lane, a.R)];
      const uint64_t next = a.out_off[min<uint64_t>(rw + WAVE, a.R)];
      uint32_t src = 0;
#pragma unroll
      for (int step = WAVE / 2; step > 0; step >>= 1) {
        const uint64_t o = (uint64_t)__shfl((unsigned long long)off, (int)(src + step), WAVE);
        src = o <= e ? src + step : src;
      }
      if (!found && (next > e || rw + WAVE >= a.R)) {
        row = min<uint64_t>(rw + src, a.R - 1);
        found = true;
      }
    }
    // (rw is below R here: a window that reaches R finds every lane's row)
    if (!found) row = upper_bound_minus1<uint64_t>(a.out_off, rw, a.R, e);
    const uint32_t ii = a.row_inst[row];
    const BInst& I = a.inst[ii];
    const uint32_t iv = I.a_i[row - a.inst_row0[ii]];
    const uint64_t u = a.ub_off[row] + (e - a.out_off[row]);
    if (e0 + lane < end) {
      a.out_i[e] = iv;
      if (I.kind == 1) a.out_k[e] = a.ub_k[u];
      a.out_cnt[e] = a.ub_cnt[u];
      if (I.sum) a.out_sum[e] = a.ub_sum[u];
    }
    r0 = (uint64_t)__shfl((unsigned long long)row, WAVE - 1, WAVE);
  }
}

// Join tuples of each instance (one block per instance): the sum of its
// rows' product counts, which is the sum of its output counts.
__global__ void k_inst_sums(const uint64_t* prod, const uint64_t* row0, uint64_t* out) {
  __shared__ uint64_t red[B_NW];
  uint64_t s = 0;
  for (uint64_t t = row0[blockIdx.x] + threadIdx.x; t < row0[blockIdx.x + 1]; t += blockDim.x) s += prod[t];
  s = block_sum<uint64_t, B_NT>(s, red);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// Packed output offsets at the instances' first rows (n + 1 of them).
__global__ void k_inst_offsets(const uint64_t* out_off, const uint64_t* row0, uint32_t n, uint64_t* dst) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i <= n; i += gridDim.x * blockDim.x)
    dst[i] = out_off[row0[i]];
}

unsigned grid_for(uint64_t n) {
  uint64_t b = (n + 255) / 256;
  return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(b, 256 * 64));
}

// ---- host side ----------------------------------------------------------------

struct Tuning {
  uint32_t light_max = 128;   // products above which a matrix row is heavy (light hash: 2x slots)
  uint32_t blocks_per_cu = 2; // persistent grid
  uint32_t inner_ratio = 16;  // heavy row in inner-product form when products * ratio >= nnz(E)
};

// E transposed (levels k, j) of every matrix instance, built once per batch
// and shared by the autotuner's candidate setups; keyed by E's trie and
// annotation column.
struct Transposes {
  std::map<std::pair<const lh_trie*, int32_t>, lh_trie*> by_e;
  ~Transposes() {
    for (auto& kv : by_e) free_trie(kv.second);
  }
};
constexpr uint32_t MAX_BLOCKS_PER_CU = 4;

// Everything one batch needs; kept across calls with the same plans so the
// graph is replayed rather than rebuilt.
struct BatchState {
  std::vector<const lh_plan_t*> plans;
  Tuning tune;
  uint64_t R = 0, UB = 0;
  hipStream_t s = nullptr;
  DBuf<BInst> inst;
  DBuf<uint64_t> inst_row0, prod, ub_off;
  DBuf<uint64_t> upd;          // updates per row, where they are not its products (some E repeats key pairs)
  const uint64_t* updates() const { return upd.p ? upd.p : prod.p; }
  std::vector<uint64_t> h_nj;   // join tuples per instance (fixed by the plans)
  DBuf<uint32_t> row_inst, ub, heavy_f, light_f, inner_f, heavy, light, inner, qhead, row_nnz, ub_k, err;
  std::shared_ptr<Transposes> tr;
  DBuf<uint64_t> ub_cnt;
  DBuf<double> ub_sum;
  uint32_t kw = 64;
  uint64_t n_heavy = 0, n_light = 0, n_inner = 0;
  bool has_vec = false;        // some instance is a matrix-vector product
  DBuf<uint32_t> longs;        // its long rows, listed by k_batch_vec
  std::vector<uint64_t> h_inst_row0;
  std::vector<BInst> h_inst;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  hipStream_t cap = nullptr;
  ~BatchState() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (cap) (void)hipStreamDestroy(cap);
  }
};

std::mutex g_batch_mu;
std::unique_ptr<BatchState> g_batch;

BInst describe(const lh_plan_t* p) {
  const PlanAtom& A = p->atoms[0];
  const PlanAtom& E = p->atoms[1];
  const lh_trie* ta = A.trie;
  const lh_trie* te = E.trie;
  BInst b{};
  b.kind = E.n_levels == 1 ? 0u : 1u;
  b.n_rows = (uint32_t)ta->lv[0].n;
  b.a_i = ta->lv[0].keys.p;
  b.a_off = ta->lv[0].offs.p;
  b.a_j = ta->lv[1].keys.p;
  b.a_run = run_offsets(ta);
  b.sum = p->agg == LH_AGG_SUM ? 1u : 0u;
  b.a_val = (b.sum && A.anno >= 0) ? ta->annos[A.anno].p : nullptr;
  b.e_j = te->lv[0].keys.p;
  b.e_n0 = (uint32_t)te->lv[0].n;
  // distinct sorted keys, as many as the largest key + 1: exactly 0 .. n - 1
  b.e_dense = (b.e_n0 > 0 && (uint64_t)te->key_max[0] + 1 == te->lv[0].n) ? 1u : 0u;
  b.e_pool = te->lv[0].pool.p;
  b.e_bsw = UINT64_MAX;
  b.e_bsb = 0;
  b.e_bsw_of = te->lv[0].bs_word.p;
  b.e_bsb_of = te->lv[0].bs_base.p;
  if (b.kind == 1) {
    b.e_off = te->lv[0].offs.p;
    b.e_k = te->lv[1].keys.p;
    b.n_k = te->key_max[1] + 1;
  }
  b.e_run = run_offsets(te);
  b.nnz_e = E.n_levels == 2 ? te->lv[1].n : 0;
  b.e_val = (b.sum && E.anno >= 0) ? te->annos[E.anno].p : nullptr;
  b.lsb = p->exact_lsb;
  b.D = p->exact_digits;
  b.n_j = ta->key_max[1] + 1;
  return b;
}

// E transposed: the same rows keyed (k, j), bag semantics, sorted arrays.
lh_trie* transpose_e(const lh_trie* te, int32_t anno, hipStream_t s) {
  const uint32_t* keys[2] = {row_keys(te, 0), row_keys(te, 1)};
  const double* annos[1] = {anno >= 0 ? te->annos[anno].p : nullptr};
  const uint32_t level_order[2] = {1, 0};
  return build_trie(te->n_rows, 2, keys, anno >= 0 ? 1u : 0u, annos, 0, nullptr, level_order,
                    LH_BAG | LH_LAYOUT_UINT, nullptr, 0, s);
}

void attach_transpose(BInst& b, const lh_plan_t* p, Transposes& tr, hipStream_t s) {
  const PlanAtom& E = p->atoms[1];
  const int32_t anno = b.sum ? E.anno : -1;
  auto key = std::make_pair(E.trie, anno);
  auto it = tr.by_e.find(key);
  if (it == tr.by_e.end()) it = tr.by_e.emplace(key, transpose_e(E.trie, anno, s)).first;
  const lh_trie* t = it->second;
  b.bt_n0 = (uint32_t)t->lv[0].n;
  b.bt_k = t->lv[0].keys.p;
  b.bt_off = t->lv[0].offs.p;
  b.bt_j = t->lv[1].keys.p;
  b.bt_run = run_offsets(t);
  b.bt_val = anno >= 0 ? t->annos[0].p : nullptr;
}

std::string cache_path() {
  const char* e = std::getenv("LH_AUTOTUNE_CACHE");
  if (e && *e) return e;
  const char* h = std::getenv("HOME");
  return std::string(h ? h : "/tmp") + "/.cache/lh_autotune.txt";
}

// "<arch>_cu<CUs>" of the current device (its properties are asked for once).
std::string device_name() {
  static std::mutex mu;
  static std::map<int, std::string> names;
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::lock_guard<std::mutex> lk(mu);
  auto it = names.find(dev);
  if (it == names.end()) {
    hipDeviceProp_t prop;
    (void)hipGetDeviceProperties(&prop, dev);
    it = names.emplace(dev, std::string(prop.gcnArchName) + "_cu" + std::to_string(prop.multiProcessorCount)).first;
  }
  return it->second;
}

std::string signature(const BatchState& b) {
  std::ostringstream os;
  uint64_t rows_log = 0, ub_log = 0;
  while ((1ull << rows_log) < b.R) rows_log++;
  while ((1ull << ub_log) < b.UB) ub_log++;
  os << "v5_" << device_name() << "_inst" << b.plans.size() << "_r" << rows_log
     << "_u" << ub_log;
  return os.str();
}

bool load_tuning(const std::string& sig, Tuning& t) {
  std::ifstream f(cache_path());
  std::string key;
  Tuning x;
  while (f >> key >> x.light_max >> x.blocks_per_cu >> x.inner_ratio) {
    if (key == sig) {
      t = x;
      return true;
    }
  }
  return false;
}

void save_tuning(const std::string& sig, const Tuning& t) {
  std::string path = cache_path();
  std::error_code ec;  // an unwritable cache only costs the next run a re-tune
  std::filesystem::create_directories(std::filesystem::path(path).parent_path(), ec);
  std::ofstream f(path, std::ios::app);
  f << sig << " " << t.light_max << " " << t.blocks_per_cu << " " << t.inner_ratio << "\n";
}

// What the plans alone decide: instances, rows, products, output bounds.
void setup_rows(BatchState& b, hipStream_t s) {
  const uint32_t n = (uint32_t)b.plans.size();
  b.s = s;
  b.h_inst.resize(n);
  b.h_inst_row0.assign(n + 1, 0);
  b.tr = std::make_shared<Transposes>();
  for (uint32_t i = 0; i < n; i++) {
    b.h_inst[i] = describe(b.plans[i]);
    b.h_inst[i].row_base = b.h_inst_row0[i];
    b.h_inst_row0[i + 1] = b.h_inst_row0[i] + b.h_inst[i].n_rows;
  }
  b.R = b.h_inst_row0[n];
  if (b.R >= (1ull << 32)) fail(LH_ERR_OVERFLOW, "batch: more than 2^32 rows");
  b.inst.alloc(n, s);
  LH_HIP(hipMemcpyAsync(b.inst.p, b.h_inst.data(), n * sizeof(BInst), hipMemcpyHostToDevice, s));
  b.inst_row0.alloc(n + 1, s);
  LH_HIP(hipMemcpyAsync(b.inst_row0.p, b.h_inst_row0.data(), (n + 1) * sizeof(uint64_t), hipMemcpyHostToDevice, s));
  k_inst_roots<<<1, 256, 0, s>>>(b.inst.p, n);
  LH_HIP(hipGetLastError());
  b.row_inst.alloc(b.R, s);
  b.prod.alloc(b.R, s);
  b.ub.alloc(b.R, s);
  bool repeats = false;
  for (const BInst& I : b.h_inst) repeats = repeats || (I.kind == 1 && I.e_run);
  b.upd.alloc(repeats ? b.R : 0, s);
  if (b.R) {
    k_row_products<<<(unsigned)std::min<uint64_t>((b.R + B_NT - 1) / B_NT, 1u << 16), B_NT, 0, s>>>(
        b.inst.p, b.inst_row0.p, n, b.R, b.row_inst.p, b.prod.p, b.upd.p, b.ub.p);
    LH_HIP(hipGetLastError());
  }
  b.ub_off.alloc(b.R + 1, s);
  b.h_nj.assign(n, 0);
  DBuf<uint64_t> dnj(n, s);
  if (n) {
    k_inst_sums<<<n, B_NT, 0, s>>>(b.prod.p, b.inst_row0.p, dnj.p);
    LH_HIP(hipGetLastError());
    LH_HIP(hipMemcpyAsync(b.h_nj.data(), dnj.p, n * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
  }
  b.UB = scan_u32_to_u64(b.ub.p, b.ub_off.p, b.R, s);
  b.heavy_f.alloc(b.R, s);
  b.light_f.alloc(b.R, s);
  b.inner_f.alloc(b.R, s);
  b.heavy.alloc(b.R, s);
  b.light.alloc(b.R, s);
  b.inner.alloc(b.R, s);
  b.qhead.alloc(4, s);
  b.has_vec = false;
  for (const BInst& I : b.h_inst) b.has_vec = b.has_vec || I.kind == 0;
  b.longs.alloc(b.has_vec ? b.R : 0, s);
  b.row_nnz.alloc(b.R, s);
  b.ub_k.alloc(b.UB, s);
  b.ub_cnt.alloc(b.UB, s);
  b.ub_sum.alloc(b.UB, s);
  b.err.alloc(1, s);
  // heavy rows: the window of k values their bitmap covers
  uint32_t nk = 0;
  for (const BInst& I : b.h_inst)
    if (I.kind == 1) nk = std::max(nk, I.n_k);
  b.kw = std::max<uint32_t>(64, std::min<uint32_t>(KW_MAX, (nk + 63) / 64 * 64));
}

// What the tuning decides as well: row classes, their queues, and E
// transposed for the instances that have inner-product rows.
void setup_classes(BatchState& b, hipStream_t s) {
  const uint32_t n = (uint32_t)b.plans.size();
  b.n_heavy = b.n_light = b.n_inner = 0;
  if (!b.R) return;
  DBuf<uint32_t> has_inner(n, s);
  fill_u32(has_inner.p, 0, n, s);
  k_row_classes<<<grid_for(b.R), 256, 0, s>>>(b.inst.p, b.row_inst.p, b.updates(), b.R, b.tune.light_max,
                                              b.tune.inner_ratio, b.heavy_f.p, b.light_f.p, b.inner_f.p, has_inner.p);
  LH_HIP(hipGetLastError());
  std::vector<uint32_t> h(n);
  LH_HIP(hipMemcpyAsync(h.data(), has_inner.p, n * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  b.n_heavy = select_flagged(b.heavy_f.p, b.R, b.heavy.p, s);
  b.n_light = select_flagged(b.light_f.p, b.R, b.light.p, s);
  b.n_inner = select_flagged(b.inner_f.p, b.R, b.inner.p, s);   // in row order: grouped by instance
  if (b.n_inner) {
    bool added = false;
    for (uint32_t i = 0; i < n; i++)
      if (h[i] && !b.h_inst[i].bt_k) {
        attach_transpose(b.h_inst[i], b.plans[i], *b.tr, s);
        added = true;
      }
    if (added) {
      LH_HIP(hipMemcpyAsync(b.inst.p, b.h_inst.data(), n * sizeof(BInst), hipMemcpyHostToDevice, s));
      k_inst_roots<<<1, 256, 0, s>>>(b.inst.p, n);
      LH_HIP(hipGetLastError());
    }
  }
  if (b.n_heavy > 1) {
    // heavy rows longest first (LPT)
    DBuf<uint64_t> k0(b.n_heavy, s), k1(b.n_heavy, s);
    DBuf<uint32_t> other(b.n_heavy, s);
    k_heavy_keys<<<grid_for(b.n_heavy), 256, 0, s>>>(b.heavy.p, b.n_heavy, b.updates(), k0.p);
    LH_HIP(hipGetLastError());
    uint64_t* const kb[2] = {k0.p, k1.p};
    uint32_t* const vb[2] = {b.heavy.p, other.p};
    if (radix_sort_between(kb, vb, b.n_heavy, HEAVY_KEY_BITS, s))
      LH_HIP(hipMemcpyAsync(b.heavy.p, other.p, b.n_heavy * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
  }
  LH_HIP(hipStreamSynchronize(s));  // the host's arrays were read
}

void launch_compute(BatchState& b, hipStream_t s) {
  int dev = 0, cus = 256;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  k_fill_u32_dev<<<1, 64, 0, s>>>(b.qhead.p, 0u, 4);
  k_fill_u32_dev<<<1, 64, 0, s>>>(b.err.p, 0u, 1);
  BatchArgs a{};
  a.inst = b.inst.p;
  a.row_inst = b.row_inst.p;
  a.inst_row0 = b.inst_row0.p;
  a.ub_off = b.ub_off.p;
  a.heavy = b.heavy.p;
  a.n_heavy = b.n_heavy;
  a.light = b.light.p;
  a.n_light = b.n_light;
  a.inner = b.inner.p;
  a.n_inner = b.n_inner;
  a.qhead = b.qhead.p;
  a.row_nnz = b.row_nnz.p;
  a.ub_k = b.ub_k.p;
  a.ub_cnt = b.ub_cnt.p;
  a.ub_sum = b.ub_sum.p;
  a.err = b.err.p;
  a.prod = b.prod.p;
  a.kw = b.kw;
  const unsigned grid = (unsigned)(cus * std::min(b.tune.blocks_per_cu, MAX_BLOCKS_PER_CU));
  if (b.n_inner) k_batch_inner<<<grid, I_NT, 0, s>>>(a);
  if (b.n_heavy) k_batch_heavy<<<grid, B_NT, 0, s>>>(a);
  if (b.has_vec && b.R) {
    k_batch_vec<<<(unsigned)std::min<uint64_t>((b.R * 8 + B_NT - 1) / B_NT, 1u << 16), B_NT, 0, s>>>(a, b.R, b.longs.p);
    k_batch_vec_long<<<(unsigned)(4 * cus), B_NT, 0, s>>>(a, b.longs.p);
  }
  if (!b.n_light) return;
  if (b.tune.light_max <= 64) k_batch_light<128><<<grid, B_NT, 0, s>>>(a);
  else k_batch_light<256><<<grid, B_NT, 0, s>>>(a);
}

void build_graph(BatchState& b) {
  if (b.exec) (void)hipGraphExecDestroy(b.exec);
  if (b.graph) (void)hipGraphDestroy(b.graph);
  b.exec = nullptr;
  b.graph = nullptr;
  if (!b.cap) LH_HIP(hipStreamCreateWithFlags(&b.cap, hipStreamNonBlocking));
  LH_HIP(hipStreamBeginCapture(b.cap, hipStreamCaptureModeThreadLocal));
  launch_compute(b, b.cap);
  hipError_t e = hipStreamEndCapture(b.cap, &b.graph);
  if (e != hipSuccess) hip_fail(e, "hipStreamEndCapture", __FILE__, __LINE__);
  LH_HIP(hipGraphInstantiate(&b.exec, b.graph, nullptr, nullptr, 0));
}

float time_replay(BatchState& b, hipStream_t s) {
  hipEvent_t e0, e1;
  LH_HIP(hipEventCreate(&e0));
  LH_HIP(hipEventCreate(&e1));
  LH_HIP(hipEventRecord(e0, s));
  LH_HIP(hipGraphLaunch(b.exec, s));
  LH_HIP(hipEventRecord(e1, s));
  LH_HIP(hipEventSynchronize(e1));
  float ms = 0;
  LH_HIP(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return ms;
}

// The project's autotuner: time each candidate's graph, keep the fastest,
// remember it per device and batch signature.  The light/heavy split and
// the inner-product ratio change the row classes and queues; the grid only
// changes the captured launch, so it is tried on each of them.
void autotune(BatchState& b, hipStream_t s) {
  const std::string sig = signature(b);
  if (load_tuning(sig, b.tune)) {
    setup_classes(b, s);
    return;
  }
  float best = 3.0e38f;
  Tuning win = b.tune;
  for (uint32_t lm : {64u, 128u})
    for (uint32_t ir : {4u, 16u, 64u}) {
      b.tune.light_max = lm;
      b.tune.inner_ratio = ir;
      setup_classes(b, s);
      for (uint32_t bp : {1u, 2u, 4u}) {
        b.tune.blocks_per_cu = bp;
        build_graph(b);
        const float ms = time_replay(b, s);
        if (ms < best) {
          best = ms;
          win = b.tune;
        }
      }
    }
  b.tune = win;
  setup_classes(b, s);
  build_graph(b);
  save_tuning(sig, win);
}

struct SharedOut {
  DBuf<uint32_t> out_i, out_k;
  DBuf<uint64_t> out_cnt;
  DBuf<double> out_sum;
};

}  // namespace

int row_union_kind(const lh_plan_t* p) {
  if (p->atoms.size() != 2 || !p->groups.empty()) return -1;
  const PlanAtom& A = p->atoms[0];
  const PlanAtom& E = p->atoms[1];
  if (A.n_levels != 2) return -1;
  // attribute roles: i = A's first level, j = A's second level
  const uint32_t i = A.attr_of_level[0], j = A.attr_of_level[1];
  if (p->order[0] != i || p->order[1] != j) return -1;
  if (E.n_levels == 1) {
    if (p->n_attrs != 2 || E.attr_of_level[0] != j) return -1;
    if (p->out_attrs.size() != 1 || p->out_attrs[0] != i) return -1;
    return 0;
  }
  if (E.n_levels == 2) {
    if (p->n_attrs != 3 || E.attr_of_level[0] != j) return -1;
    const uint32_t k = E.attr_of_level[1];
    if (p->order[2] != k) return -1;
    if (p->out_attrs.size() != 2 || p->out_attrs[0] != i || p->out_attrs[1] != k) return -1;
    return 1;
  }
  return -1;
}

bool run_batch(lh_plan_t* const* plans, uint32_t n, hipStream_t s, std::vector<lh_result_impl*>& out) {
  for (uint32_t i = 0; i < n; i++)
    if (row_union_kind(plans[i]) < 0) return false;
  std::lock_guard<std::mutex> lk(g_batch_mu);
  std::vector<const lh_plan_t*> pv(plans, plans + n);
  if (!g_batch || g_batch->plans != pv) {
    g_batch.reset();
    auto b = std::make_unique<BatchState>();
    b->plans = pv;
    setup_rows(*b, s);
    autotune(*b, s);
    g_batch = std::move(b);
  } else if (!g_batch->exec) {
    build_graph(*g_batch);  // plans that come again are replayed
  }
  BatchState& b = *g_batch;
  {
    ProfScope ps("batch_graph", s, b.R, b.UB);
    if (b.exec) LH_HIP(hipGraphLaunch(b.exec, s));
    else launch_compute(b, s);
    LH_HIP(hipGetLastError());
  }
  // pack: scan the per-row output counts, one shared output block
  DBuf<uint64_t> out_off(b.R + 1, s);
  const uint64_t total = scan_u32_to_u64(b.row_nnz.p, out_off.p, b.R, s);
  if (read_scalar(b.err.p, s)) fail(LH_ERR_UNSUPPORTED, "an annotation product did not fit the exact accumulator");
  auto sh = std::make_shared<SharedOut>();
  sh->out_i.alloc(total, s);
  sh->out_k.alloc(total, s);
  sh->out_cnt.alloc(total, s);
  sh->out_sum.alloc(total, s);
  PackArgs2 pa{};
  pa.inst = b.inst.p;
  pa.row_inst = b.row_inst.p;
  pa.inst_row0 = b.inst_row0.p;
  pa.ub_off = b.ub_off.p;
  pa.out_off = out_off.p;
  pa.ub_k = b.ub_k.p;
  pa.ub_cnt = b.ub_cnt.p;
  pa.ub_sum = b.ub_sum.p;
  pa.out_i = sh->out_i.p;
  pa.out_k = sh->out_k.p;
  pa.out_cnt = sh->out_cnt.p;
  pa.out_sum = sh->out_sum.p;
  pa.R = b.R;
  if (total) {
    ProfScope ps("batch_pack", s, b.R, total);
    const uint64_t per = (uint64_t)PACK_SPAN * B_NW;
    if (total / per >= (1ull << 31)) fail(LH_ERR_OVERFLOW, "batch: too many output rows");
    k_pack_rows<<<(unsigned)((total + per - 1) / per), B_NT, 0, s>>>(pa, total);
    LH_HIP(hipGetLastError());
  }
  // each instance's rows are contiguous: its outputs are [offs[i], offs[i + 1])
  std::vector<uint64_t> offs(n + 1);
  {
    DBuf<uint64_t> d(n + 1, s);
    k_inst_offsets<<<(n + 256) / 256, 256, 0, s>>>(out_off.p, b.inst_row0.p, n, d.p);
    LH_HIP(hipGetLastError());
    LH_HIP(hipMemcpyAsync(offs.data(), d.p, (n + 1) * sizeof(uint64_t), hipMemcpyDeviceToHost, s));
    LH_HIP(hipStreamSynchronize(s));
  }
  for (uint32_t i = 0; i < n; i++) {
    const BInst& I = b.h_inst[i];
    const uint64_t o0 = offs[i], o1 = offs[i + 1];
    auto* r = new lh_result_impl();
    memset(&r->pub, 0, sizeof(r->pub));
    r->shared = sh;
    r->colptr.push_back(sh->out_i.p ? sh->out_i.p + o0 : nullptr);
    if (I.kind == 1) r->colptr.push_back(sh->out_k.p ? sh->out_k.p + o0 : nullptr);
    r->pub.n_rows = o1 - o0;
    r->pub.n_cols = (uint32_t)r->colptr.size();
    r->pub.out_keys = r->colptr.data();
    r->pub.counts = sh->out_cnt.p ? sh->out_cnt.p + o0 : nullptr;
    r->pub.sums = I.sum ? (sh->out_sum.p ? sh->out_sum.p + o0 : nullptr) : nullptr;
    r->pub.exact = I.sum;
    r->pub.n_join_tuples = b.h_nj[i];
    out.push_back(r);
  }
  return true;
}

void batch_forget_plan(const lh_plan_t* p) {
  std::lock_guard<std::mutex> lk(g_batch_mu);
  if (g_batch && std::find(g_batch->plans.begin(), g_batch->plans.end(), p) != g_batch->plans.end()) g_batch.reset();
}

}  // namespace lh
