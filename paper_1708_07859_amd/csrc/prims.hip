// Device-wide primitives: scans, reductions, fills, gathers, LSD radix sort.
#include <algorithm>
#include <climits>
#include <cstring>
#include <type_traits>

#include "device_common.h"
#include "lh_internal.h"

namespace lh {

namespace {

constexpr int SC_NT = 256;
constexpr int SC_ITEMS = 8;
constexpr int SC_TILE = SC_NT * SC_ITEMS;

// Device-wide exclusive scans.  Launches and host round trips bound the
// short ones (a launch costs 2 to 3 us of a dependent chain, a read-back of
// a device scalar 15 us), so a scan is one kernel up to SC_ONE elements, two
// up to SC_SELF tiles (each block sums the tiles before its own), three and
// more beyond (the tile sums are scanned first), with no clears, and the
// total goes to the host by a store into pinned memory from the kernel that
// knows it.  With up to seven kernels, two clears and a copy per scan, as
// before, a noalloc SpGEMM of 30,000 products took 684 us (now 330), a
// triangle COUNT of 11,000 edges 863 us (585), 128 set pairs 534 us (352).
constexpr int SO_NT = 1024;                     // the one-block scan
constexpr int SO_ITEMS = 8;
constexpr uint64_t SC_ONE = 2ull * SO_NT * SO_ITEMS;
constexpr uint64_t SC_SELF = 1024;              // tiles: at most four sums per thread of a tile

// Per-tile sums of the input.
template <class TI, class TO>
__global__ __launch_bounds__(SC_NT) void k_tile_sums(const TI* in, uint64_t n, TO* sums) {
  __shared__ TO lds[SC_NT / WAVE];
  uint64_t base = (uint64_t)blockIdx.x * SC_TILE;
  TO s = 0;
#pragma unroll
  for (int i = 0; i < SC_ITEMS; i++) {
    uint64_t idx = base + (uint64_t)i * SC_NT + threadIdx.x;
    if (idx < n) s += (TO)in[idx];
  }
  TO tot = block_sum<TO, SC_NT>(s, lds);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Exclusive scan of in[0, n) by one block, the total in out[n] and, when
// asked, in *host (pinned).  Thread t owns SO_ITEMS consecutive elements of
// each round.
template <class TI, class TO>
__global__ __launch_bounds__(SO_NT) void k_scan_one(const TI* in, uint64_t n, TO* out, TO* host) {
  __shared__ TO lds[SO_NT / WAVE];
  TO carry = 0;
  for (uint64_t r0 = 0; r0 < n; r0 += (uint64_t)SO_NT * SO_ITEMS) {
    const uint64_t i0 = r0 + (uint64_t)threadIdx.x * SO_ITEMS;
    TO v[SO_ITEMS], s = 0;
#pragma unroll
    for (int i = 0; i < SO_ITEMS; i++) {
      v[i] = i0 + i < n ? (TO)in[i0 + i] : (TO)0;
      s += v[i];
    }
    TO tot;
    TO run = block_excl_scan<TO, SO_NT>(s, lds, tot) + carry;
#pragma unroll
    for (int i = 0; i < SO_ITEMS; i++) {
      if (i0 + i < n) out[i0 + i] = run;
      run += v[i];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) {
    out[n] = carry;
    if (host) *host = carry;
  }
}

// Exclusive scan of each tile plus its tile offset; thread t owns
// SC_ITEMS consecutive elements.  SELF: `tile_off` holds the tiles' sums and
// every block adds up those before its own (at most SC_SELF of them).  The
// last block stores the total in out[n] and, when asked, in *host (pinned).
template <class TI, class TO, bool SELF>
__global__ __launch_bounds__(SC_NT) void k_tile_scan(const TI* in, uint64_t n, const TO* tile_off, TO* out, TO* host) {
  __shared__ TO lds[SC_NT / WAVE];
  __shared__ TI stage[SC_TILE];
  uint64_t base = (uint64_t)blockIdx.x * SC_TILE;
  // coalesced load into LDS
#pragma unroll
  for (int i = 0; i < SC_ITEMS; i++) {
    uint64_t idx = base + (uint64_t)i * SC_NT + threadIdx.x;
    stage[i * SC_NT + threadIdx.x] = idx < n ? in[idx] : (TI)0;
  }
  TO off;
  if constexpr (SELF) {
    TO p = 0;
    for (uint32_t t = threadIdx.x; t < blockIdx.x; t += SC_NT) p += tile_off[t];
    off = block_sum<TO, SC_NT>(p, lds);  // ends with a barrier
  } else {
    off = tile_off[blockIdx.x];
    __syncthreads();
  }
  TO v[SC_ITEMS];
  TO s = 0;
#pragma unroll
  for (int i = 0; i < SC_ITEMS; i++) {
    v[i] = (TO)stage[threadIdx.x * SC_ITEMS + i];
    s += v[i];
  }
  TO tot;
  TO run = block_excl_scan<TO, SC_NT>(s, lds, tot) + off;
  if (blockIdx.x + 1 == gridDim.x && threadIdx.x == 0) {
    out[n] = off + tot;
    if (host) *host = off + tot;
  }
  __syncthreads();
  // write back through LDS as TO (reuse needs a separate buffer for 64-bit)
  __shared__ TO ostage[SC_TILE];
#pragma unroll
  for (int i = 0; i < SC_ITEMS; i++) {
    ostage[threadIdx.x * SC_ITEMS + i] = run;
    run += v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < SC_ITEMS; i++) {
    uint64_t idx = base + (uint64_t)i * SC_NT + threadIdx.x;
    if (idx < n) out[idx] = ostage[i * SC_NT + threadIdx.x];
  }
}

// Exclusive scan of in[0, n) into out[0, n) and the total into out[n] and,
// when asked, into *host (pinned); nothing waits here.
template <class TI, class TO>
void scan_dev(const TI* in, TO* out, uint64_t n, hipStream_t s, TO* host = nullptr) {
  if (n <= SC_ONE) {
    k_scan_one<TI, TO><<<1, SO_NT, 0, s>>>(in, n, out, host);
    LH_HIP(hipGetLastError());
    return;
  }
  const uint64_t ntiles = (n + SC_TILE - 1) / SC_TILE;
  DBuf<TO> sums(ntiles, s);
  k_tile_sums<TI, TO><<<(unsigned)ntiles, SC_NT, 0, s>>>(in, n, sums.p);
  LH_HIP(hipGetLastError());
  if (ntiles <= SC_SELF) {
    k_tile_scan<TI, TO, true><<<(unsigned)ntiles, SC_NT, 0, s>>>(in, n, sums.p, out, host);
  } else {
    DBuf<TO> offs(ntiles + 1, s);
    scan_dev<TO, TO>(sums.p, offs.p, ntiles, s);
    k_tile_scan<TI, TO, false><<<(unsigned)ntiles, SC_NT, 0, s>>>(in, n, offs.p, out, host);
  }
  LH_HIP(hipGetLastError());
}

// The same, and the total read back to the host.
template <class TI, class TO>
TO scan_impl(const TI* in, TO* out, uint64_t n, hipStream_t s) {
  TO* host = static_cast<TO*>(pinned_scratch_or_null());
  scan_dev<TI, TO>(in, out, n, s, host);
  if (!host) return read_scalar(out + n, s);
  LH_HIP(hipStreamSynchronize(s));
  return *static_cast<volatile TO*>(host);
}

// Largest of in[0, n).  The body is read as 16-byte vectors, four rounds
// in flight per thread; the elements before the first 16-byte boundary and
// after the last whole vector are read singly.
__global__ __launch_bounds__(256) void k_reduce_max_u32(const uint32_t* in, uint64_t n, uint32_t* out) {
  __shared__ uint32_t s_m[256 / WAVE];
  const uint64_t head = min<uint64_t>(n, (4u - (((uintptr_t)in >> 2) & 3u)) & 3u);
  const uint4* body = reinterpret_cast<const uint4*>(in + head);
  const uint64_t nv = (n - head) / 4, tail = head + nv * 4;
  const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
  uint32_t m = 0;
  if (gid < head) m = in[gid];
  if (gid < n - tail) m = max(m, in[tail + gid]);
  uint64_t i = gid;
  for (; i + 3 * stride < nv; i += 4 * stride) {
    const uint4 a = body[i], b = body[i + stride], c = body[i + 2 * stride], d = body[i + 3 * stride];
    m = max(m, max(max(max(a.x, a.y), max(a.z, a.w)), max(max(b.x, b.y), max(b.z, b.w))));
    m = max(m, max(max(max(c.x, c.y), max(c.z, c.w)), max(max(d.x, d.y), max(d.z, d.w))));
  }
  for (; i < nv; i += stride) {
    const uint4 a = body[i];
    m = max(m, max(max(a.x, a.y), max(a.z, a.w)));
  }
#pragma unroll
  for (int d = WAVE / 2; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d, WAVE));
  if (lane_id() == 0) s_m[threadIdx.x / WAVE] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t b = 0;
    for (int w = 0; w < 256 / WAVE; w++) b = max(b, s_m[w]);
    atomicMax(out, b);
  }
}

struct MaxCols {
  const uint32_t* col[MAX_COLS];
  uint64_t n[MAX_COLS];
};

// Row y of the grid: the largest of column y, into out[y] (cleared before).
__global__ __launch_bounds__(256) void k_max_cols(MaxCols a, uint32_t* out) {
  __shared__ uint32_t s_m[256 / WAVE];
  const uint32_t* col = a.col[blockIdx.y];
  const uint64_t n = a.n[blockIdx.y];
  uint32_t m = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) m = max(m, col[i]);
#pragma unroll
  for (int d = WAVE / 2; d > 0; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d, WAVE));
  if (lane_id() == 0) s_m[threadIdx.x / WAVE] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t b = 0;
    for (int w = 0; w < 256 / WAVE; w++) b = max(b, s_m[w]);
    if (b) atomicMax(&out[blockIdx.y], b);
  }
}

__global__ void k_iota(uint32_t* out, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    out[i] = (uint32_t)i;
}

template <class T>
__global__ void k_fill(T* out, T v, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    out[i] = v;
}

template <class T>
__global__ void k_gather(const T* src, const uint32_t* idx, T* dst, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    dst[i] = src[idx[i]];
}

__global__ void k_scatter_flagged(const uint32_t* flags, const uint64_t* off, uint64_t n, uint32_t* out) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    if (flags[i]) out[off[i]] = (uint32_t)i;
}

unsigned grid_for(uint64_t n) {
  uint64_t b = (n + 255) / 256;
  return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(b, 256 * 64));
}

// ---------------------------------------------------------------------------
// LSD radix sort, 8-bit digits, one kernel per pass.  Memory bounds a pass:
// every key is read once and written once, in runs of equal digits.  One
// kernel first counts the digits of all passes in a single read of the
// input; a pass then needs, for its tile's first slot of each digit, only
// the counts of the tiles before it, which it adds up from what they publish
// (decoupled look-back) while its own keys are ranked.  A sort of key
// columns reads the columns in its first pass (packing each row's key on the
// fly) and writes the sorted columns in its last (unpacking them).  Keys of
// 65 to 96 bits are two words; a value (the row permutation, or the one
// column that must follow) travels along.  Sorts of one tile run all passes
// in one launch, in LDS.
// Tiles of 4096 keys by 512 threads: runs of 16 keys (128 bytes) per digit
// on average, and 33 KB of LDS leaves four tiles (32 waves) on a CU; tiles
// of 8192 keys measured the same on 64 M keys and 30% slower on 1 M.
// 64 M 44-bit keys, six passes: 0.36 ms of counting and 0.37 ms per pass
// (2.8 TB/s), 2.56 ms in all; a count, a scan of seven kernels and a scatter
// per pass took 3.7 ms.  A whole trie build of 20 M rows of 66
// bits with an annotation: 5.2 ms, 7.4 ms when the row permutation was
// sorted by two packed words and the columns gathered through it.
// ---------------------------------------------------------------------------
constexpr int RS_NT = 512;
constexpr int RS_ITEMS = 8;
constexpr int RS_TILE = RS_NT * RS_ITEMS;
constexpr int RS_NW = RS_NT / WAVE;
constexpr int RS_MAXP = 12;    // passes: 96 bits
constexpr int RH_COPIES = 2;   // histogram copies per block (lanes spread over them)
constexpr uint32_t RS_GROUP = 32;  // tiles per group of the look-back
constexpr int RS_LOOK = 8;     // tiles looked back at per round
constexpr int RS_GLOOK = 4;    // groups looked back at per round

// Key columns packed into one key: column c at bit shift[c] of 64, or of 96
// (wide: the low 32 bits in a word of their own).
struct PackArgs {
  const uint32_t* col[LH_MAX_KEYS];
  uint32_t shift[LH_MAX_KEYS];
  uint32_t ncols;
};

// One key unpacked into key columns: bits[c] bits at shift[c].
struct UnpackCols {
  uint32_t* col[LH_MAX_KEYS];
  uint32_t shift[LH_MAX_KEYS];
  uint32_t bits[LH_MAX_KEYS];
  uint32_t ncols;
};

template <bool WIDE>
__device__ __forceinline__ uint64_t pack_row(const PackArgs& a, uint64_t r, uint32_t& x) {
  uint64_t k = 0;
  x = 0;
#pragma unroll
  for (uint32_t c = 0; c < LH_MAX_KEYS; c++)
    if (c < a.ncols) {
      const uint64_t v = a.col[c][r];
      const uint32_t sh = a.shift[c];
      if constexpr (!WIDE) {
        k |= v << sh;
      } else if (sh >= 32) {
        k |= v << (sh - 32);
      } else {
        x |= (uint32_t)(v << sh);
        k |= v >> (32 - sh);
      }
    }
  return k;
}

template <bool WIDE>
__device__ __forceinline__ void unpack_row(const UnpackCols& a, uint64_t r, uint64_t k, uint32_t x) {
#pragma unroll
  for (uint32_t c = 0; c < LH_MAX_KEYS; c++)
    if (c < a.ncols) {
      const uint32_t sh = a.shift[c];
      uint64_t v;
      if constexpr (!WIDE) v = k >> sh;
      else v = sh >= 32 ? k >> (sh - 32) : (((uint64_t)(uint32_t)k << 32) | x) >> sh;
      // (a column of no bits has shift up to the key's width: its value is 0)
      a.col[c][r] = a.bits[c] ? (uint32_t)(v & ((1ull << a.bits[c]) - 1)) : 0u;
    }
}

// Eight bits of a key at a wave-uniform shift: one funnel shift of the two
// words that can hold them (a 64-bit shift by a register is several times
// dearer, and a pass takes each element's digit three times).
template <bool WIDE>
__device__ __forceinline__ uint32_t digit_at(uint64_t k, uint32_t x, uint32_t shift) {
  const uint32_t k0 = (uint32_t)k, k1 = (uint32_t)(k >> 32);
  uint32_t lo, hi;
  if constexpr (WIDE) {
    lo = shift < 32 ? x : shift < 64 ? k0 : k1;
    hi = shift < 32 ? k0 : shift < 64 ? k1 : 0u;
  } else {
    lo = shift < 32 ? k0 : k1;
    hi = shift < 32 ? k1 : 0u;
  }
  return __builtin_amdgcn_alignbit(hi, lo, shift & 31u) & 255u;
}

// Digit counts of every pass, in one read of the keys: hist[p * 256 + d],
// cleared before.  Lanes spread over copies of the LDS counters, and a wave
// whose lanes all hold one digit (hub vertices, high digits) adds once.
template <bool FROM_COLS, bool WIDE>
__global__ __launch_bounds__(RS_NT) void k_rs_hist(const uint64_t* keys, const uint32_t* xkeys, PackArgs pa, uint64_t n,
                                                   uint32_t lo_bit, uint32_t passes, uint32_t* hist) {
  __shared__ uint32_t h[RS_MAXP * 256 * RH_COPIES];
  const uint32_t nh = passes * 256 * RH_COPIES;
  for (uint32_t i = threadIdx.x; i < nh; i += RS_NT) h[i] = 0;
  __syncthreads();
  const uint32_t copy = lane_id() & (RH_COPIES - 1);
  const uint64_t stride = (uint64_t)gridDim.x * RS_NT * 4;
  for (uint64_t i0 = (uint64_t)blockIdx.x * RS_NT * 4 + threadIdx.x; i0 - threadIdx.x < n; i0 += stride) {
    uint64_t k[4];
    uint32_t x[4];
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const uint64_t i = i0 + (uint64_t)j * RS_NT;
      k[j] = 0;
      x[j] = 0;
      if (i < n) {
        if constexpr (FROM_COLS) k[j] = pack_row<WIDE>(pa, i, x[j]);
        else {
          k[j] = keys[i];
          if constexpr (WIDE) x[j] = xkeys[i];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const bool in = i0 + (uint64_t)j * RS_NT < n;
      const uint64_t live = ballot(in);
      if (!live) continue;
#pragma unroll
      for (uint32_t p = 0; p < (WIDE ? 12u : 8u); p++) {
        if (p >= passes) break;
        const uint32_t d = digit_at<WIDE>(k[j], x[j], lo_bit + 8 * p);
        const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
        if (ballot(in && d != d0) == 0) {  // (lane 0 is in whenever any lane is)
          if (lane_id() == 0) atomicAdd(&h[(p * 256 + d0) * RH_COPIES], (uint32_t)__popcll(live));
        } else if (in) {
          atomicAdd(&h[(p * 256 + d) * RH_COPIES + copy], 1u);
        }
      }
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < passes * 256; i += RS_NT) {
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < RH_COPIES; j++) c += h[i * RH_COPIES + j];
    if (c) atomicAdd(&hist[i], c);
  }
}

struct RsArgs {
  PackArgs pa;             // first pass of a sort of columns
  UnpackCols ua;           // its last
  const uint64_t* kin;
  const uint32_t* xin;     // wide: the keys' low words
  const void* vin;         // null: every element's value is its input position
  uint64_t* kout;
  uint32_t* xout;
  void* vout;
  uint64_t n;
  uint32_t shift;          // of the pass's digit
  uint32_t tag;            // of the pass, in the status words (from 1)
  uint32_t passes;         // one tile: passes run here
  const uint32_t* hist;    // digit counts of the pass
  uint32_t* status;        // per tile and digit: tag << 16 | the tile's count
  uint64_t* gsum;          // per group and digit, of this pass: tiles added so far << 40 | their count
  uint64_t* gpref;         // per group and digit: tag << 34 | count of all tiles before the group
  uint32_t* ticket;        // tiles handed out so far
};

// One pass over one tile (ONE: every pass of a sort of a single tile).
// Wave w holds the tile's elements [w * RS_ITEMS * 64, (w + 1) * RS_ITEMS *
// 64), item i of lane l at offset i * 64 + l, so a wave's items in order are
// the input order.  A wave ranks its items one after another against digit
// counters of its own (eight ballots find a lane's equal-digit peers; no
// block barrier between items, the wave's LDS operations run in order), one prefix
// over the waves per digit places every element in LDS in digit order, and
// the tile is written out in that order, each digit's run to consecutive
// slots.  The key, its low word and its value go through the same LDS one
// after another.
// Look-back: a tile publishes its digit counts and adds them to its group's;
// it adds up the tiles before it in its group, and the group's first tile
// adds up the groups before (until one whose own prefix is known) and
// publishes that for the others.  Walking back tile by tile instead cost as
// much as the rest of the pass: the reads of other XCDs' words, not their
// latency, were the limit (twice the words per round made it slower).
// Tiles are handed out by a ticket, so all that a tile waits for comes from
// tiles that have started, and each publishes its counts before it waits
// itself: every wait ends.  A word holds a count and the pass (or the number
// of tiles) that makes it valid, and is written and read whole, so no other
// memory has to be ordered with it.
template <int VB, bool FROM_COLS, bool TO_COLS, bool WIDE, bool ONE>
__global__ __launch_bounds__(RS_NT, WIDE || ONE ? 4 : 8) void k_rs_pass(RsArgs a) {
  __shared__ __align__(16) unsigned char s_raw[RS_TILE * 8];
  __shared__ uint32_t s_gbase[256];   // global slot of tile slot 0, per digit (modulo 2^32)
  __shared__ uint32_t s_red[RS_NW];
  __shared__ uint32_t s_tile;
  uint64_t* sk = reinterpret_cast<uint64_t*>(s_raw);
  uint32_t* s32 = reinterpret_cast<uint32_t*>(s_raw);
  uint32_t (*wcnt)[256] = reinterpret_cast<uint32_t(*)[256]>(s_raw);  // per wave, before the keys are staged
  const int tid = threadIdx.x, w = tid / WAVE, lane = tid & (WAVE - 1);
  uint32_t tile = 0;
  if constexpr (!ONE) {
    if (tid == 0) s_tile = atomicAdd(a.ticket, 1u);
    __syncthreads();
    tile = s_tile;
  }
  const uint64_t base = (uint64_t)tile * RS_TILE;
  const uint32_t ntile = (uint32_t)min<uint64_t>(RS_TILE, a.n - base);
  const uint32_t wbase = (uint32_t)w * RS_ITEMS * WAVE;
  uint64_t kk[RS_ITEMS];
  uint32_t xx[WIDE ? RS_ITEMS : 1];
  uint32_t vv[VB == 4 ? RS_ITEMS : 1];
  uint64_t vd[VB == 8 ? RS_ITEMS : 1];
#pragma unroll
  for (int i = 0; i < RS_ITEMS; i++) {
    const uint32_t li = wbase + (uint32_t)i * WAVE + lane;
    kk[i] = 0;
    uint32_t x = 0;
    if (li < ntile) {
      if constexpr (FROM_COLS) kk[i] = pack_row<WIDE>(a.pa, base + li, x);
      else {
        kk[i] = a.kin[base + li];
        if constexpr (WIDE) x = a.xin[base + li];
      }
    }
    if constexpr (WIDE) xx[i] = x;
  }
  auto load_values = [&]() {
#pragma unroll
    for (int i = 0; i < RS_ITEMS; i++) {
      const uint32_t li = wbase + (uint32_t)i * WAVE + lane;
      if constexpr (VB == 4) {
        vv[i] = (uint32_t)(base + li);
        if (a.vin && li < ntile) vv[i] = static_cast<const uint32_t*>(a.vin)[base + li];
      } else if constexpr (VB == 8) {
        vd[i] = li < ntile ? static_cast<const uint64_t*>(a.vin)[base + li] : 0ull;
      }
    }
  };
  if constexpr (ONE) load_values();
  uint32_t lp[RS_ITEMS], pos[RS_ITEMS];
  for (uint32_t pass = 0; pass < (ONE ? a.passes : 1u); pass++) {
    const uint32_t shift = a.shift + 8 * pass;
#pragma unroll
    for (int j = 0; j < RS_NW; j++)
      if (tid < 256) wcnt[j][tid] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RS_ITEMS; i++) {
      const bool valid = wbase + (uint32_t)i * WAVE + lane < ntile;
      const uint32_t d = digit_at<WIDE>(kk[i], WIDE ? xx[WIDE ? i : 0] : 0u, shift);
      // lanes of the same digit: those whose bit b agrees, for all b
      const uint64_t live = ballot(valid);
      uint32_t plo = (uint32_t)live, phi = (uint32_t)(live >> 32);
#pragma unroll
      for (int b = 0; b < 8; b++) {
        const uint32_t bit = (uint32_t)((int32_t)(d << (31 - b)) >> 31);  // all ones or zero
        const uint64_t m = ballot(bit != 0);
        plo &= ~((uint32_t)m ^ bit);
        phi &= ~((uint32_t)(m >> 32) ^ bit);
      }
      const uint64_t peers = ((uint64_t)phi << 32) | plo;
      const uint32_t below = lanes_below(peers);
      const uint32_t pre = valid ? wcnt[w][d] : 0u;
      lp[i] = pre + below;
      // the lowest peer moves the wave's count on, after every peer has read it
      // and before any lane reads it for the next item
      wave_lds_sync();
      if (valid && below == 0) wcnt[w][d] = pre + (uint32_t)__popcll(peers);
      wave_lds_sync();
    }
    __syncthreads();
    uint32_t c = 0;
    if (tid < 256) {
#pragma unroll
      for (int j = 0; j < RS_NW; j++) c += wcnt[j][tid];
      if constexpr (!ONE) {
        __hip_atomic_store(&a.status[(uint64_t)tile * 256 + tid], (a.tag << 16) | c, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        (void)__hip_atomic_fetch_add(&a.gsum[(uint64_t)(tile / RS_GROUP) * 256 + tid], (1ull << 40) | c,
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    uint32_t tot;
    const uint32_t lstart = block_excl_scan<uint32_t, RS_NT>(c, s_red, tot);
    uint32_t gstart = 0;  // first slot of digit tid in the output
    if constexpr (!ONE) gstart = block_excl_scan<uint32_t, RS_NT>(tid < 256 ? a.hist[tid] : 0u, s_red, tot);
    if (tid < 256) {
      uint32_t slot = lstart;
#pragma unroll
      for (int j = 0; j < RS_NW; j++) {
        const uint32_t t = wcnt[j][tid];
        wcnt[j][tid] = slot;
        slot += t;
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RS_ITEMS; i++)
      lp[i] += wcnt[w][digit_at<WIDE>(kk[i], WIDE ? xx[WIDE ? i : 0] : 0u, shift)];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RS_ITEMS; i++)
      if (wbase + (uint32_t)i * WAVE + lane < ntile) sk[lp[i]] = kk[i];
    if constexpr (!ONE) {
      load_values();
      if (tid < 256) {
        const uint32_t g = tile / RS_GROUP;
        uint32_t before = 0;  // elements of the digit in the tiles before
        if (tile % RS_GROUP == 0) {
          for (int64_t j = (int64_t)g - 1; j >= 0;) {
            uint64_t gs[RS_GLOOK], gp[RS_GLOOK];
#pragma unroll
            for (int q = 0; q < RS_GLOOK; q++) {
              const uint64_t at = (uint64_t)max<int64_t>(0, j - q) * 256 + tid;
              gs[q] = __hip_atomic_load(&a.gsum[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              gp[q] = __hip_atomic_load(&a.gpref[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            bool wait = false;
#pragma unroll
            for (int q = 0; q < RS_GLOOK; q++) {
              if (wait || j < 0) continue;
              if ((gs[q] >> 40) != RS_GROUP) {
                wait = true;
                continue;
              }
              before += (uint32_t)gs[q];
              if ((gp[q] >> 34) == a.tag) {
                before += (uint32_t)gp[q];
                j = -1;
              } else {
                j--;
              }
            }
            if (wait) __builtin_amdgcn_s_sleep(1);
          }
          __hip_atomic_store(&a.gpref[(uint64_t)g * 256 + tid], ((uint64_t)a.tag << 34) | before, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        } else {
          for (uint32_t t = g * RS_GROUP; t < tile;) {
            uint32_t st[RS_LOOK];
#pragma unroll
            for (int j = 0; j < RS_LOOK; j++)
              st[j] = __hip_atomic_load(&a.status[(uint64_t)min(t + j, tile) * 256 + tid], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
            bool wait = false;
#pragma unroll
            for (int j = 0; j < RS_LOOK; j++) {
              if (wait || t >= tile) continue;
              if ((st[j] >> 16) != a.tag) {
                wait = true;
              } else {
                before += st[j] & 0xffffu;
                t++;
              }
            }
            if (wait) __builtin_amdgcn_s_sleep(1);
          }
          for (;;) {
            const uint64_t gp = __hip_atomic_load(&a.gpref[(uint64_t)g * 256 + tid], __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
            if ((gp >> 34) == a.tag) {
              before += (uint32_t)gp;
              break;
            }
            __builtin_amdgcn_s_sleep(2);
          }
        }
        s_gbase[tid] = gstart + before - lstart;
      }
    }
    __syncthreads();
    // slot t of the tile: its key, and where it goes
#pragma unroll
    for (int i = 0; i < RS_ITEMS; i++) {
      const uint32_t t = (uint32_t)i * RS_NT + tid;
      pos[i] = t;
      if constexpr (ONE) {
        // back into the wave's items for the next pass
        const uint32_t li = wbase + (uint32_t)i * WAVE + lane;
        kk[i] = li < ntile ? sk[li] : 0ull;
        pos[i] = li;
      } else if constexpr (!WIDE) {
        if (t < ntile) {
          const uint64_t k = sk[t];
          pos[i] = s_gbase[digit_at<false>(k, 0u, shift)] + t;
          if constexpr (TO_COLS) unpack_row<false>(a.ua, pos[i], k, 0u);
          else a.kout[pos[i]] = k;
        }
      } else {
        kk[i] = t < ntile ? sk[t] : 0ull;
      }
    }
    if constexpr (WIDE) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < RS_ITEMS; i++)
        if (wbase + (uint32_t)i * WAVE + lane < ntile) s32[lp[i]] = xx[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < RS_ITEMS; i++) {
        const uint32_t t = pos[i];
        const uint32_t x = t < ntile ? s32[t] : 0u;
        if constexpr (ONE) xx[i] = x;
        else if (t < ntile) {
          pos[i] = s_gbase[digit_at<true>(kk[i], x, shift)] + t;
          if constexpr (TO_COLS) unpack_row<true>(a.ua, pos[i], kk[i], x);
          else {
            a.kout[pos[i]] = kk[i];
            a.xout[pos[i]] = x;
          }
        }
      }
    }
    if constexpr (VB == 4) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < RS_ITEMS; i++)
        if (wbase + (uint32_t)i * WAVE + lane < ntile) s32[lp[i]] = vv[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < RS_ITEMS; i++) {
        const uint32_t t = ONE ? pos[i] : (uint32_t)i * RS_NT + tid;
        if constexpr (ONE) vv[i] = t < ntile ? s32[t] : 0u;
        else if (t < ntile) static_cast<uint32_t*>(a.vout)[pos[i]] = s32[t];
      }
    } else if constexpr (VB == 8) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < RS_ITEMS; i++)
        if (wbase + (uint32_t)i * WAVE + lane < ntile) sk[lp[i]] = vd[i];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < RS_ITEMS; i++) {
        const uint32_t t = ONE ? pos[i] : (uint32_t)i * RS_NT + tid;
        if constexpr (ONE) vd[i] = t < ntile ? sk[t] : 0ull;
        else if (t < ntile) static_cast<uint64_t*>(a.vout)[pos[i]] = sk[t];
      }
    }
    if constexpr (ONE) __syncthreads();
  }
  if constexpr (ONE) {
#pragma unroll
    for (int i = 0; i < RS_ITEMS; i++) {
      const uint32_t li = wbase + (uint32_t)i * WAVE + lane;
      if (li >= ntile) continue;
      if constexpr (TO_COLS) unpack_row<WIDE>(a.ua, li, kk[i], WIDE ? xx[WIDE ? i : 0] : 0u);
      else a.kout[li] = kk[i];
      if constexpr (VB == 4) static_cast<uint32_t*>(a.vout)[li] = vv[i];
      if constexpr (VB == 8) static_cast<uint64_t*>(a.vout)[li] = vd[i];
    }
  }
}

template <int VB, bool WIDE>
void launch_rs_pass(bool from_cols, bool to_cols, unsigned grid, hipStream_t s, const RsArgs& a) {
  if (from_cols && to_cols) k_rs_pass<VB, true, true, WIDE, false><<<grid, RS_NT, 0, s>>>(a);
  else if (from_cols) k_rs_pass<VB, true, false, WIDE, false><<<grid, RS_NT, 0, s>>>(a);
  else if (to_cols) k_rs_pass<VB, false, true, WIDE, false><<<grid, RS_NT, 0, s>>>(a);
  else k_rs_pass<VB, false, false, WIDE, false><<<grid, RS_NT, 0, s>>>(a);
  LH_HIP(hipGetLastError());
}

__global__ void k_pack(PackArgs a, const uint32_t* perm, uint64_t* out, uint64_t n) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
{
    uint32_t x;
    out[i] = pack_row<false>(a, perm ? perm[i] : (uint32_t)i, x);
  }
}

__device__ __forceinline__ int32_t lowest_bit_exp(double v) {
  uint64_t b = (uint64_t)__double_as_longlong(v);
  uint32_t ex = (uint32_t)(b >> 52) & 0x7ffu;
  uint64_t mant = b & ((1ull << 52) - 1);
  if (ex == 0) return -1074 + (int32_t)__builtin_ctzll(mant);
  mant |= 1ull << 52;
  return (int32_t)ex - 1075 + (int32_t)__builtin_ctzll(mant);
}

__global__ void k_anno_stats(const double* v, uint64_t n, AnnoAcc* acc) {
  int32_t q = INT_MAX;
  uint64_t m = 0;
  uint32_t bad = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    double x = v[i];
    if (!isfinite(x)) { bad = 1; continue; }
    if (x == 0.0) continue;
    q = min(q, lowest_bit_exp(x));
    uint64_t ab = (uint64_t)__double_as_longlong(fabs(x));
    m = max(m, ab);
  }
#pragma unroll
  for (int d = WAVE / 2; d > 0; d >>= 1) {
    q = min(q, __shfl_xor(q, d, WAVE));
    m = max(m, (uint64_t)__shfl_xor((unsigned long long)m, d, WAVE));
    bad |= (uint32_t)__shfl_xor((int)bad, d, WAVE);
  }
  // one update per workgroup, and only when it changes the result (the
  // same three words are the target of every workgroup)
  __shared__ int32_t s_q[8];
  __shared__ unsigned long long s_m[8];
  __shared__ uint32_t s_b[8];
  const int w = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
  if (lane_id() == 0) {
    s_q[w] = q;
    s_m[w] = m;
    s_b[w] = bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int j = 1; j < nw; j++) {
      q = min(q, s_q[j]);
      m = max(m, (uint64_t)s_m[j]);
      bad |= s_b[j];
    }
    const uint32_t qe = (uint32_t)(INT_MAX - (int64_t)q);
    if (qe > __hip_atomic_load(&acc->qenc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&acc->qenc, qe);
    if (m > __hip_atomic_load(&acc->maxabs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&acc->maxabs, (unsigned long long)m);
    if (bad && !__hip_atomic_load(&acc->nonfinite, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicOr(&acc->nonfinite, 1u);
  }
}

}  // namespace

uint64_t scan_u32_to_u64(const uint32_t* in, uint64_t* out, uint64_t n, hipStream_t s) {
  return scan_impl<uint32_t, uint64_t>(in, out, n, s);
}
uint64_t scan_u64(const uint64_t* in, uint64_t* out, uint64_t n, hipStream_t s) {
  return scan_impl<uint64_t, uint64_t>(in, out, n, s);
}
uint32_t scan_u32(const uint32_t* in, uint32_t* out, uint64_t n, hipStream_t s) {
  return scan_impl<uint32_t, uint32_t>(in, out, n, s);
}
void scan_u32_dev(const uint32_t* in, uint32_t* out, uint64_t n, hipStream_t s) {
  scan_dev<uint32_t, uint32_t>(in, out, n, s);
}
void scan_u32_to_u64_dev(const uint32_t* in, uint64_t* out, uint64_t n, hipStream_t s) {
  scan_dev<uint32_t, uint64_t>(in, out, n, s);
}

uint32_t reduce_max_u32(const uint32_t* in, uint64_t n, hipStream_t s) {
  DBuf<uint32_t> r(1, s);
  LH_HIP(hipMemsetAsync(r.p, 0, sizeof(uint32_t), s));
  if (n) {
    k_reduce_max_u32<<<std::min(grid_for((n + 3) / 4), 2048u), 256, 0, s>>>(in, n, r.p);
    LH_HIP(hipGetLastError());
  }
  return read_scalar(r.p, s);
}

void column_maxima(const uint32_t* const* cols, const uint64_t* n, uint32_t ncols, uint32_t* out, hipStream_t s) {
  if (ncols > MAX_COLS) fail(LH_ERR_UNSUPPORTED, "more than 24 columns");
  MaxCols a{};
  uint64_t most = 0;
  for (uint32_t c = 0; c < ncols; c++) {
    a.col[c] = cols[c];
    a.n[c] = n[c];
    most = std::max(most, n[c]);
  }
  for (uint32_t c = 0; c < ncols; c++) out[c] = 0;
  if (!most) return;
  struct Maxima {
    uint32_t v[MAX_COLS];
  };
  DBuf<Maxima> m(1, s);
  LH_HIP(hipMemsetAsync(m.p, 0, sizeof(Maxima), s));
  k_max_cols<<<dim3(std::min(grid_for((most + 7) / 8), 1024u), ncols), 256, 0, s>>>(a, m.p->v);
  LH_HIP(hipGetLastError());
  const Maxima h = read_scalar(m.p, s);
  for (uint32_t c = 0; c < ncols; c++) out[c] = h.v[c];
}

uint64_t select_flagged(const uint32_t* flags, uint64_t n, uint32_t* out, hipStream_t s) {
  DBuf<uint64_t> off(n + 1, s);
  uint64_t m = scan_u32_to_u64(flags, off.p, n, s);
  if (m) {
    k_scatter_flagged<<<grid_for(n), 256, 0, s>>>(flags, off.p, n, out);
    LH_HIP(hipGetLastError());
  }
  return m;
}

// Runs of a sorted column: their number and the longest.  A wave takes
// RS_GROUPS groups of 64 consecutive values, all loads issued together; a
// ballot of each group's run heads gives every run that ends inside the
// group its length, and a run still going at a group's end is carried into
// the next group.  One still going at the wave's last value is followed
// into the next 64 values with one more load and a ballot; only a run
// longer than that gallops to its end (probes 1, 2, 4, ... past them, then
// bisects the last step).  Each block writes its count and longest run
// (atomics of every block on one address would serialize).
constexpr int RS_GROUPS = 8;

struct RunStats {
  unsigned long long distinct;
  unsigned int longest;
  unsigned int pad;
};

__global__ __launch_bounds__(256) void k_run_stats(const uint32_t* v, uint64_t n, RunStats* part) {
  __shared__ uint32_t s_red[256 / WAVE];
  const int lane = lane_id();
  uint32_t heads = 0, longest = 0;
  constexpr uint64_t span = (uint64_t)RS_GROUPS * WAVE;
  const uint64_t wave = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / WAVE;
  const uint64_t nwaves = (uint64_t)gridDim.x * blockDim.x / WAVE;
  for (uint64_t c0 = wave * span; c0 < n; c0 += nwaves * span) {
    uint32_t xs[RS_GROUPS];
#pragma unroll
    for (int g = 0; g < RS_GROUPS; g++) {
      const uint64_t i = c0 + (uint64_t)g * WAVE + lane;
      xs[g] = i < n ? v[i] : 0u;
    }
    const uint32_t before = c0 > 0 ? v[c0 - 1] : 0u;
    bool open = false;      // a run started at os (value xo) is still going (uniform over the wave)
    uint64_t os = 0;
    uint32_t xo = 0;
#pragma unroll
    for (int g = 0; g < RS_GROUPS; g++) {
      const uint64_t g0 = c0 + (uint64_t)g * WAVE, i = g0 + lane;
      const uint32_t x = xs[g];
      const uint32_t last_before = g ? (uint32_t)__shfl((int)xs[g > 0 ? g - 1 : 0], WAVE - 1, WAVE) : before;
      uint32_t p = (uint32_t)__shfl_up((int)x, 1, WAVE);
      if (lane == 0) p = last_before;
      const bool head = i < n && (i == 0 || p != x);
      const uint64_t Hh = ballot(head);
      // lanes past the end count as heads: a run ends at the next set bit
      const uint64_t H = Hh | ballot(i >= n);
      if (open && H) {
        if (lane == 0) longest = max(longest, (uint32_t)(g0 + (uint64_t)__builtin_ctzll(H) - os));
        open = false;
      }
      if (head) heads++;
      const uint64_t above = lane < WAVE - 1 ? H >> (lane + 1) : 0ull;
      if (head && above) longest = max(longest, (uint32_t)__builtin_ctzll(above) + 1u);
      // the last head's run reaches the group's last lane (every lane in range)
      if (Hh && !((H >> (63 - __builtin_clzll(Hh))) >> 1)) {
        open = true;
        os = g0 + (uint64_t)(63 - __builtin_clzll(Hh));
        xo = (uint32_t)__shfl((int)x, WAVE - 1, WAVE);
      }
    }
    if (open) {  // it reaches c0 + span - 1 < n
      const uint64_t e0 = c0 + span, k = e0 + lane;
      const uint64_t D = ballot(k >= n || v[k] != xo);
      uint64_t end = e0 + (D ? (uint64_t)__builtin_ctzll(D) : 0u);
      if (!D && lane == 0) {
        uint64_t lo = e0 + WAVE - 1, step = 1;  // v[lo] == xo
        while (lo + step < n && v[lo + step] == xo) {
          lo += step;
          step <<= 1;
        }
        uint64_t hi = min<uint64_t>(lo + step, n);  // v[hi] != xo, or hi == n
        while (hi - lo > 1) {
          const uint64_t mid = lo + (hi - lo) / 2;
          if (v[mid] == xo) lo = mid;
          else hi = mid;
        }
        end = hi;
      }
      if (lane == 0) longest = max(longest, (uint32_t)(end - os));
    }
  }
  const uint32_t h = block_sum<uint32_t, 256>(heads, s_red);  // ends with a barrier: s_red is free
#pragma unroll
  for (int d = WAVE / 2; d > 0; d >>= 1) longest = max(longest, (uint32_t)__shfl_xor((int)longest, d, WAVE));
  if (lane == 0) s_red[threadIdx.x / WAVE] = longest;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t m = 0;
    for (int w = 0; w < 256 / WAVE; w++) m = max(m, s_red[w]);
    part[blockIdx.x] = RunStats{h, m, 0u};
  }
}

// The blocks' partial run statistics summed and maximized by one block.
__global__ __launch_bounds__(256) void k_run_stats_total(const RunStats* part, uint32_t nb, RunStats* out) {
  __shared__ unsigned long long s_d[256 / WAVE];
  __shared__ uint32_t s_m[256 / WAVE];
  unsigned long long d = 0;
  uint32_t m = 0;
  for (uint32_t b = threadIdx.x; b < nb; b += blockDim.x) {
    d += part[b].distinct;
    m = max(m, part[b].longest);
  }
  d = wave_sum(d);
#pragma unroll
  for (int o = WAVE / 2; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, WAVE));
  if (lane_id() == 0) {
    s_d[threadIdx.x / WAVE] = d;
    s_m[threadIdx.x / WAVE] = m;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    RunStats r{0ull, 0u, 0u};
    for (int w = 0; w < 256 / WAVE; w++) {
      r.distinct += s_d[w];
      r.longest = max(r.longest, s_m[w]);
    }
    *out = r;
  }
}

void column_freq(const uint32_t* col, uint64_t n, uint32_t range, uint64_t& distinct, uint64_t& freq_max,
                 hipStream_t s) {
  // sort the values (no atomics: hub values would serialize them), then
  // the distinct values are the runs and the largest frequency the longest
  // run
  distinct = 0;
  freq_max = 0;
  if (!n) return;
  const uint32_t bits = range ? 32 - __builtin_clz(range) : 0;
  DBuf<uint32_t> sorted(n, s);
  uint32_t* out = sorted.p;
  if (!sort_packed(&col, &bits, 1, n, SortValue{}, &out, s)) fail(LH_ERR_DEVICE, "column statistics: sort failed");
  sorted_run_stats(sorted.p, n, distinct, freq_max, s);
}

void sorted_run_stats(const uint32_t* sorted, uint64_t n, uint64_t& distinct, uint64_t& freq_max, hipStream_t s) {
  distinct = 0;
  freq_max = 0;
  if (!n) return;
  const unsigned nb = grid_for((n + RS_GROUPS - 1) / RS_GROUPS);
  DBuf<RunStats> part(nb, s), r(1, s);
  k_run_stats<<<nb, 256, 0, s>>>(sorted, n, part.p);
  LH_HIP(hipGetLastError());
  k_run_stats_total<<<1, 256, 0, s>>>(part.p, nb, r.p);
  LH_HIP(hipGetLastError());
  const RunStats h = read_scalar(r.p, s);
  distinct = h.distinct;
  freq_max = h.longest;
}

void iota_u32(uint32_t* out, uint64_t n, hipStream_t s) {
  if (!n) return;
  k_iota<<<grid_for(n), 256, 0, s>>>(out, n);
  LH_HIP(hipGetLastError());
}
void fill_u32(uint32_t* out, uint32_t v, uint64_t n, hipStream_t s) {
  if (!n) return;
  k_fill<uint32_t><<<grid_for(n), 256, 0, s>>>(out, v, n);
  LH_HIP(hipGetLastError());
}
void fill_u64(uint64_t* out, uint64_t v, uint64_t n, hipStream_t s) {
  if (!n) return;
  k_fill<uint64_t><<<grid_for(n), 256, 0, s>>>(out, v, n);
  LH_HIP(hipGetLastError());
}
void gather_u32(const uint32_t* src, const uint32_t* idx, uint32_t* dst, uint64_t n, hipStream_t s) {
  if (!n) return;
  k_gather<uint32_t><<<grid_for(n), 256, 0, s>>>(src, idx, dst, n);
  LH_HIP(hipGetLastError());
}
void gather_f64(const double* src, const uint32_t* idx, double* dst, uint64_t n, hipStream_t s) {
  if (!n) return;
  k_gather<double><<<grid_for(n), 256, 0, s>>>(src, idx, dst, n);
  LH_HIP(hipGetLastError());
}

namespace {

// One radix sort.  Passes cover bits [lo_bit, lo_bit + 8 * passes) of the
// keys.  The first pass reads io.pa's columns when from_cols (else kin, xin)
// and the last writes io.ua's columns when to_cols (else the keys).  Pass p
// writes buffers (p + phase) & 1.  Values (vb bytes each, 0: none) start in
// vin (null: the input positions, vb = 4).
struct RadixIO {
  PackArgs pa{};
  UnpackCols ua{};
  bool from_cols = false, to_cols = false, wide = false;
  const uint64_t* kin = nullptr;
  uint64_t* kbuf[2] = {nullptr, nullptr};
  uint32_t* xbuf[2] = {nullptr, nullptr};
  int vb = 0;
  const void* vin = nullptr;
  void* vbuf[2] = {nullptr, nullptr};
  uint32_t phase = 0;
};

// (keys that are no columns have one word, and a row number or nothing with them)
template <int VB, bool WIDE>
void launch_one_tile(const RadixIO& io, const RsArgs& a, hipStream_t s) {
  if (io.from_cols) {
    k_rs_pass<VB, true, true, WIDE, true><<<1, RS_NT, 0, s>>>(a);
  } else {
    if constexpr (WIDE || VB == 8) fail(LH_ERR_UNSUPPORTED, "radix sort: wide keys or values without columns");
    else k_rs_pass<VB, false, false, false, true><<<1, RS_NT, 0, s>>>(a);
  }
  LH_HIP(hipGetLastError());
}

template <class F>
void by_value_and_width(const RadixIO& io, F&& f) {
  using std::integral_constant;
  if (io.wide) {
    if (io.vb == 0) f(integral_constant<int, 0>{}, std::true_type{});
    else if (io.vb == 4) f(integral_constant<int, 4>{}, std::true_type{});
    else f(integral_constant<int, 8>{}, std::true_type{});
  } else {
    if (io.vb == 0) f(integral_constant<int, 0>{}, std::false_type{});
    else if (io.vb == 4) f(integral_constant<int, 4>{}, std::false_type{});
    else f(integral_constant<int, 8>{}, std::false_type{});
  }
}

void radix_passes(const RadixIO& io, uint64_t n, uint32_t lo_bit, uint32_t passes, hipStream_t s) {
  RsArgs a{};
  a.pa = io.pa;
  a.ua = io.ua;
  a.n = n;
  a.kin = io.kin;
  a.vin = io.vin;
  const uint64_t ntiles = (n + RS_TILE - 1) / RS_TILE;
  const uint64_t kb = io.wide ? 12 : 8;
  const uint64_t in_bytes = io.from_cols ? 4ull * io.pa.ncols : kb, out_bytes = io.to_cols ? 4ull * io.ua.ncols : kb;
  if (ntiles == 1 && io.from_cols == io.to_cols) {
    // one tile: every pass in one launch, the last pass's buffers written
    a.shift = lo_bit;
    a.passes = passes;
    a.kout = io.kbuf[(passes - 1 + io.phase) & 1];
    a.vout = io.vbuf[(passes - 1 + io.phase) & 1];
    ProfScope ps("sort_scatter", s, n, (in_bytes + out_bytes + (io.vb ? 2 * io.vb : 0)) * n);
    by_value_and_width(io, [&](auto vb, auto wide) { launch_one_tile<vb.value, wide.value>(io, a, s); });
    return;
  }
  // digit counts of all passes, the tickets and the look-back's words (the
  // tiles' counts and the groups' prefixes are tagged by pass), cleared once
  const uint64_t ngroups = (ntiles + RS_GROUP - 1) / RS_GROUP;
  const uint64_t head = (uint64_t)RS_MAXP * 256 + RS_MAXP + 4;  // 32-bit words before the 64-bit ones (even)
  DBuf<uint32_t> ws(head + ngroups * 512 * (passes + 1) + ntiles * 256, s);
  LH_HIP(hipMemsetAsync(ws.p, 0, ws.n * sizeof(uint32_t), s));
  {
    // elements: the pass's algorithmic bytes (its keys read)
    ProfScope ps("sort_hist", s, n, in_bytes * n);
    const unsigned grid = (unsigned)std::min<uint64_t>(ntiles, 1024);
    if (io.from_cols && io.wide) k_rs_hist<true, true><<<grid, RS_NT, 0, s>>>(nullptr, nullptr, io.pa, n, lo_bit, passes, ws.p);
    else if (io.from_cols) k_rs_hist<true, false><<<grid, RS_NT, 0, s>>>(nullptr, nullptr, io.pa, n, lo_bit, passes, ws.p);
    else k_rs_hist<false, false><<<grid, RS_NT, 0, s>>>(io.kin, nullptr, io.pa, n, lo_bit, passes, ws.p);
  }
  LH_HIP(hipGetLastError());
  a.gpref = reinterpret_cast<uint64_t*>(ws.p + head);
  a.status = ws.p + head + ngroups * 512 * (passes + 1);
  for (uint32_t p = 0; p < passes; p++) {
    const bool fc = p == 0 && io.from_cols, tc = p + 1 == passes && io.to_cols;
    const uint32_t to = (p + io.phase) & 1;
    a.shift = lo_bit + p * 8;
    a.tag = p + 1;
    a.hist = ws.p + p * 256;
    a.ticket = ws.p + RS_MAXP * 256 + p;
    a.gsum = a.gpref + ngroups * 256 * (p + 1);
    a.kout = io.kbuf[to];
    a.xout = io.xbuf[to];
    a.vout = io.vbuf[to];
    // elements: the pass's algorithmic bytes (keys, and values when they
    // travel, read once and written once; values made from positions are
    // written only)
    const uint64_t vbytes = io.vb ? (a.vin ? 2 : 1) * io.vb : 0;
    ProfScope ps("sort_scatter", s, n, ((fc ? in_bytes : kb) + (tc ? out_bytes : kb) + vbytes) * n);
    by_value_and_width(io, [&](auto vb, auto wide) { launch_rs_pass<vb.value, wide.value>(fc, tc, (unsigned)ntiles, s, a); });
    a.kin = a.kout;
    a.xin = a.xout;
    a.vin = a.vout;
  }
}

}  // namespace

void radix_sort_pairs(uint64_t* keys, uint32_t* vals, uint64_t* tkeys, uint32_t* tvals, uint64_t n,
                      uint32_t bits, hipStream_t s, uint32_t lo_bit) {
  // vals == nullptr: keys only
  if (n <= 1 || bits <= lo_bit) return;
  if (n >= (1ull << 32)) fail(LH_ERR_OVERFLOW, "radix sort: more than 2^32 - 1 keys");
  const uint32_t passes = (bits - lo_bit + 7) / 8;
  // pass p writes buffer (p + 1) & 1: the first writes the temporaries,
  // the last the caller's buffers when the count is even
  RadixIO io;
  io.kin = keys;
  io.kbuf[0] = keys;
  io.kbuf[1] = tkeys;
  io.vb = vals ? 4 : 0;
  io.vin = vals;
  io.vbuf[0] = vals;
  io.vbuf[1] = tvals;
  io.phase = 1;
  radix_passes(io, n, lo_bit, passes, s);
  if (passes & 1) {
    LH_HIP(hipMemcpyAsync(keys, tkeys, n * sizeof(uint64_t), hipMemcpyDeviceToDevice, s));
    if (vals) LH_HIP(hipMemcpyAsync(vals, tvals, n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
  }
}

uint32_t radix_sort_between(uint64_t* const k[2], uint32_t* const v[2], uint64_t n, uint32_t bits, hipStream_t s) {
  if (n <= 1 || !bits) return 0;
  if (n >= (1ull << 32)) fail(LH_ERR_OVERFLOW, "radix sort: more than 2^32 - 1 keys");
  const uint32_t passes = (bits + 7) / 8;
  RadixIO io;
  io.kin = k[0];
  io.vin = v[0];
  io.vb = 4;
  for (int i = 0; i < 2; i++) {
    io.kbuf[i] = k[i];
    io.vbuf[i] = v[i];
  }
  io.phase = 1;
  radix_passes(io, n, 0, passes, s);
  return passes & 1;
}

void lex_sort_perm(const uint32_t* const* cols, const uint32_t* bits, uint32_t ncols, uint64_t n, uint32_t* perm,
                   hipStream_t s) {
  iota_u32(perm, n, s);
  if (n <= 1) return;
  DBuf<uint64_t> k(n, s), tk(n, s);
  DBuf<uint32_t> tv(n, s);
  int end = (int)ncols;
  while (end > 0) {
    int start = end - 1;
    uint32_t tot = bits[start];
    while (start > 0 && tot + bits[start - 1] <= 64) {
      start--;
      tot += bits[start];
    }
    if (tot > 0) {
      PackArgs a{};
      a.ncols = (uint32_t)(end - start);
      uint32_t sh = 0;
      for (int c = end - 1; c >= start; c--) {  // least significant column at the bottom
        a.col[c - start] = cols[c];
        a.shift[c - start] = sh;
        sh += bits[c];
      }
      k_pack<<<grid_for(n), 256, 0, s>>>(a, perm, k.p, n);
      LH_HIP(hipGetLastError());
      radix_sort_pairs(k.p, perm, tk.p, tv.p, n, tot, s);
    }
    end = start;
  }
}

bool sort_packed(const uint32_t* const* cols, const uint32_t* bits, uint32_t ncols, uint64_t n, const SortValue& val,
                 uint32_t* const* sorted, hipStream_t s, uint32_t sorted_tail) {
  uint32_t tot = 0;
  for (uint32_t c = 0; c < ncols; c++) tot += bits[c];
  if (tot > 96 || ncols > LH_MAX_KEYS) return false;
  if (!n) return true;
  if (n >= (1ull << 32)) fail(LH_ERR_OVERFLOW, "radix sort: more than 2^32 - 1 keys");
  RadixIO io;
  io.wide = tot > 64;
  io.pa.ncols = io.ua.ncols = ncols;
  uint32_t sh = 0;
  for (int c = (int)ncols - 1; c >= 0; c--) {  // the last column lowest
    io.pa.col[c] = cols[c];
    // (a leading column of no bits holds zeros: any shift below the width)
    io.pa.shift[c] = io.ua.shift[c] = bits[c] ? sh : 0;
    io.ua.bits[c] = bits[c];
    io.ua.col[c] = sorted[c];
    sh += bits[c];
  }
  uint32_t tail_bits = 0;
  for (uint32_t c = ncols - std::min(sorted_tail, ncols); c < ncols; c++) tail_bits += bits[c];
  const uint32_t passes = tot > tail_bits ? (tot - tail_bits + 7) / 8 : 0;
  if (!passes) {
    // in order already: every value fits its column's bits, so the sorted
    // columns are copies
    for (uint32_t c = 0; c < ncols; c++)
      LH_HIP(hipMemcpyAsync(sorted[c], cols[c], n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
    if (val.bytes && val.in) LH_HIP(hipMemcpyAsync(val.out, val.in, n * val.bytes, hipMemcpyDeviceToDevice, s));
    else if (val.bytes) iota_u32(static_cast<uint32_t*>(val.out), n, s);
    return true;
  }
  // the first pass packs the columns, the last unpacks into `sorted`; the
  // values end in val.out
  DBuf<uint64_t> k(passes > 1 ? n : 0, s), tk(passes > 2 ? n : 0, s);
  DBuf<uint32_t> x(passes > 1 && io.wide ? n : 0, s), tx(passes > 2 && io.wide ? n : 0, s);
  DBuf<uint64_t> tv(val.bytes && passes > 1 ? (n * val.bytes + 7) / 8 : 0, s);
  // pass p writes buffer (p + phase) & 1: the last writes vbuf[0] =
  // val.out, the first writes k
  io.phase = (passes - 1) & 1;
  io.from_cols = io.to_cols = true;
  io.kbuf[io.phase] = k.p;
  io.kbuf[io.phase ^ 1] = tk.p;
  io.xbuf[io.phase] = x.p;
  io.xbuf[io.phase ^ 1] = tx.p;
  io.vb = (int)val.bytes;
  io.vin = val.in;
  io.vbuf[0] = val.out;
  io.vbuf[1] = tv.p;
  radix_passes(io, n, tail_bits, passes, s);
  return true;
}

void anno_stats_into(const double* v, uint64_t n, AnnoAcc* acc, hipStream_t s) {
  if (!n) return;
  k_anno_stats<<<std::min(grid_for((n + 3) / 4), 4096u), 256, 0, s>>>(v, n, acc);
  LH_HIP(hipGetLastError());
}

AnnoStats decode_anno_stats(const AnnoAcc& a) {
  AnnoStats st;
  st.qmin = (int32_t)((int64_t)INT_MAX - (int64_t)a.qenc);
  memcpy(&st.maxabs, &a.maxabs, sizeof st.maxabs);
  st.nonfinite = a.nonfinite;
  return st;
}

AnnoStats anno_stats(const double* v, uint64_t n, hipStream_t s) {
  DBuf<AnnoAcc> acc(1, s);
  LH_HIP(hipMemsetAsync(acc.p, 0, sizeof(AnnoAcc), s));
  anno_stats_into(v, n, acc.p, s);
  return decode_anno_stats(read_scalar(acc.p, s));
}

}  // namespace lh
