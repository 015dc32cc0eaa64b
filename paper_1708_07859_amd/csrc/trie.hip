// Trie construction (section 2.2): lexicographic sort of the key tuples in
// level order, head flags per level, per-level keys and child offsets,
// set-mode deduplication or bag-mode runs, annotation/meta gathering and the
// per-set uint/bitset layout.
#include <algorithm>
#include <cstring>
#include <memory>

#include "device_common.h"
#include "lh_internal.h"

namespace lh {

namespace {

constexpr int TB_NT = 256;  // rows per tile in the level builder
constexpr int TB_NW = TB_NT / WAVE;

struct LevelCols {
  const uint32_t* k[LH_MAX_KEYS];  // sorted key column per level
  uint32_t n_levels;
};

__device__ __forceinline__ uint32_t head_mask(const LevelCols& c, uint64_t r) {
  // bit l set when row r starts a new node at level l
  // (levels unrolled: constant indices keep the column pointers in registers)
  uint32_t m = 0;
  bool h = (r == 0);
#pragma unroll
  for (uint32_t l = 0; l < LH_MAX_KEYS; l++) {
    if (l < c.n_levels) {
      if (!h) h = c.k[l][r] != c.k[l][r - 1];
      if (h) m |= 1u << l;
    }
  }
  return m;
}

// Heads per level per tile: counts[l * ntiles + tile].
__global__ __launch_bounds__(TB_NT) void k_head_counts(LevelCols c, uint64_t n, uint32_t* counts, uint32_t ntiles) {
  __shared__ uint32_t w_cnt[TB_NW][LH_MAX_KEYS];
  uint64_t r = (uint64_t)blockIdx.x * TB_NT + threadIdx.x;
  uint32_t m = r < n ? head_mask(c, r) : 0;
  const int w = threadIdx.x / WAVE;
#pragma unroll
  for (uint32_t l = 0; l < LH_MAX_KEYS; l++) {
    if (l < c.n_levels) {
      uint64_t b = ballot((m >> l) & 1u);
      if (lane_id() == 0) w_cnt[w][l] = (uint32_t)__popcll(b);
    }
  }
  __syncthreads();
  if (threadIdx.x < c.n_levels) {
    uint32_t t = 0;
    for (int j = 0; j < TB_NW; j++) t += w_cnt[j][threadIdx.x];
    counts[(uint64_t)threadIdx.x * ntiles + blockIdx.x] = t;
  }
}

struct EmitArgs {
  LevelCols c;
  uint32_t* keys_out[LH_MAX_KEYS];   // level keys
  uint32_t* offs_out[LH_MAX_KEYS];   // level child offsets (levels 0..L-2)
  uint32_t* run_out;                 // bag: leaf run starts (sorted-row index); may be null
  uint32_t* kept_out;                // set: sorted-row index of each kept row; may be null
  uint32_t* rowkeys_out[LH_MAX_KEYS]; // set: each kept row's keys of the levels above the last; null when not wanted
  uint32_t* parent_out[LH_MAX_KEYS]; // level l >= 1: the level l-1 node above each node; may be null
  uint32_t* samp_out[LH_MAX_KEYS];   // line samples of each level
  const uint32_t* tile_off;          // [l * ntiles + tile]: one scan over all levels' counts
  uint32_t level_base[LH_MAX_KEYS];  // tile_off of the level's first tile
  uint32_t level_n[LH_MAX_KEYS];     // nodes per level
  uint32_t ntiles;
};

__global__ __launch_bounds__(TB_NT) void k_emit_levels(EmitArgs a, uint64_t n) {
  __shared__ uint32_t w_cnt[TB_NW][LH_MAX_KEYS];
  uint64_t r = (uint64_t)blockIdx.x * TB_NT + threadIdx.x;
  uint32_t m = r < n ? head_mask(a.c, r) : 0;
  const int w = threadIdx.x / WAVE;
  uint32_t rank[LH_MAX_KEYS];
#pragma unroll
  for (uint32_t l = 0; l < LH_MAX_KEYS; l++) {
    rank[l] = 0;
    if (l < a.c.n_levels) {
      uint64_t b = ballot((m >> l) & 1u);
      rank[l] = lanes_below(b);
      if (lane_id() == 0) w_cnt[w][l] = (uint32_t)__popcll(b);
    }
  }
  __syncthreads();
  if (r >= n) return;
  const uint32_t L = a.c.n_levels;
  uint32_t pos_prev = 0;
#pragma unroll
  for (uint32_t l = 0; l < LH_MAX_KEYS; l++) {
    if (l >= L || !((m >> l) & 1u)) continue;
    uint32_t pre = 0;
    for (int j = 0; j < w; j++) pre += w_cnt[j][l];
    uint32_t pos = a.tile_off[(uint64_t)l * a.ntiles + blockIdx.x] - a.level_base[l] + pre + rank[l];
    const uint32_t key = a.c.k[l][r];
    a.keys_out[l][pos] = key;
    if (!(pos & ((1u << LINE_SHIFT) - 1))) a.samp_out[l][pos >> LINE_SHIFT] = key;
    if (l > 0 && a.parent_out[l]) {
      // the parent is the last level l-1 node starting at or before row r
      uint32_t pp = 0;
      for (int j = 0; j < w; j++) pp += w_cnt[j][l - 1];
      a.parent_out[l][pos] = a.tile_off[(uint64_t)(l - 1) * a.ntiles + blockIdx.x] - a.level_base[l - 1] + pp +
                             rank[l - 1] + ((m >> (l - 1)) & 1u) - 1u;
    }
    // a head at level l-1 is also a head at l: its first child is pos
    if (l > 0 && ((m >> (l - 1)) & 1u)) a.offs_out[l - 1][pos_prev] = pos;
    if (l + 1 == L) {
      if (a.run_out) a.run_out[pos] = (uint32_t)r;
      if (a.kept_out) a.kept_out[pos] = (uint32_t)r;
#pragma unroll
      for (uint32_t j = 0; j < LH_MAX_KEYS; j++)
        if (j + 1 < L && a.rowkeys_out[j]) a.rowkeys_out[j][pos] = a.c.k[j][r];
    }
    pos_prev = pos;
  }
  if (r + 1 == n) {  // closing offsets
#pragma unroll
    for (uint32_t l = 0; l + 1 < LH_MAX_KEYS; l++)
      if (l + 1 < L) a.offs_out[l][a.level_n[l]] = a.level_n[l + 1];
#pragma unroll
    for (uint32_t l = 0; l < LH_MAX_KEYS; l++)
      if (l + 1 == L && a.run_out) a.run_out[a.level_n[l]] = (uint32_t)n;
  }
}

// Nodes of each level, from the scan of all levels' tile counts.
__global__ void k_level_totals(const uint32_t* tile_off, uint32_t ntiles, uint32_t n_levels, uint32_t* out) {
  const uint32_t l = threadIdx.x;
  if (l < n_levels) out[l] = tile_off[(uint64_t)(l + 1) * ntiles] - tile_off[(uint64_t)l * ntiles];
}

// What the build needs to know of its input: every level's largest key and,
// when asked, how much of it is in order (bit t-1 of the mask stays set while
// rows i-1, i are in lexicographic order of the last t levels, for every i;
// equal tuples are in order).
struct InputStats {
  uint32_t key_max[LH_MAX_KEYS];
  uint32_t tail_mask;
};

// One pass over the columns, four rows in flight per thread; each lane takes
// row i - 1 from the lane below.  A wave that has seen every order broken
// compares no more.  Each block writes its result (atomics of every block on
// one address would serialize); k_input_total combines them.
template <bool TAIL>
__global__ __launch_bounds__(256) void k_input_stats(LevelCols c, uint64_t n, uint32_t all, InputStats* part) {
  constexpr int R = 4;
  __shared__ InputStats s_st[256 / WAVE];
  const int K = (int)c.n_levels, lane = lane_id();
  uint32_t mx[LH_MAX_KEYS], known = all;
#pragma unroll
  for (int l = 0; l < LH_MAX_KEYS; l++) mx[l] = 0;
  const uint64_t stride = (uint64_t)gridDim.x * 256 * R;
  for (uint64_t i0 = (uint64_t)blockIdx.x * 256 * R; i0 < n; i0 += stride) {
    const bool check = TAIL && __any(known != 0);
    uint32_t m[R];
    bool ord[R];
#pragma unroll
    for (int j = 0; j < R; j++) {
      m[j] = all;
      ord[j] = true;  // order of the suffix from level l on
    }
    // constant level indices: the column pointers stay in registers
#pragma unroll
    for (int l = LH_MAX_KEYS - 1; l >= 0; l--) {
      if (l >= K) continue;
      uint32_t b[R];
#pragma unroll
      for (int j = 0; j < R; j++) {
        const uint64_t i = i0 + (uint64_t)j * 256 + threadIdx.x;
        b[j] = i < n ? c.k[l][i] : 0u;
        mx[l] = max(mx[l], b[j]);
      }
      if (!check) continue;
#pragma unroll
      for (int j = 0; j < R; j++) {
        const uint64_t i = i0 + (uint64_t)j * 256 + threadIdx.x;
        uint32_t a = (uint32_t)__shfl_up((int)b[j], 1, 64);
        if (lane == 0 && i > 0 && i < n) a = c.k[l][i - 1];
        if (i == 0 || i >= n) continue;
        ord[j] = a < b[j] || (a == b[j] && ord[j]);
        if (!ord[j]) m[j] &= ~(1u << (K - 1 - l));
      }
    }
#pragma unroll
    for (int j = 0; j < R; j++) known &= m[j];
  }
#pragma unroll
  for (int l = 0; l < LH_MAX_KEYS; l++) {
    if (l >= K) continue;
    for (int o = 32; o > 0; o >>= 1) mx[l] = max(mx[l], (uint32_t)__shfl_xor((int)mx[l], o, 64));
    if (lane == 0) s_st[threadIdx.x / WAVE].key_max[l] = mx[l];
  }
  for (int o = 32; o > 0; o >>= 1) known &= (uint32_t)__shfl_xor((int)known, o, 64);
  if (lane == 0) s_st[threadIdx.x / WAVE].tail_mask = known;
  __syncthreads();
  if ((int)threadIdx.x < K) {
    uint32_t v = 0;
    for (int w = 0; w < 256 / WAVE; w++) v = max(v, s_st[w].key_max[threadIdx.x]);
    part[blockIdx.x].key_max[threadIdx.x] = v;
  }
  if (threadIdx.x == 0) {
    uint32_t v = all;
    for (int w = 0; w < 256 / WAVE; w++) v &= s_st[w].tail_mask;
    part[blockIdx.x].tail_mask = v;
  }
}

// The blocks' results combined by one block: thread group l takes level l.
__global__ __launch_bounds__(576) void k_input_total(const InputStats* part, uint32_t nb, uint32_t n_levels,
                                                     uint32_t all, InputStats* out) {
  const uint32_t l = threadIdx.x / WAVE;  // wave 8: the mask
  if (l < LH_MAX_KEYS) {
    uint32_t v = 0;
    for (uint32_t b = lane_id(); l < n_levels && b < nb; b += WAVE) v = max(v, part[b].key_max[l]);
    for (int o = 32; o > 0; o >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, o, 64));
    if (lane_id() == 0) out->key_max[l] = v;
  } else {
    uint32_t v = all;
    for (uint32_t b = lane_id(); b < nb; b += WAVE) v &= part[b].tail_mask;
    for (int o = 32; o > 0; o >>= 1) v &= (uint32_t)__shfl_xor((int)v, o, 64);
    if (lane_id() == 0) out->tail_mask = v;
  }
}

// ---- layouts ---------------------------------------------------------------

struct SetRange {
  const uint32_t* offs;  // parent offsets (null for level 0)
  uint64_t root_n;       // level-0 size
};

__device__ __forceinline__ void set_range(const SetRange& sr, uint64_t s, uint32_t& b, uint32_t& e) {
  if (!sr.offs) { b = 0; e = (uint32_t)sr.root_n; }
  else { b = sr.offs[s]; e = sr.offs[s + 1]; }
}

// All levels' sets, numbered one level after another.
struct LayoutSets {
  SetRange sr[LH_MAX_KEYS];
  const uint32_t* keys[LH_MAX_KEYS];
  const uint8_t* choice[LH_MAX_KEYS];  // learned choices, or null
  uint64_t first[LH_MAX_KEYS + 1];     // number of each level's first set
  uint64_t* bs_word[LH_MAX_KEYS];
  uint32_t* bs_base[LH_MAX_KEYS];
  uint32_t n_levels;
};

// Set i of all: its level's entry of an array indexed by level.
#define LH_LEVEL_OF(sets, i, l)                       \
  uint32_t l = 0;                                     \
  _Pragma("unroll") for (uint32_t q = 1; q < LH_MAX_KEYS; q++) \
    if (q < (sets).n_levels && (i) >= (sets).first[q]) l = q

// Words of each set's bitset (0: a sorted array).
__global__ void k_layout_words(LayoutSets ls, uint64_t total, uint32_t mode, uint32_t* words) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (uint64_t)gridDim.x * blockDim.x) {
    LH_LEVEL_OF(ls, i, l);
    const uint64_t s = i - ls.first[l];
    const uint32_t* keys = ls.keys[l];
    uint32_t b, e;
    set_range(ls.sr[l], s, b, e);
    uint32_t nw = 0;
    if (e > b) {
      uint32_t lo = keys[b], hi = keys[e - 1];
      uint64_t card = e - b;
      uint64_t span = (uint64_t)hi - lo + 1;
      bool bs = false;
      // plain rule: a bitset when the set fills at least 1/32 of its window
      if (mode == LH_LAYOUT_PLAIN || mode == LH_LAYOUT_LEARNED) bs = span <= 32ull * card;
      else if (mode == LH_LAYOUT_BITSET) bs = span <= 4096ull * card;
      if (ls.choice[l] && ls.choice[l][s]) bs = ls.choice[l][s] == 2;
      if (bs) nw = ((hi - (lo & ~63u)) >> 6) + 1;
    }
    words[i] = nw;
  }
}

// Null words: every set a sorted array.
__global__ void k_layout_desc(LayoutSets ls, uint64_t total, const uint32_t* words, const uint64_t* woff) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (uint64_t)gridDim.x * blockDim.x) {
    LH_LEVEL_OF(ls, i, l);
    const uint64_t s = i - ls.first[l];
    uint32_t b, e;
    set_range(ls.sr[l], s, b, e);
    const bool bs = words && words[i] != 0;
    ls.bs_word[l][s] = bs ? woff[i] - woff[ls.first[l]] : UINT64_MAX;
    ls.bs_base[l][s] = (e > b) ? (ls.keys[l][b] & ~63u) : 0u;
  }
}

// Bitset words before each level's first, and all of them.
__global__ void k_layout_totals(LayoutSets ls, const uint64_t* woff, uint64_t* out) {
  const uint32_t l = threadIdx.x;
  if (l <= ls.n_levels) out[l] = woff[ls.first[l]];
}

// Bitset words from the keys.  A wave takes 64 consecutive keys; the keys
// of one (set, word) pair are consecutive (keys are sorted within a set, and
// sets follow each other), so the pairs are runs of lanes, marked by a
// ballot.  When some run holds more than one key, an OR over each lane's
// rest of its run (doubling steps, bounded by the run's end) gathers each
// word's bits in the run's first lane, which writes the word.  A run that
// goes on in the neighbouring wave (its first or last key's neighbour there
// is in the same word) ORs its part atomically into the word (the pool
// starts zeroed); words without keys stay zero.  Waves without a bitset key do no
// lane exchange at all.  Null bs_word: the keys form one set whose window
// starts at 0 at word 0 (the root index).  rank (null: not wanted) gets, for
// every word with a key, the position of its first key in the level: a
// position inside a bitset is then one load and a popcount, and nothing has
// to be counted or scanned for it.
__global__ __launch_bounds__(256) void k_layout_fill(const uint32_t* keys, const uint32_t* parent, uint64_t n,
                                                     const uint64_t* bs_word, const uint32_t* bs_base, uint64_t* pool,
                                                     uint32_t* rank) {
  const int lane = threadIdx.x & 63;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t j0 = (uint64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~63u); j0 < n; j0 += stride) {
    const uint64_t j = j0 + lane;
    uint64_t tag = ~0ull, bits = 0, w = 0;  // tag: set << 32 | word (words < 2^26), ~0 for no key
    if (j < n) {
      const uint32_t st = parent ? parent[j] : 0u;
      const uint64_t w0 = bs_word ? bs_word[st] : 0u;
      if (w0 != UINT64_MAX) {
        const uint32_t d = keys[j] - (bs_word ? bs_base[st] : 0u);
        tag = ((uint64_t)st << 32) | (d >> 6);
        bits = 1ull << (d & 63u);
        w = w0 + (d >> 6);
      }
    }
    const bool live = tag != ~0ull;
    const uint64_t L = ballot(live);
    if (!L) continue;  // uniform: no bitset key in the wave
    const uint64_t prev = __shfl_up(tag, 1, WAVE);
    const bool head = live && (lane == 0 || prev != tag);
    // runs start at heads; lanes without a key are runs of their own
    const uint64_t S = ballot(head) | ~L;
    const uint64_t above = lane < WAVE - 1 ? S >> (lane + 1) : 0ull;
    const uint32_t end = above ? (uint32_t)lane + 1u + (uint32_t)__builtin_ctzll(above) : (uint32_t)WAVE;
    if (L & ~S) {  // uniform: some run holds two keys or more
#pragma unroll
      for (int o = 1; o < WAVE; o <<= 1) {
        const uint64_t ob = __shfl_down(bits, o, WAVE);
        if ((uint32_t)lane + (uint32_t)o < end) bits |= ob;
      }
    }
    if (head) {
      // does the run go on in the wave before (lane 0) or after (a run
      // reaching the last lane)?  The neighbouring key shares the word when
      // it has the same set and the same offset >> 6.
      const uint32_t st = (uint32_t)(tag >> 32), word = (uint32_t)tag;
      const uint32_t base = bs_word ? bs_base[st] : 0u;
      bool shared = false;
      if (lane == 0 && j > 0)
        shared = (parent ? parent[j - 1] : 0u) == st && ((keys[j - 1] - base) >> 6) == word;
      if (rank && !shared) rank[w] = (uint32_t)j;
      if (end == (uint32_t)WAVE && j0 + WAVE < n)
        shared = shared || ((parent ? parent[j0 + WAVE] : 0u) == st && ((keys[j0 + WAVE] - base) >> 6) == word);
      if (shared) atomicOr((unsigned long long*)&pool[w], (unsigned long long)bits);
      else pool[w] = bits;
    }
  }
}

// The longest of n runs given by their offsets, into *out (cleared before).
__global__ __launch_bounds__(256) void k_max_run(const uint32_t* offs, uint64_t n, uint32_t* out) {
  uint32_t m = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256)
    m = max(m, offs[i + 1] - offs[i]);
  for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
  if ((threadIdx.x & 63) == 0 && m > 1) atomicMax(out, m);
}

unsigned grid_for(uint64_t n) {
  uint64_t b = (n + 255) / 256;
  return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(b, 256 * 64));
}

uint32_t bitlen(uint32_t v) { return v ? 32 - __builtin_clz(v) : 0; }

}  // namespace

__global__ void k_count_bitsets(const uint64_t* bs_word, uint64_t n, unsigned long long* out) {
  uint32_t c = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    c += bs_word[i] != UINT64_MAX;
  for (int o = 32; o > 0; o >>= 1) c += (uint32_t)__shfl_xor((int)c, o, 64);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(out, (unsigned long long)c);
}

uint64_t count_bitsets(const lh_trie* t, uint32_t l, hipStream_t s) {
  const Level& L = t->lv[l];
  if (!L.n_sets || !L.pool_words) return 0;
  DBuf<unsigned long long> c(1, s);
  LH_HIP(hipMemsetAsync(c.p, 0, sizeof(unsigned long long), s));
  k_count_bitsets<<<std::min<unsigned>(grid_for(L.n_sets), 1024), 256, 0, s>>>(L.bs_word.p, L.n_sets, c.p);
  LH_HIP(hipGetLastError());
  return read_scalar(c.p, s);
}

// Per-set layouts of every level, their bitsets and the root index: sized
// together (one round trip), cleared together, filled level by level.
static void build_layouts(lh_trie* t, uint32_t mode, const std::vector<DBuf<uint32_t>>& parent, hipStream_t s) {
  const uint32_t nl = t->n_levels;
  LayoutSets ls{};
  ls.n_levels = nl;
  std::vector<DBuf<uint8_t>> choice(nl);
  bool any = false;
  for (uint32_t l = 0; l < nl; l++) {
    Level& L = t->lv[l];
    L.n_sets = (l == 0) ? 1 : t->lv[l - 1].n;
    L.bs_word.alloc(L.n_sets, s);
    L.bs_base.alloc(L.n_sets, s);
    ls.sr[l] = SetRange{l == 0 ? nullptr : t->lv[l - 1].offs.p, t->lv[0].n};
    ls.keys[l] = L.keys.p;
    ls.bs_word[l] = L.bs_word.p;
    ls.bs_base[l] = L.bs_base.p;
    ls.first[l + 1] = ls.first[l] + L.n_sets;
    if (mode == LH_LAYOUT_LEARNED && L.n_sets && learned_layout_choices(t, l, s, choice[l])) ls.choice[l] = choice[l].p;
  }
  const uint64_t total = ls.first[nl];
  uint64_t base[LH_MAX_KEYS + 1] = {};
  DBuf<uint32_t> words;
  DBuf<uint64_t> woff;
  if (mode != LH_LAYOUT_UINT && total) {
    words.alloc(total, s);
    woff.alloc(total + 1, s);
    k_layout_words<<<grid_for(total), 256, 0, s>>>(ls, total, mode, words.p);
    LH_HIP(hipGetLastError());
    scan_u32_to_u64_dev(words.p, woff.p, total, s);
    struct Bounds {
      uint64_t v[LH_MAX_KEYS + 1];
    };
    HostOut<Bounds> out(s);
    k_layout_totals<<<1, WAVE, 0, s>>>(ls, woff.p, out.p()->v);
    LH_HIP(hipGetLastError());
    const Bounds h = out.get();
    for (uint32_t l = 0; l <= nl; l++) base[l] = h.v[l];
  }
  if (total) {
    k_layout_desc<<<grid_for(total), 256, 0, s>>>(ls, total, base[nl] ? words.p : nullptr, woff.p);
    LH_HIP(hipGetLastError());
  }
  // root index, when level 0 holds at least one key per 64 of its span
  const uint64_t n0 = t->lv[0].n;
  const uint64_t span = (uint64_t)t->key_max[0] + 1;
  const uint64_t root_words = n0 && span <= 64 * n0 && span <= (1ull << 32) ? (span + 63) / 64 : 0;
  const uint64_t all = base[nl] + root_words;
  if (!all) return;
  t->words.alloc(all, s);
  ProfScope ps("layout_fill", s, total, all);
  LH_HIP(hipMemsetAsync(t->words.p, 0, all * sizeof(uint64_t), s));
  // positions inside bitset sets are needed when a deeper level hangs below or
  // the rows of a bag are reached through them: a set's last level has no ranks
  const uint64_t ranked = base[(t->flags & LH_BAG) ? nl : nl - 1];
  t->ranks.alloc(ranked + root_words, s);
  for (uint32_t l = 0; l < nl; l++) {
    Level& L = t->lv[l];
    L.pool_words = base[l + 1] - base[l];
    if (!L.pool_words) continue;
    L.pool.p = t->words.p + base[l];
    if (l + 1 < nl || (t->flags & LH_BAG)) L.bs_rank.p = t->ranks.p + base[l];
    k_layout_fill<<<grid_for(L.n), 256, 0, s>>>(L.keys.p, l ? parent[l].p : nullptr, L.n, L.bs_word.p, L.bs_base.p,
                                                L.pool.p, L.bs_rank.p);
    LH_HIP(hipGetLastError());
  }
  if (root_words) {
    t->root_span = span;
    t->root_bits.p = t->words.p + base[nl];
    t->root_rank.p = t->ranks.p + ranked;
    k_layout_fill<<<grid_for(n0), 256, 0, s>>>(t->lv[0].keys.p, nullptr, n0, nullptr, nullptr, t->root_bits.p,
                                               t->root_rank.p);
    LH_HIP(hipGetLastError());
  }
}

namespace {

struct LevelOffs {
  const uint32_t* offs[LH_MAX_KEYS];  // child offsets of levels 0 .. n_levels-2
  const uint32_t* run;                // bag: run offsets of the last level
  uint32_t n_levels;
};

// Rows under each level-0 node: its child range composed down to the last
// level (and through the runs of a bag trie).
__global__ void k_level0_rows(LevelOffs lo, uint64_t n0, uint32_t* rows) {
  for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n0; p += (uint64_t)gridDim.x * blockDim.x) {
    uint32_t b = (uint32_t)p, e = (uint32_t)p + 1;
    for (uint32_t l = 0; l + 1 < lo.n_levels; l++) {
      b = lo.offs[l][b];
      e = lo.offs[l][e];
    }
    if (lo.run) {
      b = lo.run[b];
      e = lo.run[e];
    }
    rows[p] = e - b;
  }
}

}  // namespace

void ensure_column_stats(lh_trie* t, hipStream_t s) {
  if (t->col_stats) return;
  // the first column: its values are the level-0 keys, each shared by the
  // rows under its node
  if (t->n_levels && t->lv[0].n) {
    LevelOffs lo{};
    lo.n_levels = t->n_levels;
    for (uint32_t l = 0; l + 1 < t->n_levels; l++) lo.offs[l] = t->lv[l].offs.p;
    lo.run = (t->flags & LH_BAG) ? t->lv[t->n_levels - 1].offs.p : nullptr;
    DBuf<uint32_t> rows(t->lv[0].n, s);
    k_level0_rows<<<grid_for(t->lv[0].n), 256, 0, s>>>(lo, t->lv[0].n, rows.p);
    LH_HIP(hipGetLastError());
    t->col_distinct[0] = t->lv[0].n;
    t->col_freq_max[0] = reduce_max_u32(rows.p, t->lv[0].n, s);
  } else if (t->n_levels) {
    t->col_distinct[0] = 0;
    t->col_freq_max[0] = 0;
  }
  // A two-level trie without row columns: sort its rows by (level 1,
  // level 0) (level 0 is in order already, so only level 1's bits are
  // sorted) and keep them; the statistics come from the sorted runs and a
  // copy of the trie in the swapped level order takes the rows unsorted.
  if (t->n_levels == 2 && t->annos.empty() && t->meta.empty() && t->key_bits[0] + t->key_bits[1] <= 64 &&
      t->n_rows) {
    const uint32_t* cols[2] = {row_keys(t, 1), row_keys(t, 0)};
    const uint32_t bits[2] = {t->key_bits[1], t->key_bits[0]};
    t->tsorted[0].alloc(t->n_rows, s);
    t->tsorted[1].alloc(t->n_rows, s);
    uint32_t* out[2] = {t->tsorted[0].p, t->tsorted[1].p};
    sort_packed(cols, bits, 2, t->n_rows, SortValue{}, out, s, 1);
    sorted_run_stats(t->tsorted[0].p, t->n_rows, t->col_distinct[1], t->col_freq_max[1], s);
    t->col_stats = true;
    return;
  }
  for (uint32_t l = 1; l < t->n_levels; l++) {
    if (t->key_max[l] < (1u << 28)) {
      column_freq(row_keys(t, l), t->n_rows, t->key_max[l], t->col_distinct[l], t->col_freq_max[l], s);
    } else {
      t->col_distinct[l] = t->n_rows;
      t->col_freq_max[l] = 1;
    }
  }
  t->col_stats = true;
}

// The most trailing levels whose order a presorted-tail mask shows (0: not
// even the last level's).
static uint32_t tail_of_mask(uint32_t mask, uint32_t n_keys) {
  for (uint32_t t = n_keys; t >= 1; t--)
    if (mask >> (t - 1) & 1u) return t;
  return 0;
}

namespace {
constexpr uint32_t BUILD_ANNOS = 8;  // annotation columns whose statistics come with the rest
struct BuildOut {
  AnnoAcc anno[BUILD_ANNOS];
  uint32_t max_run;
};
}  // namespace

lh_trie* build_trie(uint64_t n_rows, uint32_t n_keys, const uint32_t* const* keys, uint32_t n_annos,
                    const double* const* annos, uint32_t n_meta, const uint32_t* const* meta,
                    const uint32_t* level_order, uint32_t flags, const uint32_t* sel, uint64_t n_sel,
                    hipStream_t s, uint32_t sorted_tail, bool detect_sorted) {
  const uint64_t n = sel ? n_sel : n_rows;
  sorted_tail = std::min(sorted_tail, n_keys);
  if (n >= (1ull << 32) - 1) fail(LH_ERR_OVERFLOW, "trie build: 2^32 - 1 rows or more");
  const bool bag = (flags & LH_BAG) != 0;
  std::unique_ptr<lh_trie> t(new lh_trie());
  t->magic = TRIE_MAGIC;
  t->n_levels = n_keys;
  t->flags = flags;
  t->n_input = n;
  for (uint32_t l = 0; l < n_keys; l++) t->level_order[l] = level_order ? level_order[l] : l;

  // Input columns in level order (compacted through `sel` if given).
  std::vector<DBuf<uint32_t>> selcols;
  const uint32_t* col[LH_MAX_KEYS];
  for (uint32_t l = 0; l < n_keys; l++) {
    const uint32_t* src = keys[t->level_order[l]];
    if (sel) {
      selcols.emplace_back(n, s);
      gather_u32(src, sel, selcols.back().p, n, s);
      src = selcols.back().p;
    }
    col[l] = src;
  }
  // every level's largest key and, when asked, the presorted tail: one pass
  // over the columns, one read back
  if (n) {
    LevelCols c{};
    c.n_levels = n_keys;
    for (uint32_t l = 0; l < n_keys; l++) c.k[l] = col[l];
    const bool detect = detect_sorted && sorted_tail == 0 && n > 1;
    const uint32_t all = (1u << n_keys) - 1;
    const unsigned nb = std::min(grid_for((n + 3) / 4), 2048u);
    DBuf<InputStats> part(nb, s);
    HostOut<InputStats> out(s);
    {
      ProfScope ps("trie_input", s, n, 0);
      if (detect) k_input_stats<true><<<nb, 256, 0, s>>>(c, n, all, part.p);
      else k_input_stats<false><<<nb, 256, 0, s>>>(c, n, all, part.p);
    }
    LH_HIP(hipGetLastError());
    k_input_total<<<1, (LH_MAX_KEYS + 1) * WAVE, 0, s>>>(part.p, nb, n_keys, all, out.p());
    LH_HIP(hipGetLastError());
    const InputStats h = out.get();
    for (uint32_t l = 0; l < n_keys; l++) {
      t->key_max[l] = h.key_max[l];
      t->key_bits[l] = bitlen(t->key_max[l]);
    }
    if (detect) sorted_tail = tail_of_mask(h.tail_mask, n_keys);
  } else {
    for (uint32_t l = 0; l < n_keys; l++) t->key_max[l] = t->key_bits[l] = 0;
  }

  // Keys of up to 96 bits are sorted packed and unpacked into the sorted
  // columns (no gathers); wider keys take the multi-pass sort by
  // permutation.  A bag's only annotation or meta column travels through the
  // packed sort's passes itself: four more bytes per row and pass than the
  // permutation, against a gather that reads a 64-byte line per row (47 M
  // rows after one pass: 0.82 ms).  More columns are gathered by the
  // permutation.
  uint32_t tot_bits = 0;
  for (uint32_t l = 0; l < n_keys; l++) tot_bits += t->key_bits[l];
  const bool carry = bag && n_annos + n_meta == 1 && sorted_tail < n_keys && tot_bits <= 96;
  const bool need_perm = (n_annos || n_meta) && !carry;
  DBuf<uint32_t> perm(need_perm ? n : 0, s);
  SortValue val;
  DBuf<double> carry_anno, sel_anno;
  DBuf<uint32_t> carry_meta, sel_meta;
  if (carry && n_annos) {
    carry_anno.alloc(n, s);
    if (sel) {
      sel_anno.alloc(n, s);
      gather_f64(annos[0], sel, sel_anno.p, n, s);
    }
    val = SortValue{sel ? sel_anno.p : annos[0], carry_anno.p, 8};
  } else if (carry) {
    carry_meta.alloc(n, s);
    if (sel) {
      sel_meta.alloc(n, s);
      gather_u32(meta[0], sel, sel_meta.p, n, s);
    }
    val = SortValue{sel ? sel_meta.p : meta[0], carry_meta.p, 4};
  } else if (need_perm) {
    val = SortValue{nullptr, perm.p, 4};
  }
  LevelCols lc{};
  lc.n_levels = n_keys;
  std::vector<DBuf<uint32_t>> sorted;
  uint32_t* sorted_p[LH_MAX_KEYS];
  // rows already in order: a set trie reads the input columns as they are;
  // other tries copy them (a bag keeps its sorted columns) with the
  // identity permutation
  const bool in_order = sorted_tail >= n_keys && !need_perm && !bag && !sel;
  const bool copy_order = sorted_tail >= n_keys && !in_order;
  for (uint32_t l = 0; l < n_keys; l++) {
    if (in_order) {
      sorted.emplace_back();
      sorted_p[l] = nullptr;
      lc.k[l] = col[l];
    } else {
      sorted.emplace_back(n, s);
      sorted_p[l] = sorted.back().p;
      lc.k[l] = sorted.back().p;
    }
  }
  if (in_order) {
    // nothing to sort
  } else if (copy_order) {
    for (uint32_t l = 0; l < n_keys && n; l++)
      LH_HIP(hipMemcpyAsync(sorted_p[l], col[l], n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
    if (need_perm && (sel || !bag)) iota_u32(perm.p, n, s);  // else the rows are copied as they are (below)
  } else if (!sort_packed(col, t->key_bits, n_keys, n, val, sorted_p, s, sorted_tail)) {
    if (!need_perm) perm.alloc(n, s);
    // a stable sort by the leading levels keeps the presorted tail's order
    lex_sort_perm(col, t->key_bits, n_keys - sorted_tail, n, perm.p, s);
    for (uint32_t l = 0; l < n_keys; l++) gather_u32(col[l], perm.p, sorted_p[l], n, s);
  }

  uint32_t ntiles = (uint32_t)((n + TB_NT - 1) / TB_NT);
  uint64_t cn = (uint64_t)ntiles * n_keys;
  DBuf<uint32_t> counts(cn ? cn : 1, s), toff(cn + 1, s);
  if (n) {
    ProfScope ps("trie_head_counts", s, n, 0);
    k_head_counts<<<ntiles, TB_NT, 0, s>>>(lc, n, counts.p, ntiles);
    LH_HIP(hipGetLastError());
  }
  // one scan over all levels' tile counts (modulo 2^32: a level's offsets
  // are differences from its first tile's)
  EmitArgs ea{};
  std::vector<uint64_t> level_n(n_keys, 0);
  if (n) {
    scan_u32_dev(counts.p, toff.p, cn, s);
    struct LevelTotals {
      uint32_t v[LH_MAX_KEYS];
    };
    HostOut<LevelTotals> out(s);
    k_level_totals<<<1, WAVE, 0, s>>>(toff.p, ntiles, n_keys, out.p()->v);
    LH_HIP(hipGetLastError());
    const LevelTotals h = out.get();
    uint32_t at = 0;
    for (uint32_t l = 0; l < n_keys; l++) {
      level_n[l] = h.v[l];
      ea.level_n[l] = h.v[l];
      ea.level_base[l] = at;
      at += h.v[l];
    }
  }
  ea.c = lc;
  ea.tile_off = toff.p;
  ea.ntiles = ntiles;
  for (uint32_t l = 0; l < n_keys; l++) {
    Level& L = t->lv[l];
    L.n = level_n[l];
    L.keys.alloc(L.n, s);
    ea.keys_out[l] = L.keys.p;
    L.samp.alloc((L.n + (1u << LINE_SHIFT) - 1) >> LINE_SHIFT, s);
    ea.samp_out[l] = L.samp.p;
    if (l + 1 < n_keys) {
      L.offs.alloc(L.n + 1, s);
      ea.offs_out[l] = L.offs.p;
    }
  }
  const uint64_t n_leaf = n_keys ? level_n[n_keys - 1] : 0;
  DBuf<uint32_t> kept;
  if (bag) {
    t->lv[n_keys - 1].offs.alloc(n_leaf + 1, s);
    ea.run_out = t->lv[n_keys - 1].offs.p;
  } else {
    // a set keeps the leaf heads' rows: their keys are written as the
    // heads are found (the row positions only when columns follow them);
    // their last keys are the last level's keys
    for (uint32_t l = 0; l + 1 < n_keys; l++) {
      t->skeys[l].alloc(n_leaf, s);
      ea.rowkeys_out[l] = t->skeys[l].p;
    }
    if (need_perm) {
      kept.alloc(n_leaf, s);
      ea.kept_out = kept.p;
    }
  }
  // parents of each level's nodes, for the bitset fill of levels below 0
  std::vector<DBuf<uint32_t>> parent(n_keys);
  for (uint32_t l = 1; l < n_keys; l++) {
    parent[l].alloc(level_n[l], s);
    ea.parent_out[l] = parent[l].p;
  }
  if (n) {
    ProfScope ps("trie_emit_levels", s, n, 0);
    k_emit_levels<<<ntiles, TB_NT, 0, s>>>(ea, n);
    LH_HIP(hipGetLastError());
  }
  if (!n) {  // closing offsets of an empty trie
    for (uint32_t l = 0; l + 1 < n_keys; l++) fill_u32(t->lv[l].offs.p, 0, 1, s);
    if (bag) fill_u32(t->lv[n_keys - 1].offs.p, 0, 1, s);
  }
  // what the host reads when everything is queued: the longest run, where
  // some key tuple repeats, and the annotations' statistics
  const bool runs = bag && n_leaf < n;
  DBuf<BuildOut> bout(runs || n_annos ? 1 : 0, s);
  if (bout.p) LH_HIP(hipMemsetAsync(bout.p, 0, sizeof(BuildOut), s));
  if (runs) {
    k_max_run<<<std::min(grid_for(n_leaf), 1024u), 256, 0, s>>>(t->lv[n_keys - 1].offs.p, n_leaf, &bout.p->max_run);
    LH_HIP(hipGetLastError());
  }

  // Rows in trie order: bag keeps every sorted row, set keeps leaf heads.
  // Their keys are the sorted columns themselves (bag), or the sorted
  // columns at the leaf heads, written by the level emission (set).
  t->n_rows = bag ? n : n_leaf;
  const uint32_t* rowsel = perm.p;  // sorted position -> input row
  DBuf<uint32_t> keptrows;
  if (!bag && need_perm) {  // (a set relation carries neither; kept for safety)
    keptrows.alloc(n_leaf, s);
    gather_u32(perm.p, kept.p, keptrows.p, n_leaf, s);
    rowsel = keptrows.p;
  }
  if (bag)
    for (uint32_t l = 0; l < n_keys; l++) t->skeys[l] = std::move(sorted[l]);
  // annotation / meta columns (bag relations only); `sel` maps rows first
  DBuf<uint32_t> srcrow;
  const uint32_t* rowmap = rowsel;
  if (sel && need_perm) {
    srcrow.alloc(t->n_rows, s);
    gather_u32(sel, rowsel, srcrow.p, t->n_rows, s);
    rowmap = srcrow.p;
  }
  // a presorted bag keeps its input rows in order: plain copies
  const bool same_rows = copy_order && bag && !sel;
  std::vector<AnnoStats> late;
  for (uint32_t a = 0; a < n_annos; a++) {
    if (carry) t->annos.push_back(std::move(carry_anno));
    else t->annos.emplace_back(t->n_rows, s);
    if (carry) {
      // sorted with the keys
    } else if (same_rows) {
      if (t->n_rows)
        LH_HIP(hipMemcpyAsync(t->annos.back().p, annos[a], t->n_rows * sizeof(double), hipMemcpyDeviceToDevice, s));
    } else {
      gather_f64(annos[a], rowmap, t->annos.back().p, t->n_rows, s);
    }
    if (a < BUILD_ANNOS) anno_stats_into(t->annos.back().p, t->n_rows, &bout.p->anno[a], s);
    else late.push_back(anno_stats(t->annos.back().p, t->n_rows, s));
  }
  for (uint32_t m = 0; m < n_meta; m++) {
    if (carry) t->meta.push_back(std::move(carry_meta));
    else t->meta.emplace_back(t->n_rows, s);
    if (carry) {
      // sorted with the keys
    } else if (same_rows) {
      if (t->n_rows)
        LH_HIP(hipMemcpyAsync(t->meta.back().p, meta[m], t->n_rows * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
    } else {
      gather_u32(meta[m], rowmap, t->meta.back().p, t->n_rows, s);
    }
  }

  build_layouts(t.get(), flags & LH_LAYOUT_MASK, parent, s);
  if (bout.p) {
    const BuildOut h = read_scalar(bout.p, s);
    if (runs) t->max_run = h.max_run;
    t->astats.clear();
    for (uint32_t a = 0; a < std::min(n_annos, BUILD_ANNOS); a++) t->astats.push_back(decode_anno_stats(h.anno[a]));
    for (const AnnoStats& st : late) t->astats.push_back(st);
  }
  LH_HIP(hipStreamSynchronize(s));
  return t.release();
}

}  // namespace lh
