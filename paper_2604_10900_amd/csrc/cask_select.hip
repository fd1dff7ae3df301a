// Selection: stage-1 prefix eviction (Section 2.2 of the paper) and the stage-2 split of the
// decode trace into protected core, representative seeds and donor scratch (Section 2.1).
//
// "Top k" is exact and order-defined: higher float score first, equal scores by ascending
// cache index.  One workgroup per unit finds the k-th keys of the three ranks a unit needs (prefix
// keep, core, core + seeds) over an order-preserving key image of the scores (rank_select), then
// marks the elements; when the k-th value is shared by more elements than there are places left, an
// ordered block scan hands the places to the lowest indices -- no atomics decide membership.
//
// The ordered walk gives every kept row its output slot (ascending source order, representatives at
// their seed's position: |R| <= B with C subset of R, Section 2.3) and every seed its ordinal: from
// the keys still in registers where the unit fits them, else from the roles in memory.
#include <type_traits>

#include "cask_common.h"

namespace cask {

namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

struct Kth {
  uint32_t key;   // key of the k-th element in the order
  int take_eq;    // how many elements equal to `key` belong to the top k
  int total_eq;   // how many elements equal to `key` exist in the range
};

// The number of keys a thread holds is the template parameter PER of the selection.  A wave owns
// 64 PER consecutive rows, touched 64 at a time (coalesced): the layout of the ordered walk, so that
// a unit of at most 1024 PER rows reads its scores once and goes from keys to slots in registers.
// The straight-line code over a thread's keys costs what PER says whatever the unit's length, so the
// launcher takes the smallest instance that covers the longest unit; units beyond the largest take
// kSelMany keys at a time (MANY) and read them again in every step.
constexpr int kSelMost = 36;  // (the keys, nothing else, live across the steps: 36 of the 128 registers)
constexpr int kSelMany = 16;

constexpr int kBins = 2048;
constexpr int kCand = 64;  // candidates of a boundary bin that one wave ranks
constexpr int kCrowd = 1024;
struct SelectLds {
  int hist[3][2 * kBins];  // two copies of a bin side by side: scores crowd, and equal addresses serialise
  uint32_t cand[3][kCand];
  int n_cand[3];
  uint32_t wave_tot[3][kSelWaves];
  uint32_t wave_lo[kSelWaves], wave_hi[kSelWaves];
  uint32_t bin_lo[3], bin_hi[3];  // of a crowded bin: its smallest and largest key
  int found[3][4];
};

// Rank queries answered together: query 0 asks for the key of rank k[0] among rows [0, P), queries 1
// and 2 for ranks k[1], k[2] among [P, hi).  1 <= k <= rows of the range; k <= 0: not asked.
struct RankQuery {
  int P, hi, k[3];
};

template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp(int old, int x) {
  return __builtin_amdgcn_update_dpp(old, x, CTRL, ROWS, 0xF, false);
}
// inclusive sum over the lanes of a wave
__device__ __forceinline__ int wave_scan(int v) {
  v += dpp<0x111, 0xF>(0, v);  // row_shr 1, 2, 4, 8
  v += dpp<0x112, 0xF>(0, v);
  v += dpp<0x114, 0xF>(0, v);
  v += dpp<0x118, 0xF>(0, v);
  v += dpp<0x142, 0xA>(0, v);  // last lane of a row of 16 to the next row
  v += dpp<0x143, 0xC>(0, v);  // lane 31 to the upper half
  return v;
}
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t x, Op op) {  // op(x, x) == x
  int v = (int)x;
  v = (int)op((uint32_t)v, (uint32_t)dpp<0x111, 0xF>(v, v));
  v = (int)op((uint32_t)v, (uint32_t)dpp<0x112, 0xF>(v, v));
  v = (int)op((uint32_t)v, (uint32_t)dpp<0x114, 0xF>(v, v));
  v = (int)op((uint32_t)v, (uint32_t)dpp<0x118, 0xF>(v, v));
  v = (int)op((uint32_t)v, (uint32_t)dpp<0x142, 0xA>(v, v));
  v = (int)op((uint32_t)v, (uint32_t)dpp<0x143, 0xC>(v, v));
  return (uint32_t)__builtin_amdgcn_readlane(v, 63);
}
// sum of w[0 .. wave) of sixteen per-wave totals, the same in every lane of the wave; *total: of all
// (unsigned: the totals may be two 16-bit counts in a word)
__device__ __forceinline__ uint32_t before_wave(const uint32_t* w, int wave, uint32_t* total) {
  const int lane = threadIdx.x & 63;
  uint32_t v = lane < kSelWaves ? w[lane] : 0u;
  v += (uint32_t)dpp<0x111, 0xF>(0, (int)v);
  v += (uint32_t)dpp<0x112, 0xF>(0, (int)v);
  v += (uint32_t)dpp<0x114, 0xF>(0, (int)v);
  v += (uint32_t)dpp<0x118, 0xF>(0, (int)v);
  *total = (uint32_t)__builtin_amdgcn_readlane((int)v, kSelWaves - 1);
  return wave > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)v, wave - 1) : 0u;
}

// keys of rows base + 64 PER wave + 64 e + lane, e < PER, rows outside [lo, hi) taken from its ends
// (they are not counted anywhere, but stay out of the way of the smallest and largest key); all
// loads are in flight together
template <int PER>
__device__ __forceinline__ void load_keys(const float* __restrict__ s, int i0, int lo, int hi, uint32_t (&key)[PER]) {
  float v[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) v[e] = s[min(max(i0 + e * 64, lo), hi - 1)];
#pragma unroll
  for (int e = 0; e < PER; ++e) key[e] = score_key(v[e]);
}

// Steps: the smallest and largest key; a histogram of 2048 equal bins between them (the bins follow
// the keys that are there, where digits of fixed weight would put most of a unit's scores, a few
// binades, into a few of them); per query the bin its rank falls into.  A bin of at most 64 keys is
// ranked by one wave; a larger one gets a histogram of its own.  Where it holds more than kCrowd keys, they are first
// looked at for being one value that many rows share, which ends the search (16 units of 36 864 rows of two
// values, stage 2, 57.4 us, 85.5 with the bin taken apart to the last bit; smaller bins are seldom of one value,
// and the look costs as much as a step).  Each step costs a few vector
// instructions per key, and with sixteen waves to a compute unit an instruction per key is 16 cycles:
// that, not the LDS, is the bound.  (A radix select of four 8-bit passes, about 48 instructions per
// key and pass, took 3.4 us a pass at nine keys a thread.)
// `early`: the caller only compares keys against the result when a query's k-th value is not
// shared beyond the rank (take_eq == total_eq), so a query is settled as soon as its boundary bin is
// taken whole; the key is then the bin's lower end ("key >= result" still separates the top k).
// All threads of the block must call it, with at least one query asked.
template <int PER, bool MANY>
__device__ __forceinline__ void rank_select(const float* __restrict__ s, const RankQuery& q, int i0, Kth (&out)[3],
                                            uint32_t (&key)[PER], SelectLds& L, bool early) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool dec = q.k[1] > 0 || q.k[2] > 0;
  const int lo = q.k[0] > 0 ? 0 : q.P, hi = dec ? q.hi : q.P;  // the rows that are looked at
  // f(): with `key` holding the thread's keys from row i on.  (The row is hidden from the optimiser, here
  // and below: it would keep the outcome of every comparison with it for the next step, two scalar
  // registers each, and spill them lane by lane.)
  auto over_keys = [&](auto f) {
    if constexpr (MANY) {
      for (int base = 0; base < hi; base += kSelThreads * PER) {
        if (base + kSelThreads * PER <= lo) continue;
        load_keys<PER>(s, base + i0, lo, hi, key);
        f(base + i0);
      }
    } else {
      int i = i0;
      asm volatile("" : "+v"(i));
      f(i);
    }
  };
  if constexpr (!MANY) load_keys<PER>(s, i0, lo, hi, key);
  *reinterpret_cast<int4*>(&L.hist[0][tid * 4]) = make_int4(0, 0, 0, 0);
  *reinterpret_cast<int4*>(&L.hist[1][tid * 4]) = make_int4(0, 0, 0, 0);
  if (tid < 3) L.n_cand[tid] = 0;
  auto smaller = [](uint32_t x, uint32_t y) { return x < y ? x : y; };
  auto larger = [](uint32_t x, uint32_t y) { return x > y ? x : y; };
  uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
  over_keys([&](int) {
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      kmin = smaller(kmin, key[e]);
      kmax = larger(kmax, key[e]);
    }
  });
  kmin = wave_reduce(kmin, smaller);
  kmax = wave_reduce(kmax, larger);
  if (lane == 0) {
    L.wave_lo[wv] = kmin;
    L.wave_hi[wv] = kmax;
  }
  __syncthreads();
  kmin = wave_reduce(L.wave_lo[lane & (kSelWaves - 1)], smaller);
  kmax = wave_reduce(L.wave_hi[lane & (kSelWaves - 1)], larger);

  // query j's k-th key lies in [base[j], base[j] + 2^shift), `eq[j]` keys of its range do, and `rem[j]` of
  // them belong to the top k (the values are the same in every thread)
  const uint32_t span = kmax - kmin;
  int shift = span == 0u ? 0 : max(0, 32 - __clz((int)span) - 11);
  uint32_t base[3] = {kmin, kmin, kmin};
  int rem[3] = {q.k[0], q.k[1], q.k[2]}, eq[3] = {0, 0, 0};
  bool open[3] = {q.k[0] > 0, q.k[1] > 0, q.k[2] > 0};
  // queries 1 and 2 share the first histogram; from the second step on each has its own
  auto count_step = [&](auto first_c, int coarser) {  // coarser: the shift of the bins that are taken apart
    constexpr bool kFirst = decltype(first_c)::value;
    over_keys([&](int i) {
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const int row = i + e * 64;
        if (kFirst) {
          if (row >= lo && row < hi)
            atomicAdd(&L.hist[0][(row >= q.P ? 2 * kBins : 0) + ((key[e] - kmin) >> shift) * 2 + (lane & 1)], 1);
        } else {
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            const uint32_t off = key[e] - base[j];
            if (open[j] && (off >> coarser) == 0u && (j == 0 ? row < q.P : row >= q.P && row < q.hi))
              atomicAdd(&L.hist[j][(off >> shift) * 2 + (lane & 1)], 1);
          }
        }
      }
    });
    __syncthreads();
    // a lane's two bins, from the top: thread t has bins 2047 - 2 t and 2046 - 2 t
    int above[3], hi_bin[3], lo_bin[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      if (kFirst && j == 2) {
        above[2] = above[1], hi_bin[2] = hi_bin[1], lo_bin[2] = lo_bin[1];
      } else {
        const int4 c = *reinterpret_cast<const int4*>(&L.hist[j][(kBins - 2 - 2 * tid) * 2]);
        lo_bin[j] = c.x + c.y;
        hi_bin[j] = c.z + c.w;
        const int incl = wave_scan(lo_bin[j] + hi_bin[j]);
        if (lane == 63) L.wave_tot[j][wv] = (uint32_t)incl;
        above[j] = incl - lo_bin[j] - hi_bin[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      if (!open[j]) continue;
      uint32_t total;
      const int before = above[j] + (int)before_wave(L.wave_tot[kFirst && j == 2 ? 1 : j], wv, &total);
      if (before < rem[j] && rem[j] <= before + hi_bin[j] + lo_bin[j]) {
        const bool low = rem[j] > before + hi_bin[j];
        L.found[j][0] = kBins - 1 - 2 * tid - (low ? 1 : 0);
        L.found[j][1] = rem[j] - before - (low ? hi_bin[j] : 0);
        L.found[j][2] = low ? lo_bin[j] : hi_bin[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 3; ++j)
      if (open[j]) {
        base[j] += (uint32_t)__builtin_amdgcn_readfirstlane(L.found[j][0]) << shift;
        rem[j] = __builtin_amdgcn_readfirstlane(L.found[j][1]);
        eq[j] = __builtin_amdgcn_readfirstlane(L.found[j][2]);
        if (shift == 0 || (early && rem[j] == eq[j])) open[j] = false;
      }
  };
  count_step(std::true_type{}, 32);
  while (open[0] || open[1] || open[2]) {
    bool few = true;
#pragma unroll
    for (int j = 0; j < 3; ++j) few = few && (!open[j] || eq[j] <= kCand);
    if (few) {
      over_keys([&](int i) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
          const int row = i + e * 64;
#pragma unroll
          for (int j = 0; j < 3; ++j)
            if (open[j] && ((key[e] - base[j]) >> shift) == 0u && (j == 0 ? row < q.P : row >= q.P && row < q.hi))
              L.cand[j][atomicAdd(&L.n_cand[j], 1)] = key[e];  // (their order does not matter)
        }
      });
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (open[j] && wv == j) {
          const uint32_t mine = L.cand[j][lane];
          int more = 0, same = 0;
          for (int c = 0; c < eq[j]; ++c) {
            const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, c);
            more += other > mine ? 1 : 0;
            same += other == mine ? 1 : 0;
          }
          if (lane < eq[j] && more < rem[j] && rem[j] <= more + same) {  // (equal keys write the same)
            L.found[j][0] = (int)mine;
            L.found[j][1] = rem[j] - more;
            L.found[j][2] = same;
          }
        }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (open[j]) {
          base[j] = (uint32_t)__builtin_amdgcn_readfirstlane(L.found[j][0]);
          rem[j] = __builtin_amdgcn_readfirstlane(L.found[j][1]);
          eq[j] = __builtin_amdgcn_readfirstlane(L.found[j][2]);
          open[j] = false;
        }
    } else {
#pragma unroll
      for (int j = 0; j < 3; ++j) *reinterpret_cast<int4*>(&L.hist[j][tid * 4]) = make_int4(0, 0, 0, 0);
      if (tid < 3) L.bin_lo[tid] = 0xFFFFFFFFu, L.bin_hi[tid] = 0u;
      __syncthreads();
      if ((open[0] && eq[0] > kCrowd) || (open[1] && eq[1] > kCrowd) || (open[2] && eq[2] > kCrowd)) {
#pragma unroll 1
        for (int j = 0; j < 3; ++j) {
          if (!(j == 0 ? open[0] && eq[0] > kCrowd : j == 1 ? open[1] && eq[1] > kCrowd : open[2] && eq[2] > kCrowd)) continue;
          const uint32_t from = j == 0 ? base[0] : j == 1 ? base[1] : base[2];
          const int first = j == 0 ? 0 : q.P, end = j == 0 ? q.P : q.hi;
          uint32_t low = 0xFFFFFFFFu, top = 0u;
          over_keys([&](int i) {
#pragma unroll
            for (int e = 0; e < PER; ++e) {
              const int row = i + e * 64;
              const bool in = ((key[e] - from) >> shift) == 0u && row >= first && row < end;
              low = smaller(low, in ? key[e] : 0xFFFFFFFFu);
              top = larger(top, in ? key[e] : 0u);
            }
          });
          low = wave_reduce(low, smaller);
          top = wave_reduce(top, larger);
          if (lane == 0) {
            atomicMin(&L.bin_lo[j], low);
            atomicMax(&L.bin_hi[j], top);
          }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 3; ++j)
          if (open[j] && eq[j] > kCrowd && L.bin_lo[j] == L.bin_hi[j]) {
            base[j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.bin_lo[j]);
            open[j] = false;
          }
        if (!(open[0] || open[1] || open[2])) break;
      }
      const int coarser = shift;
      shift = max(0, shift - 11);
      count_step(std::false_type{}, coarser);
    }
  }
  __syncthreads();  // the caller may reuse the LDS
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    out[j].key = base[j];
    out[j].take_eq = rem[j];
    out[j].total_eq = eq[j];
  }
}

// Exclusive block scan of a small per-thread count (two 16-bit fields packed in one int).
// Returns the exclusive prefix; *total receives the block total.  `wsum` is kSelWaves ints.
__device__ inline int block_excl_scan(int v, uint32_t* wsum, int* total) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) wsum[wv] = (uint32_t)incl;
  __syncthreads();
  int base = 0, tot = 0;
  for (int w = 0; w < kSelWaves; ++w) {
    const int x = (int)wsum[w];
    if (w < wv) base += x;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return base + incl - v;
}

// Ordered walk over the roles of a unit: output slot of every kept row, ordinal of every seed.
// A wave owns IDX * 64 consecutive rows, read and written 64 consecutive rows at a time
// (coalesced); positions inside the wave come from ballots with a running carry (kept rows in
// the low half of an unsigned word, seeds in the high half: a wave sees at most 2304 rows, a
// chunk at most 36 864), and one exchange of the wave totals per chunk of kSelThreads * IDX rows
// orders the waves.
// Inlined on purpose: as a called function its pointers lose their address space and the
// ballots' scalar registers are spilled lane by lane, which made the walk issue-bound.
constexpr int kIdxPer = 16;

__device__ __forceinline__ bool role_is_kept(int r) {
  // prefix survivor, core, seed, recent
  return r <= CASK_ROLE_RECENT && ((0x2E >> r) & 1);
}

// Where the walk's results of one unit go (pointers already at the unit; any but `seed` may be null).
struct WalkOut {
  int32_t* slot;    // output slot of the kept rows
  int32_t* assign;  // what a row maps to, folding donors excepted (see index_rows)
  int assign_mode;  // 1: output slots, 2: unit-local rows
  int32_t* src;
  int32_t* seed;
};

// One chunk of the walk: the roles r[e] of rows i0 + 64 e (rows past N hold PREFIX_DROP).  Rows that
// are kept map to their slot or to themselves, all others to nothing: the donors that fold are entered
// by whoever groups them.  Returns the chunk's totals (kept | seeds << 16).
template <int IDX>
__device__ __forceinline__ uint32_t index_rows(int B, int N, int P, int hi, int i0, int (&r)[IDX], int kept_before,
                                               int seeds_before, const WalkOut& o, uint32_t* ws) {
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t pos[IDX];  // kept rows | seeds << 16 before this row inside the wave
  uint32_t run = 0;
#pragma unroll
  for (int e = 0; e < IDX; ++e) {
    const unsigned long long bk = __ballot(role_is_kept(r[e])), bs = __ballot(r[e] == CASK_ROLE_SEED);
    const uint32_t nk = __builtin_amdgcn_mbcnt_hi((unsigned)(bk >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bk, 0));
    const uint32_t ns = __builtin_amdgcn_mbcnt_hi((unsigned)(bs >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bs, 0));
    pos[e] = run + nk + (ns << 16);
    run += (uint32_t)__popcll(bk) + ((uint32_t)__popcll(bs) << 16);
    // the positions are final here: keep them from being recomputed behind the barrier out
    // of ballots that would have to be kept alive in scalar registers
    asm volatile("" : "+v"(pos[e]));
  }
  if ((threadIdx.x & 63) == 0) ws[wv] = run;
  __syncthreads();
  uint32_t tot;
  const uint32_t base = before_wave(ws, wv, &tot);
  asm volatile("" : "+v"(i0));  // (see rank_select)
#pragma unroll
  for (int e = 0; e < IDX; ++e) {
    asm volatile("" : "+v"(r[e]));
    const int i = i0 + e * 64;
    const uint32_t at = base + pos[e];  // inside the chunk: at most 36 864 in either half
    const int slot = kept_before + (int)(at & 0xFFFFu), ord = seeds_before + (int)(at >> 16);
    const bool kept = role_is_kept(r[e]);
    // a caller-supplied role array could keep more rows than the budget: never write past
    // the unit's B output slots
    const bool fits = kept && slot < B;
    if (i < N) {
      if (o.assign) {
        // (a caller-supplied role array may mark prefix or recent rows inside the donor range: not kept there)
        const bool counts = (i >= P && i < hi) ? r[e] == CASK_ROLE_CORE || r[e] == CASK_ROLE_SEED : kept;
        o.assign[i] = !counts ? -1 : (o.assign_mode == 1 ? (fits ? slot : -1) : i);
      }
      if (kept && o.slot) o.slot[i] = fits ? slot : -1;
      if (fits && o.src) o.src[slot] = i;
      if (r[e] == CASK_ROLE_SEED && ord < B) o.seed[ord] = i;
    }
  }
  return tot;
}

template <int IDX>
__device__ __forceinline__ void index_walk(int B, int u, int N, int P, int hi, const uint8_t* __restrict__ ro,
                                           const WalkOut& o, int32_t* __restrict__ out_len, int32_t* __restrict__ n_seeds,
                                           uint32_t (&wsum)[2][kSelWaves]) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int kept_before = 0, seeds_before = 0;  // of the chunks walked so far
  for (int cb = 0; cb < N; cb += kSelThreads * IDX) {
    const int i0 = cb + wv * (64 * IDX) + lane;
    int r[IDX];
#pragma unroll
    for (int e = 0; e < IDX; ++e) r[e] = (i0 + e * 64 < N) ? (int)ro[i0 + e * 64] : (int)CASK_ROLE_PREFIX_DROP;
    // two buffers: one barrier per chunk
    const uint32_t tot = index_rows<IDX>(B, N, P, hi, i0, r, kept_before, seeds_before, o, wsum[(cb / (kSelThreads * IDX)) & 1]);
    kept_before += (int)(tot & 0xFFFFu);
    seeds_before += (int)(tot >> 16);
  }
  if (tid == 0) {
    if (out_len) out_len[u] = kept_before < B ? kept_before : B;
    n_seeds[u] = seeds_before < B ? seeds_before : B;
  }
}

__device__ __forceinline__ WalkOut walk_out(const WalkArrays& w, int B, int u, int64_t row0) {
  WalkOut o;
  o.slot = w.slot_of ? w.slot_of + row0 : nullptr;
  o.assign = w.assign ? w.assign + row0 : nullptr;
  o.assign_mode = w.assign_mode;
  o.src = w.out_src ? w.out_src + (size_t)u * B : nullptr;
  o.seed = w.seed_rows + (size_t)u * B;
  return o;
}

// Measured, the radix select of 8-bit digits with the roles written out and read back before the walk,
// then now: 112 units of 8448 rows 22.4 / 16.2 us, 112 of 33 024 65 / 44 (two to three chunks of keys read
// in every pass before), 1024 of 4600 - 33 000 206 / 142; one stage without the walk, 56 of 6256, 14.6 / 9.0.
// Held to 64 registers for two workgroups a compute unit it spills scalars: 16.2 -> 19.1 us.
template <int PER, bool MANY>  // (two workgroups to a compute unit where the keys leave the registers for it)
__global__ __launch_bounds__(kSelThreads) void select_kernel(
    KParams kp, const int64_t* __restrict__ row_off, const int32_t* __restrict__ prefix_len,
    const float* __restrict__ scores, uint8_t* __restrict__ role, int32_t* __restrict__ status,
    int do_prefix, int do_decode, int do_index, WalkArrays walk) {
  __shared__ __attribute__((aligned(16))) SelectLds L;
  __shared__ uint32_t wsum[2][kSelWaves];
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int64_t row0 = row_off[u];
  const int N = (int)(row_off[u + 1] - row0);
  const int P = prefix_len[u];
  const UnitPlan pl = make_plan(kp, P, N);
  const float* s = scores + row0;
  uint8_t* ro = role + row0;
  if (tid == 0 && status) status[u] = pl.status;

  // which ranks have to be found: prefix rank p_keep, decode ranks C (core) and C + M (core
  // and seeds).  A rank of 0 selects nothing, a rank >= the range everything.
  const int hi = N - pl.r_eff;
  const int n = hi - P;
  const int C = pl.core, CM = pl.core + seed_range(kp, pl, n);
  const bool exhausted = (pl.status & CASK_ST_PREFIX_BUDGET_EXHAUSTED) != 0;
  const bool pre_sel = do_prefix && P > 0 && pl.p_keep > 0 && pl.p_keep < P;
  const bool dec_sel = do_decode && n > 0 && !exhausted && C < n;
  const bool all_seed = CM >= n;
  RankQuery q;
  q.P = P;
  q.hi = hi;
  q.k[0] = pre_sel ? pl.p_keep : 0;
  q.k[1] = (dec_sel && C > 0) ? C : 0;
  q.k[2] = (dec_sel && !all_seed && CM > C) ? CM : 0;
  // (stage 2 alone: the keys start behind the prefix)
  const int first_row = MANY || do_prefix || do_index ? 0 : P;
  const int i0 = first_row + (tid >> 6) * (64 * PER) + lane;
  uint32_t key[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) key[e] = 0u;
  Kth kth[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) kth[j] = {0u, 0, 0};
  if (q.k[0] > 0 || q.k[1] > 0 || q.k[2] > 0) rank_select<PER, MANY>(s, q, i0, kth, key, L, true);

  // A row's role by comparison with the k-th keys (where none of them is shared beyond its rank).
  const Kth kp0 = kth[0], kc = kth[1], km = CM > C ? kth[2] : kth[1];
  const bool pre_ties = pre_sel && kp0.take_eq != kp0.total_eq;
  const bool dec_ties = dec_sel && ((C > 0 && kc.take_eq != kc.total_eq) ||
                                    (!all_seed && CM > 0 && km.take_eq != km.total_eq));
  const bool keep_all = pl.p_keep >= P, keep_none = pl.p_keep == 0;
  const bool core_all = C >= n && !exhausted;
  auto prefix_role = [&](uint32_t k) -> int {
    return keep_all || (!keep_none && k >= kp0.key) ? CASK_ROLE_PREFIX_KEEP : CASK_ROLE_PREFIX_DROP;
  };
  auto decode_role = [&](uint32_t k) -> int {
    if (exhausted) return CASK_ROLE_DECODE_EVICT;
    const bool in_c = core_all || (C > 0 && k >= kc.key);
    const bool in_cm = all_seed || (CM > 0 && k >= km.key);
    return in_c ? CASK_ROLE_CORE : (in_cm ? CASK_ROLE_SEED : CASK_ROLE_DONOR);
  };
  if (!MANY && !pre_ties && !dec_ties) {
    int r[PER], i0 = first_row + (tid >> 6) * (64 * PER) + lane;
    asm volatile("" : "+v"(i0));
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int i = i0 + e * 64;
      const int of_decode = i < hi ? decode_role(key[e]) : (int)CASK_ROLE_RECENT;
      r[e] = i < P ? prefix_role(key[e]) : of_decode;
      if (i >= N) r[e] = CASK_ROLE_PREFIX_DROP;
      asm volatile("" : "+v"(r[e]));
      if (i < N && (i < P ? do_prefix : do_decode)) ro[i] = (uint8_t)r[e];
    }
    if (do_index) {
      const uint32_t tot = index_rows<PER>(kp.B, N, P, hi, i0, r, 0, 0, walk_out(walk, kp.B, u, row0), wsum[0]);
      if (tid == 0) {
        if (walk.out_len) walk.out_len[u] = min((int)(tot & 0xFFFFu), kp.B);
        walk.n_seeds[u] = min((int)(tot >> 16), kp.B);
      }
    }
    return;
  }

  // ---- ties at a rank, or more rows than the keys of a workgroup: roles to memory first
  if (do_prefix && !pre_ties) {
    for (int i = tid; i < P; i += kSelThreads) ro[i] = (uint8_t)prefix_role(pre_sel ? score_key(s[i]) : 0u);
  } else if (do_prefix) {
    int seen = 0;  // elements equal to the k-th key at lower indices
    for (int base = 0; base < P; base += kSelThreads) {
      const int i = base + tid;
      const uint32_t key = i < P ? score_key(s[i]) : 0u;
      const int eq = (i < P && key == kp0.key) ? 1 : 0;
      int tot;
      const int ex = block_excl_scan(eq, wsum[0], &tot);
      if (i < P) {
        const bool keep = key > kp0.key || (eq && seen + ex < kp0.take_eq);
        ro[i] = keep ? CASK_ROLE_PREFIX_KEEP : CASK_ROLE_PREFIX_DROP;
      }
      seen += tot;
    }
  }
  if (do_decode) {
    for (int i = hi + tid; i < N; i += kSelThreads) ro[i] = CASK_ROLE_RECENT;
    if (!dec_ties) {
      for (int i = P + tid; i < hi; i += kSelThreads) ro[i] = (uint8_t)decode_role(dec_sel ? score_key(s[i]) : 0u);
    } else {
      int seen_c = 0, seen_m = 0;
      for (int base = P; base < hi; base += kSelThreads) {
        const int i = base + tid;
        const bool in = i < hi;
        const uint32_t key = in ? score_key(s[i]) : 0u;
        const int eq_c = (in && C > 0 && key == kc.key) ? 1 : 0;
        const int eq_m = (in && !all_seed && CM > 0 && key == km.key) ? 1 : 0;
        int tot;
        const int ex = block_excl_scan(eq_c | (eq_m << 16), wsum[0], &tot);
        if (in) {
          const bool in_c = C > 0 && (key > kc.key || (eq_c && seen_c + (ex & 0xFFFF) < kc.take_eq));
          const bool in_cm = all_seed || (CM > 0 && (key > km.key || (eq_m && seen_m + (ex >> 16) < km.take_eq)));
          ro[i] = in_c ? CASK_ROLE_CORE : (in_cm ? CASK_ROLE_SEED : CASK_ROLE_DONOR);
        }
        seen_c += tot & 0xFFFF;
        seen_m += tot >> 16;
      }
    }
  }
  if (do_index) {
    // the roles this workgroup just wrote are read back in index order: the barrier makes
    // them visible to all of its threads
    __syncthreads();
    index_walk<PER>(kp.B, u, N, P, hi, ro, walk_out(walk, kp.B, u, row0), walk.out_len, walk.n_seeds, wsum);
  }
}

// IDX: rows a thread takes at a time; the smallest that covers the longest unit spreads it over all sixteen
// waves (56 units of 6256 rows 7.4 -> 5.2 us).
template <int IDX>
__global__ __launch_bounds__(kSelThreads) void index_roles_kernel(KParams kp, const int64_t* __restrict__ row_off,
                                                                  const int32_t* __restrict__ prefix_len,
                                                                  const uint8_t* __restrict__ role, WalkArrays walk) {
  __shared__ uint32_t wsum[2][kSelWaves];
  const int u = blockIdx.x;
  const int64_t row0 = row_off[u];
  const int N = (int)(row_off[u + 1] - row0), P = prefix_len[u];
  index_walk<IDX>(kp.B, u, N, P, N - make_plan(kp, P, N).r_eff, role + row0, walk_out(walk, kp.B, u, row0), walk.out_len,
                      walk.n_seeds, wsum);
}

// Representative-set mass diagnostics (Section 2.6): per unit
//   rho_core = mass(C) / mass(TopK),  rho_rep = mass(R) / mass(TopK)
// with TopK the min(B, N) best rows by (score descending, index ascending), C the rows that
// protection keeps verbatim (prefix survivors, decode core, recent tail) and mass(R) the sum of
// the output rows' masses.  TopK's mass comes from one rank query (the rank-B key) and a sum
// over the keys above it plus the ties that belong; sums are carried in double.  (56 units of 6256 rows:
// 17.7 us with one instance of sixteen keys and a row's score and role at a time, 10.4 now.)
__device__ inline double block_sum(double v, double* red) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();  // `red` may still be read from the previous call
  if (lane == 0) red[wv] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < kSelWaves; ++w) t += red[w];
  return t;
}

template <int PER, bool MANY>
__global__ __launch_bounds__(kSelThreads) void mass_diag_kernel(
    KParams kp, const int64_t* __restrict__ row_off, const float* __restrict__ scores,
    const uint8_t* __restrict__ role, const float* __restrict__ out_mass,
    const int32_t* __restrict__ out_len, float* __restrict__ rho) {
  __shared__ __attribute__((aligned(16))) SelectLds L;
  __shared__ double red[kSelWaves];
  const int u = blockIdx.x, tid = threadIdx.x;
  const int64_t row0 = row_off[u];
  const int N = (int)(row_off[u + 1] - row0);
  const float* s = scores + row0;
  const uint8_t* ro = role + row0;
  const int B = kp.B;
  double top = 0.0, core = 0.0, rep = 0.0;
  const int i0 = (tid >> 6) * (64 * PER) + (tid & 63);
  Kth kth[3];
  kth[0] = {0u, 0, 0};
  uint32_t key[PER];
  if (N > B) {  // the key of rank B; with N <= B every row is in TopK
    RankQuery q;
    q.P = q.hi = N;
    q.k[0] = B;
    q.k[1] = q.k[2] = 0;
    rank_select<PER, MANY>(s, q, i0, kth, key, L, false);  // (the key itself is used below)
  }
  const Kth kt = kth[0];
  for (int base = 0; base < N; base += kSelThreads * PER) {
    float v[PER];
    int r[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int i = min(base + i0 + e * 64, N - 1);
      v[e] = s[i];
      r[e] = ro[i];
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      if (base + i0 + e * 64 >= N) continue;
      if (N <= B || score_key(v[e]) > kt.key) top += (double)v[e];
      if (r[e] == CASK_ROLE_PREFIX_KEEP || r[e] == CASK_ROLE_CORE || r[e] == CASK_ROLE_RECENT) core += (double)v[e];
    }
  }
  const int len = out_len[u];
  for (int t = tid; t < len; t += kSelThreads) rep += (double)out_mass[(size_t)u * B + t];
  top = block_sum(top, red);
  core = block_sum(core, red);
  rep = block_sum(rep, red);
  if (tid == 0) {
    if (N > B) {  // the ties at the rank-B key that belong to TopK
      const uint32_t bits = (kt.key & 0x80000000u) ? (kt.key & 0x7FFFFFFFu) : ~kt.key;
      top += (double)kt.take_eq * (double)__uint_as_float(bits);
    }
    rho[2 * u + 0] = top > 0.0 ? (float)(core / top) : 1.0f;
    rho[2 * u + 1] = top > 0.0 ? (float)(rep / top) : 1.0f;
  }
}

}  // namespace

namespace {
// calls f with the smallest instance that holds the keys of the first `rows` rows of a unit; beyond the
// largest, with the one that reads them again in every step
template <typename F>
void with_select_instance(int rows, F&& f) {
  const int need = (rows + kSelThreads - 1) / kSelThreads;
  const std::false_type all;
  if (need <= 4) f(std::integral_constant<int, 4>(), all);
  else if (need <= 6) f(std::integral_constant<int, 6>(), all);
  else if (need <= 9) f(std::integral_constant<int, 9>(), all);
  else if (need <= 12) f(std::integral_constant<int, 12>(), all);
  else if (need <= 18) f(std::integral_constant<int, 18>(), all);
  else if (need <= 25) f(std::integral_constant<int, 25>(), all);
  else if (need <= kSelMost) f(std::integral_constant<int, kSelMost>(), all);
  else f(std::integral_constant<int, kSelMany>(), std::true_type());
}
}  // namespace

hipError_t launch_select(const KParams& kp, const Batch& b, const float* scores, uint8_t* role, int32_t* status,
                         bool do_prefix, bool do_decode, const WalkArrays* walk, hipStream_t st) {
  const WalkArrays w = walk ? *walk : WalkArrays{};
  // (one stage alone looks at prefixes, or at decode traces, only: 16 units of 36 864 rows, stage 1 of 4608 rows
  // 20.4 us by the longest unit, 9.4 by the longest prefix; stage 2 of 6864 rows 24.6 and 11.3)
  const int rows = walk || (do_prefix && do_decode) ? b.max_unit_len : (do_prefix ? b.max_prefix_len : b.max_decode_len);
  with_select_instance(rows, [&](auto per, auto many) {
    select_kernel<decltype(per)::value, decltype(many)::value><<<dim3(b.n_units), dim3(kSelThreads), 0, st>>>(
        kp, b.row_off, b.prefix_len, scores, role, status, do_prefix ? 1 : 0, do_decode ? 1 : 0, walk ? 1 : 0, w);
  });
  return hipGetLastError();
}

hipError_t launch_index_roles(const KParams& kp, const Batch& b, const uint8_t* role, const WalkArrays& walk,
                              hipStream_t st) {
  auto go = [&](auto per) {
    index_roles_kernel<decltype(per)::value><<<dim3(b.n_units), dim3(kSelThreads), 0, st>>>(kp, b.row_off, b.prefix_len, role, walk);
  };
  const int need = (b.max_unit_len + kSelThreads - 1) / kSelThreads;
  if (need <= 4) go(std::integral_constant<int, 4>());
  else if (need <= 8) go(std::integral_constant<int, 8>());
  else go(std::integral_constant<int, kIdxPer>());
  return hipGetLastError();
}

hipError_t launch_mass_diag(const KParams& kp, const Batch& b, const float* scores,
                            const uint8_t* role, const float* out_mass, const int32_t* out_len,
                            float* rho, hipStream_t st) {
  with_select_instance(b.max_unit_len, [&](auto per, auto many) {
    mass_diag_kernel<decltype(per)::value, decltype(many)::value><<<dim3(b.n_units), dim3(kSelThreads), 0, st>>>(
        kp, b.row_off, scores, role, out_mass, out_len, rho);
  });
  return hipGetLastError();
}

}  // namespace cask
