// Selective consolidation of the mergeable scratch (Sections 2.1, 2.4, 2.5 of the paper):
//   similarity   every donor against every seed of its unit by key cosine; best seed kept
//                when the cosine reaches tau (bf16: MFMA contraction seeds x donors^T,
//                each lane owns one donor and scans its seeds in ascending order);
//   group + fold the two steps below in one launch, for units of at most 8192 decode rows;
//   gather       ordered list of the donors that merge (ascending row), per unit, then the
//                same list grouped by seed; spare workgroups of the launch copy the kept
//                tokens to the output bit for bit, sixteen lanes per row;
//   emit         a seed with donors becomes the weighted fold m = sum a_i,
//                k~ = sum a_i k_i / m, v~ = sum a_i v_i / m with a_i the token's score,
//                accumulated in fp32 in a fixed order (reruns are bitwise identical).
#include "cask_common.h"
#include <type_traits>

namespace cask {

namespace {

constexpr float kNegInf = -__builtin_inff();

__device__ inline bool better(float sim, int ord, float best, int best_ord) {
  return sim > best || (sim == best && ord < best_ord);
}

// ------------------------------------------------------------------ similarity, MFMA path

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// What the head dimension decides about the rows a wave turns round in LDS (layout: see below).
template <int D>
struct TurnGeom {
  static constexpr int kRowBytes = D * 2;
  static constexpr int kPieces = kRowBytes / 16;          // 16-byte pieces of a row: 16 or 8
  static constexpr int kGroupRows = 64 / kPieces;         // rows one load instruction of a wave covers: 4 or 8
  static constexpr int kGroups = 32 / kGroupRows;         // such groups in a wave's 32 rows
  // LDS pitch of a group: consecutive groups start 64 bytes (four 256-byte rows) or half the banks
  // (eight 128-byte rows) apart
  static constexpr int kGroupPitch = 1024 + (D == 128 ? 64 : 128);
  static constexpr int kAddr = kGroupRows / 2;            // k-steps with addresses of their own; the rest are offsets
  static constexpr int kPrefetch = D == 128 ? 2 : 4;      // donor tiles in flight ahead of the one being contracted
};
constexpr int kSeedBlock = 128;         // seeds held in LDS at a time
constexpr int kDonorTile = 128;         // donor rows per tile: 4 waves x 32
constexpr int kMultiTiles = 4;          // tiles per workgroup where a unit's seeds take several blocks
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ inline float sumsq_bf16x8(const uint4& v) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bf16x2 x = __builtin_bit_cast(bf16x2, w[i]);
    s = __builtin_amdgcn_fdot2_f32_bf16(x, x, s, false);
  }
  return s;
}

// What the two lanes l and l + 32 hold, the same pair in both: {lower half's, upper half's}.
struct Halves { float lower, upper; };
__device__ __forceinline__ Halves both_halves(float x) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return {__uint_as_float(s[0]), __uint_as_float(s[1])};
}
__device__ __forceinline__ float inverse_norm(float ss) { return ss > 0.f ? 1.0f / sqrtf(ss) : 0.f; }

// Whether a cosine x |donor|^-1 can reach tau, from the squared norm alone: the hardware's reciprocal root
// is within an ulp for normal numbers, so the slack is generous; what passes is compared exactly later.
__device__ __forceinline__ bool may_reach(float x, float ss, float tau) {
  return ss < 1e-30f || !(x * __builtin_amdgcn_rsqf(ss) < tau - 1e-5f * __builtin_fabsf(tau));
}

// Workgroup = `tiles_per_wg` consecutive donor tiles of one unit; wave w owns rows
// [32 w, 32 w + 32) of every tile.
//
// Memory side (d = 128; d = 64 has eight 128-byte rows to a load, four loads, and as many bytes
// in flight): a wave reads its 32 rows with 8 fully coalesced loads (4 whole 256-byte rows
// per instruction: lane l takes 16-byte piece l % 16 of row l / 16), kPrefetch tiles ahead, so
// K streams at memory speed.  The registers then hold rows across lanes, not MFMA operands;
// the wave turns them round through a private LDS region: a 4-row group is kept row by row,
// the 16-byte piece g of row r at slot g ^ r of the row (a 1 KB store per instruction), and lane
// (c32, h) reads back row c32's pieces h, h + 2, ... as the B operand of the eight k-steps; with
// the 1088-byte group pitch both spread any eight consecutive lanes over all banks.  No
// barrier: the region is the wave's own.  The staged seeds use the same layout.
//
// Compute side: the unit's seeds (kSeedBlock at a time, same layout, with inverse norms) are
// the A operand, so a lane owns one donor and sees its seeds in ascending order:
// cos = (dot * |seed|^-1) * |donor|^-1 in fp32, first maximum wins.  Of 32 seeds only the largest
// product is formed (16 multiplications and 8 maxima a lane); which seed it was, and the donor's exact
// inverse norm, are found where some lane's cosine may reach tau, which most tiles' do not: an argmax
// carried along cost six dependent instructions a seed, and the vector pipes, not the stream, were the
// bound with 64 channels and with many seeds.  Places past the last seed carry a NaN as inverse norm,
// which no maximum prefers.
// ONE_BLOCK: every unit has at most kSeedBlock seeds, so they are staged once per workgroup and
// the tile loop contains nothing but the donor stream (the host knows the bound).
// Measured, an argmax per seed and the exact norm per tile before: d = 64, 128 units of 5378 rows 28.1 -> 20.0 us
// (84 MB of keys), 20 of 4000 13.6 -> 8.2; d = 128, 282 seeds, 62.6 -> 50; 30 units of 6000 rows 16.0 -> 12.2,
// 112 of 33 024 179 -> 164 (5.8 TB/s).
// RADIUS: a merge radius is set (the epilogue then looks up every seed's cache row).
template <int D, bool ONE_BLOCK, bool RADIUS>
__global__ __launch_bounds__(256, 2) void similarity_mfma_kernel(
    KParams kp, int n_units, int chunks_per_unit, int tiles_per_wg,
    const int64_t* __restrict__ row_off, const int32_t* __restrict__ prefix_len,
    const uint16_t* __restrict__ K, const uint8_t* __restrict__ role,
    const int32_t* __restrict__ seed_rows, const int32_t* __restrict__ n_seeds,
    int32_t* __restrict__ assign_ord) {
  using TG = TurnGeom<D>;
  constexpr int kRowBytes = TG::kRowBytes, kPieces = TG::kPieces, kGroupRows = TG::kGroupRows;
  constexpr int kGroups = TG::kGroups, kGroupPitch = TG::kGroupPitch, kAddr = TG::kAddr, kPrefetch = TG::kPrefetch;
  constexpr int NK = D / 16;  // k-steps
  __shared__ __attribute__((aligned(16))) unsigned char seeds[(kSeedBlock / kGroupRows) * kGroupPitch];
  __shared__ __attribute__((aligned(16))) unsigned char turn[4][kGroups * kGroupPitch];
  __shared__ __attribute__((aligned(16))) float seed_inv[kSeedBlock];
  __shared__ __attribute__((aligned(16))) int seed_pos[kSeedBlock];  // cache row of each staged seed
  int u, chunk;
  if (!map_block(n_units, chunks_per_unit, u, chunk)) return;
  chunk = turned(u, chunk, chunks_per_unit);
  const int64_t row0 = row_off[u];
  const int N = (int)(row_off[u + 1] - row0);
  const int P = prefix_len[u];
  const UnitPlan pl = make_plan(kp, P, N);
  const int hi = N - pl.r_eff;
  const int first = P + chunk * tiles_per_wg * kDonorTile;
  if (first >= hi) return;
  const int n_tiles = min(tiles_per_wg, (hi - first + kDonorTile - 1) / kDonorTile);
  const int M = n_seeds[u];
  const int tid = threadIdx.x, lane = tid & 63;
  if (M == 0) {  // no seed to fold into: nothing to read
    const int end = min(hi, first + n_tiles * kDonorTile);
    for (int i = first + tid; i < end; i += 256) assign_ord[row0 + i] = -1;
    return;
  }
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: feeds scalar load offsets
  const int c32 = lane & 31, h = lane >> 5;
  const uint16_t* Ku = K + (size_t)row0 * D;
  const uint8_t* ro = role + row0;
  const int32_t* srow = seed_rows + (size_t)u * kp.B;
  // rows past this workgroup's share of the donor range read as zero through the descriptor's
  // bounds check, without touching memory
  const int last = min(hi, first + n_tiles * kDonorTile);
  const __amdgpu_buffer_rsrc_t krsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(Ku), 0, last * kRowBytes, 0x00020000);

  // ---- donor stream: the wave's 32 rows of tile t, kGroupRows rows per load
  // (the role of the lane's donor row rides along, so that nothing at the end of a tile has
  // to wait on memory behind the loads already issued for the tiles after it)
  uint4 dreg[kPrefetch][kGroups];
  int rreg[kPrefetch];
  auto fetch_donors = [&](int t, uint4 (&d)[kGroups], int& rl) {
    // Always issued, also for tiles past the end (their rows read as zero and are never
    // stored): with an unconditional load count the waits for a tile can leave the loads of
    // the tiles after it in flight.
    const int r0 = first + t * kDonorTile + wv * 32;
    rl = (int)ro[min(r0 + c32, N - 1)];
#pragma unroll
    for (int j = 0; j < kGroups; ++j) {
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(
          krsrc, lane * 16, (int)((unsigned)(r0 + kGroupRows * j) * (unsigned)kRowBytes), 2);  // nt: a stream read once
      d[j] = make_uint4(v[0], v[1], v[2], v[3]);
    }
  };
  // ---- seeds [sb, sb + kSeedBlock) -> LDS (a thread per 16-byte piece) + inverse norms
  auto stage_seeds = [&](int sb) {
    constexpr int kPassRows = 256 / kPieces;
    const int piece = tid % kPieces, prow = tid / kPieces;
    for (int s0 = 0; s0 < kSeedBlock && sb + s0 < M; s0 += 4 * kPassRows) {
      int idx[4];
      uint4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int ord = sb + s0 + i * kPassRows + prow;
        idx[i] = ord < M ? srow[ord] : -1;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = make_uint4(0, 0, 0, 0);
        if (idx[i] >= 0) v[i] = reinterpret_cast<const uint4*>(Ku + (size_t)idx[i] * D)[piece];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int sr = s0 + i * kPassRows + prow, gr = sr % kGroupRows;
        // (row by row with piece g of row r at slot g ^ r, like the waves' turning regions)
        *reinterpret_cast<uint4*>(seeds + (sr / kGroupRows) * kGroupPitch + gr * kRowBytes + ((piece ^ gr) * 16)) = v[i];
        float ss = sumsq_bf16x8(v[i]);
#pragma unroll
        for (int o = kPieces / 2; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
        if (piece == 0) {
          seed_inv[sr] = idx[i] < 0 ? __builtin_nanf("") : inverse_norm(ss);
          seed_pos[sr] = idx[i];
        }
      }
    }
  };
  // merge radius (0 = none): seeds further than this many cache rows from the donor are skipped
  const int radius = kp.radius > 0 ? kp.radius : 0x7fffffff;

  unsigned char* my_turn = turn[wv];
  // The wave's turning region holds a group row by row, the 16-byte piece g of row r at
  // slot g ^ r of the row: the store of a load's 64 pieces (lane = row l / kPieces, piece l % kPieces) and
  // the operand reads (lane = row c32, pieces h, h + 2, ...) then both spread any eight
  // consecutive lanes over all banks.  (Piece-major -- piece g of row r at g * 64 + r * 16 -- the
  // stores ran four lanes to a bank: 44 % of the kernel's LDS cycles were bank conflicts.)
  const int turn_st = (lane / kPieces) * kRowBytes + (((lane % kPieces) ^ (lane / kPieces)) * 16);
  const int turn_row = (c32 / kGroupRows) * kGroupPitch + (c32 % kGroupRows) * kRowBytes;
  int turn_ld[kAddr];  // k-steps 0 .. kAddr - 1: piece 2 ks + h; a later one lies whole rounds of them behind
#pragma unroll
  for (int q = 0; q < kAddr; ++q) turn_ld[q] = turn_row + (((2 * q + h) ^ (c32 % kGroupRows)) * 16);
  auto turn_at = [&](int ks) { return turn_ld[ks % kAddr] + (ks / kAddr) * (kAddr * 32); };

  // registers -> private LDS region -> B operand of this lane's donor; refills the registers
  // with tile t + kPrefetch; returns the donor's squared norm
  auto turn_donors = [&](int t, uint4 (&d)[kGroups], int& rl, bf16x8 (&bres)[NK]) -> float {
#pragma unroll
    for (int j = 0; j < kGroups; ++j)
      *reinterpret_cast<uint4*>(my_turn + j * kGroupPitch + turn_st) = d[j];
    fetch_donors(t + kPrefetch, d, rl);  // refill the registers just freed
    float ss = 0.f;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
      const uint4 v = *reinterpret_cast<const uint4*>(my_turn + turn_at(ks));
      ss += sumsq_bf16x8(v);
      bres[ks] = __builtin_bit_cast(bf16x8, v);
    }
    const Halves n = both_halves(ss);
    return n.lower + n.upper;
  };
  // The lane's donor against the staged seeds [sb, sb + m_blk), ascending ordinal: first maximum
  // wins.  `best` is the cosine without the donor's own inverse norm: a positive factor common
  // to all of a donor's seeds, applied once when the winner is settled.  `best_ord` is kept only where
  // the cosine may reach tau: a larger one that may not leaves none that does behind.
  auto against_block = [&](int sb, int m_blk, const bf16x8 (&bres)[NK], int drow, float ss, float& best, int& best_ord) {
    auto chain = [&](int s0) {
      const unsigned char* ap = seeds + (s0 / kGroupRows) * kGroupPitch;
      f32x16 acc = {0};
#pragma unroll
      for (int ks = 0; ks < NK; ++ks)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(ap + turn_at(ks)), bres[ks], acc, 0, 0, 0);
      return acc;
    };
    auto pick = [&](const f32x16& acc, int s0) {
      float v[16], top = 0.f;
#pragma unroll
      for (int g = 0; g < 4; ++g) {  // ascending seed ordinal within the lane
        const float4 si = *reinterpret_cast<const float4*>(&seed_inv[s0 + g * 8 + h * 4]);
        const float sv[4] = {si.x, si.y, si.z, si.w};
        int pv[4] = {0, 0, 0, 0};
        if (RADIUS) {
          const int4 sp = *reinterpret_cast<const int4*>(&seed_pos[s0 + g * 8 + h * 4]);
          pv[0] = sp.x, pv[1] = sp.y, pv[2] = sp.z, pv[3] = sp.w;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float x = acc[g * 4 + q] * sv[q];
          if (RADIUS && (pv[q] > drow ? pv[q] - drow : drow - pv[q]) > radius) x = __builtin_nanf("");
          v[g * 4 + q] = x;
          top = g == 0 && q == 0 ? x : fmaxf(top, x);
        }
      }
      const bool wins = top > best && may_reach(top, ss, kp.tau);
      if (__builtin_amdgcn_ballot_w64(wins) != 0ull) {
        int at = 0;
#pragma unroll
        for (int i = 15; i > 0; --i) at = v[i] == top ? (i >> 2) * 8 + (i & 3) : at;
        if (v[0] == top) at = 0;
        if (wins) best_ord = sb + s0 + h * 4 + at;
      }
      best = fmaxf(best, top);
    };
    for (int s0 = 0; s0 < m_blk; s0 += 64) {  // (two chains in flight: a pick waits for its own to end)
      const f32x16 lo = chain(s0);
      if (s0 + 32 < m_blk) {
        const f32x16 up = chain(s0 + 32);
        pick(lo, s0);
        pick(up, s0 + 32);
      } else {
        pick(lo, s0);
      }
    }
  };
  // the two half-waves hold the even and the odd groups of four seeds: lowest ordinal wins a tie
  auto settle = [&](float best, int best_ord, float ss, bool donor, int drow) {
    int ord = -1;
    if (__builtin_amdgcn_ballot_w64(best_ord >= 0) != 0ull) {
      const Halves b = both_halves(best), o = both_halves(__int_as_float(best_ord));
      const int o0 = __float_as_int(o.lower), o1 = __float_as_int(o.upper);
      const bool second = o1 >= 0 && (o0 < 0 || better(b.upper, o1, b.lower, o0));
      ord = second ? o1 : o0;
      if (!(donor && ord >= 0 && (second ? b.upper : b.lower) * inverse_norm(ss) >= kp.tau)) ord = -1;
    }
    if (h == 0 && drow < last) assign_ord[row0 + drow] = ord;  // rows past the workgroup's share belong to another one
  };

  if constexpr (ONE_BLOCK) {
#pragma unroll
    for (int t = 0; t < kPrefetch; ++t) fetch_donors(t, dreg[t], rreg[t]);
    stage_seeds(0);
    __syncthreads();
    auto tile_body = [&](int t, uint4 (&d)[kGroups], int& rl) {
      const bool donor = rl == CASK_ROLE_DONOR;
      bf16x8 bres[NK];
      const float ss = turn_donors(t, d, rl, bres);
      const int drow = first + t * kDonorTile + wv * 32 + c32;
      float best = kNegInf;
      int best_ord = -1;
      against_block(0, M, bres, drow, ss, best, best_ord);
      settle(best, best_ord, ss, donor, drow);
    };
    for (int t = 0; t < n_tiles; t += kPrefetch) {
#pragma unroll
      for (int b = 0; b < kPrefetch; ++b) {
        if (t + b >= n_tiles) return;
        tile_body(t + b, dreg[b], rreg[b]);
      }
    }
  } else {
    // More seeds than LDS holds at a time: a block of seeds is staged once and meets every tile
    // of the workgroup (at most kMultiTiles; the donors stream again per block, from L2) while
    // each tile's best seed so far waits in registers.  Staging per tile instead made a unit
    // with 282 seeds and four tiles a chain of twelve stagings and twenty-four barriers.
    float best[kMultiTiles], ss[kMultiTiles];
    int best_ord[kMultiTiles];
    bool donor[kMultiTiles];
#pragma unroll
    for (int t = 0; t < kMultiTiles; ++t) {
      best[t] = kNegInf;
      ss[t] = 0.f;
      best_ord[t] = -1;
      donor[t] = false;
    }
    for (int sb = 0; sb < M; sb += kSeedBlock) {
      if (sb > 0) __syncthreads();  // previous block fully consumed
#pragma unroll
      for (int t = 0; t < kPrefetch; ++t) fetch_donors(t, dreg[t], rreg[t]);
      stage_seeds(sb);
      __syncthreads();
      const int m_blk = min(kSeedBlock, M - sb);
      static_assert(kMultiTiles % kPrefetch == 0, "whole rounds of the register ring");
#pragma unroll
      for (int t = 0; t < kMultiTiles; ++t) {
        if (t < n_tiles) {  // (the same for the whole workgroup)
          donor[t] = rreg[t % kPrefetch] == CASK_ROLE_DONOR;
          bf16x8 bres[NK];
          ss[t] = turn_donors(t, dreg[t % kPrefetch], rreg[t % kPrefetch], bres);
          against_block(sb, m_blk, bres, first + t * kDonorTile + wv * 32 + c32, ss[t], best[t], best_ord[t]);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < kMultiTiles; ++t)
      if (t < n_tiles) settle(best[t], best_ord[t], ss[t], donor[t], first + t * kDonorTile + wv * 32 + c32);
  }
}

// ------------------------------------------------------------------ similarity, fp32 caches

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kF32Slots = 512;  // workgroups aimed at: two per compute unit (three and four measured 5 - 25 % slower)

// Sizes that follow from the head dimension.
template <int D>
struct SimF32Geom {
  static constexpr int kRowBytes = D * 4;
  static constexpr int kDonorTile = 4 * 16;                // donors of a workgroup's tile: sixteen per wave
  static constexpr int kSteps = kRowBytes / 64;            // 16-byte pieces of a row per lane
  static constexpr int kRing = D == 128 ? 2 : 4;           // tiles whose rows are held or in flight
  static constexpr int kSeeds = 32768 / kRowBytes;         // seeds held in LDS at a time
  static constexpr int kSeedPitch = kRowBytes + 16;        // sixteen rows' pieces then lie in different banks
};

__device__ inline float sumsq_f32x4(const f32x4& v) {
  return __builtin_fmaf(v[3], v[3], __builtin_fmaf(v[2], v[2], __builtin_fmaf(v[1], v[1], v[0] * v[0])));
}

// Workgroup = `tiles_per_wg` consecutive donor tiles of one unit; wave w owns rows
// [16 w, 16 (w + 1)) of every tile.
//
// The products are 16x16x4 fp32 matrix tiles (seeds x donors^T, fp32 products and sums).  A lane loads the pieces it
// needs as an operand -- lane (l16, g) pieces g, g + 4, ... of row l16, piece by piece four k-steps --
// straight into registers, kRing - 1 tiles ahead: no pass through LDS, no barrier.  (A bf16 cache
// streams faster as whole rows turned round through LDS: 5.3 against 3.9 - 4.7 TB/s; an fp32 batch
// of 32 units is bound by its products and launch, not by the stream.)  Measured, 32 units of
// 4096 rows, 52 seeds: 20.8 us; a thread per donor on the vector units took 46.
//
// The unit's seeds (kSeeds at a time, with inverse norms) are the A operand, from LDS: a lane
// owns one donor and sees every fourth group of four seeds in ascending order:
// cos = (dot * |seed|^-1) * |donor|^-1, first maximum wins.  Places past the last seed
// carry a NaN as their inverse norm, which no comparison prefers.
// ONE_BLOCK, RADIUS: as for the bf16 kernel above.
template <int D, bool ONE_BLOCK, bool RADIUS>
__global__ __launch_bounds__(256, 3) void similarity_f32_kernel(
    KParams kp, int n_units, int chunks_per_unit, int tiles_per_wg,
    const int64_t* __restrict__ row_off, const int32_t* __restrict__ prefix_len,
    const float* __restrict__ K, const uint8_t* __restrict__ role,
    const int32_t* __restrict__ seed_rows, const int32_t* __restrict__ n_seeds,
    int32_t* __restrict__ assign_ord) {
  using SG = SimF32Geom<D>;
  constexpr int kRowBytes = SG::kRowBytes, kDonorTile = SG::kDonorTile;
  constexpr int KS = SG::kSteps, kRing = SG::kRing, kSeeds = SG::kSeeds, kSeedPitch = SG::kSeedPitch;
  __shared__ __attribute__((aligned(16))) unsigned char seeds[kSeeds * kSeedPitch];
  __shared__ __attribute__((aligned(16))) float seed_inv[kSeeds];
  __shared__ __attribute__((aligned(16))) int seed_pos[kSeeds];  // cache row of each staged seed
  int u, chunk;
  if (!map_block(n_units, chunks_per_unit, u, chunk)) return;
  chunk = turned(u, chunk, chunks_per_unit);
  const int64_t row0 = row_off[u];
  const int N = (int)(row_off[u + 1] - row0);
  const int P = prefix_len[u];
  const UnitPlan pl = make_plan(kp, P, N);
  const int hi = N - pl.r_eff;
  const int first = P + chunk * tiles_per_wg * kDonorTile;
  if (first >= hi) return;
  const int n_tiles = min(tiles_per_wg, (hi - first + kDonorTile - 1) / kDonorTile);
  const int M = n_seeds[u];
  const int tid = threadIdx.x, lane = tid & 63;
  if (M == 0) {  // no seed to fold into: nothing to read
    const int end = min(hi, first + n_tiles * kDonorTile);
    for (int i = first + tid; i < end; i += 256) assign_ord[row0 + i] = -1;
    return;
  }
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: feeds scalar load offsets
  const int l16 = lane & 15, g = lane >> 4;
  const float* Ku = K + (size_t)row0 * D;
  const uint8_t* ro = role + row0;
  const int32_t* srow = seed_rows + (size_t)u * kp.B;
  // rows past this workgroup's share of the donor range read as zero through the descriptor's
  // bounds check, without touching memory
  const int last = min(hi, first + n_tiles * kDonorTile);
  const __amdgpu_buffer_rsrc_t krsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Ku), 0, (int)((unsigned)last * (unsigned)kRowBytes), 0x00020000);

  // ---- donor stream (the role of the lane's donor rides along, so that nothing at the end of a
  // tile has to wait on memory behind the loads already issued for the tiles after it)
  f32x4 dreg[kRing][KS];
  int rreg[kRing];
  const int k_off = l16 * kRowBytes + g * 16;
  auto fetch_donors = [&](int t, f32x4 (&d)[KS], int& rl) {
    // Always issued, also for tiles past the end (their rows read as zero and are never
    // stored): with an unconditional load count the waits for a tile can leave the loads of
    // the tiles after it in flight.
    const int r0 = first + t * kDonorTile + wv * 16;
    rl = (int)ro[min(r0 + l16, N - 1)];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      d[ks] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
          krsrc, k_off + ks * 64, (int)((unsigned)r0 * (unsigned)kRowBytes), 0));
  };
  // ---- seeds [sb, sb + kSeeds) -> LDS (a thread per 16-byte piece) + inverse norms
  auto stage_seeds = [&](int sb) {
    constexpr int kPieces = kRowBytes / 16, kPassRows = 256 / kPieces;
    const int piece = tid % kPieces, prow = tid / kPieces;
    for (int s0 = 0; s0 < kSeeds && sb + s0 < M; s0 += 4 * kPassRows) {
      int idx[4];
      f32x4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int ord = sb + s0 + i * kPassRows + prow;
        idx[i] = ord < M ? srow[ord] : -1;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (idx[i] >= 0) v[i] = reinterpret_cast<const f32x4*>(Ku + (size_t)idx[i] * D)[piece];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int sr = s0 + i * kPassRows + prow;
        *reinterpret_cast<f32x4*>(seeds + sr * kSeedPitch + piece * 16) = v[i];
        float ss = sumsq_f32x4(v[i]);
#pragma unroll
        for (int o = kPieces / 2; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
        if (piece == 0) {
          seed_inv[sr] = idx[i] < 0 ? __builtin_nanf("") : (ss > 0.f ? 1.0f / sqrtf(ss) : 0.f);
          seed_pos[sr] = idx[i];
        }
      }
    }
  };
  // merge radius (0 = none): seeds further than this many cache rows from the donor are skipped
  const int radius = kp.radius > 0 ? kp.radius : 0x7fffffff;

  // inverse norm of the lane's donor (every lane group holds a quarter of its channels)
  auto inverse_norm = [&](const f32x4 (&d)[KS]) {
    float ss = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ss += sumsq_f32x4(d[ks]);
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    return ss > 0.f ? 1.0f / sqrtf(ss) : 0.f;
  };
  // The lane's donor against the staged seeds [sb, sb + m_blk), ascending ordinal: first maximum wins.
  auto against_block = [&](int sb, int m_blk, const f32x4 (&d)[KS], float dinv, int drow, float& best, int& best_ord) {
    for (int s0 = 0; s0 < m_blk; s0 += 16) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(seeds + (s0 + l16) * kSeedPitch + (ks * 4 + g) * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], d[ks][e], acc, 0, 0, 0);
      }
      const f32x4 si = *reinterpret_cast<const f32x4*>(&seed_inv[s0 + g * 4]);
      int pos[4] = {0, 0, 0, 0};
      if (RADIUS) {
        const int4 sp = *reinterpret_cast<const int4*>(&seed_pos[s0 + g * 4]);
        pos[0] = sp.x, pos[1] = sp.y, pos[2] = sp.z, pos[3] = sp.w;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float sim = (acc[r] * si[r]) * dinv;
        bool near = true;
        if (RADIUS) near = (pos[r] > drow ? pos[r] - drow : drow - pos[r]) <= radius;
        if (near && sim > best) {
          best = sim;
          best_ord = sb + s0 + g * 4 + r;
        }
      }
    }
  };
  // the four lane groups hold different seeds of a donor: lowest ordinal wins a tie
  auto settle = [&](float best, int best_ord, int rl, int drow) {
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      const float ob = __shfl_xor(best, o, 64);
      const int oo = __shfl_xor(best_ord, o, 64);
      if (oo >= 0 && (best_ord < 0 || better(ob, oo, best, best_ord))) {
        best = ob;
        best_ord = oo;
      }
    }
    if (g == 0 && drow < last)  // rows past the workgroup's share belong to another one
      assign_ord[row0 + drow] = (rl == CASK_ROLE_DONOR && best_ord >= 0 && best >= kp.tau) ? best_ord : -1;
  };

  if constexpr (ONE_BLOCK) {
#pragma unroll
    for (int t = 0; t < kRing; ++t) fetch_donors(t, dreg[t], rreg[t]);
    stage_seeds(0);
    __syncthreads();
    for (int t0 = 0; t0 < n_tiles; t0 += kRing) {
#pragma unroll
      for (int b = 0; b < kRing; ++b) {
        const int drow = first + (t0 + b) * kDonorTile + wv * 16 + l16;
        float best = kNegInf;
        int best_ord = -1;
        against_block(0, M, dreg[b], inverse_norm(dreg[b]), drow, best, best_ord);
        settle(best, best_ord, rreg[b], drow);
        fetch_donors(t0 + b + kRing, dreg[b], rreg[b]);  // refill the registers just freed
      }
    }
  } else {
    // a block of seeds meets every tile of the workgroup (at most kMultiTiles), whose best seeds
    // so far wait in registers, as in the bf16 kernel
    float best[kMultiTiles];
    int best_ord[kMultiTiles], donor[kMultiTiles];
#pragma unroll
    for (int t = 0; t < kMultiTiles; ++t) {
      best[t] = kNegInf;
      best_ord[t] = -1;
      donor[t] = CASK_ROLE_PREFIX_DROP;
    }
    for (int sb = 0; sb < M; sb += kSeeds) {
      if (sb > 0) __syncthreads();  // previous block fully consumed
#pragma unroll
      for (int t = 0; t < kRing; ++t) fetch_donors(t, dreg[t], rreg[t]);
      stage_seeds(sb);
      __syncthreads();
      const int m_blk = min(kSeeds, M - sb);
      static_assert(kMultiTiles % kRing == 0, "whole rounds of the register ring");
#pragma unroll
      for (int t = 0; t < kMultiTiles; ++t) {
        if (t < n_tiles) {  // (the same for the whole workgroup)
          donor[t] = rreg[t % kRing];
          against_block(sb, m_blk, dreg[t % kRing], inverse_norm(dreg[t % kRing]), first + t * kDonorTile + wv * 16 + l16,
                        best[t], best_ord[t]);
          fetch_donors(t + kRing, dreg[t % kRing], rreg[t % kRing]);
        }
      }
    }
#pragma unroll
    for (int t = 0; t < kMultiTiles; ++t)
      if (t < n_tiles) settle(best[t], best_ord[t], donor[t], first + t * kDonorTile + wv * 16 + l16);
  }
}

// ------------------------------------------------------------------ similarity, kappa geometry

// Kappa-weighted merge distance (Section 2.5): d(k_i, k_j) = sum over rotary bands f (channels
// f and f + D/2) of w_f times the Euclidean distance inside the band.  A square root per band
// keeps this off the matrix cores: one thread per donor with its key in registers, seeds staged
// in LDS 32 at a time (every lane reads the same seed element: a broadcast), fp32 throughout.
// Nearest seed wins (first minimum in ascending seed order) if its distance is <= theta.
//
// Every term is non-negative and fp32 addition of non-negative terms is monotone, so a partial
// sum is a lower bound of the finished one.  Bands are summed in chunks of eight, heaviest
// chunk (by summed weight) first, and a wave leaves a seed as soon as no lane's partial sum can
// still win (<= theta and < its best so far).  Lanes that finish hold the full sum in the same
// order as without the early exit, so the result does not depend on it.
//
// The vector pipes bound that: seven issue slots a band, at least eight bands for every seed and wave.
// Few pairs can win, and most of the others are told by the matrix cores first: a sum of non-negative
// terms is at least their Euclidean norm, d >= |W (k_i - k_j)|_2 (W: each channel times its band's
// weight), whose square is |W k_i|^2 + |W k_j|^2 - 2 <W k_i, W k_j>.  The product comes from W k rounded
// to bf16, each channel off by at most 2^-8 of itself: a product is off by at most 2^-7 + 2^-16 of |W k_i| |W k_j|,
// twice that is at most 2^-7 + 2^-16 = 0.00783 of the sum of the squares, and kScreen covers it with the fp32
// roundings (some hundred of 2^-24).  A seed is left out for a donor only
// where the bound is above theta; what is not finite, or out of the range where that holds, is never
// left out.  The distances that remain are the ones above, seeds in ascending order: the same bits.
// (112 units x 4352 rows, 128 channels, a threshold at the planted near-duplicates: 69 -> 48 us;
// 112 x 8448 with 333 seeds 1120 -> 415.  Where nearly every pair survives it costs 5 - 16 %, but for thresholds that
// leave it off, below.  Leaving it out for the block of seeds behind one that nearly all pairs survived takes
// registers that 128 channels do not have: 48 -> 59 us above.)
constexpr float kScreen = 0.008f;
template <typename T>
__device__ inline void load8(const T* p, float* out);
template <>
__device__ inline void load8<float>(const float* p, float* out) {
  const float4 a = *reinterpret_cast<const float4*>(p);
  const float4 b = *reinterpret_cast<const float4*>(p + 4);
  out[0] = a.x, out[1] = a.y, out[2] = a.z, out[3] = a.w;
  out[4] = b.x, out[5] = b.y, out[6] = b.z, out[7] = b.w;
}
template <>
__device__ inline void load8<uint16_t>(const uint16_t* p, float* out) {
  const uint4 r = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    out[2 * j] = __uint_as_float(w[j] << 16);
    out[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
  }
}

// SCREEN: off from a threshold of 1e6 on, which the distances of no ordinary keys reach (every donor folds into its
// nearest seed): nothing would be left out, and a row is loaded once instead of once for each block of
// seeds.  The same bits either way; with / without the screen, every pair surviving: 112 x 4352 with 128 seeds, 64
// channels, 410 / 354 us, 16 x 4352 fp32 with 45 119 / 107, 20 x 8448 with 333 1434 / 1344.
template <typename T, int D, bool SCREEN>
__global__ __launch_bounds__(256, 2) void similarity_kappa_kernel(
    KParams kp, int n_units, int tiles_per_unit, const int64_t* __restrict__ row_off,
    const int32_t* __restrict__ prefix_len, const T* __restrict__ K,
    const uint8_t* __restrict__ role, const int32_t* __restrict__ seed_rows,
    const int32_t* __restrict__ n_seeds, int32_t* __restrict__ assign_ord) {
  constexpr int SEEDS = 32;
  constexpr int H = D / 2;
  constexpr int NCH = H / 8;  // chunks of eight bands
  constexpr int NK = D / 16;  // k-steps of a product tile
  constexpr int PIECES = D / 8;
  __shared__ __attribute__((aligned(16))) float sk[SEEDS][D + 4];  // (lanes read different rows: on other banks)
  __shared__ bf16x8 sw[PIECES * SEEDS];  // W k of the seeds: piece p of seed s at p * SEEDS + s
  __shared__ __attribute__((aligned(16))) float sc[SEEDS];  // the seeds' half of the screen's bar
  __shared__ __attribute__((aligned(16))) float wband[H];
  __shared__ int spos[SEEDS];
  __shared__ uint32_t chunk_order;  // four bits per position: which chunk is summed there
  const int tid = threadIdx.x, lane = tid & 63;
  const float band = kp.band_w[tid % H];  // (this load and those below without a branch: all under way at once)
  int u, tile;
  if (!map_block(n_units, tiles_per_unit, u, tile)) return;
  const int64_t row0 = row_off[u];
  const int N = (int)(row_off[u + 1] - row0);
  const int P = prefix_len[u];
  const UnitPlan pl = make_plan(kp, P, N);
  const int hi = N - pl.r_eff;
  const int base = P + tile * 256;
  if (base >= hi) return;
  const int M = n_seeds[u];
  const int c32 = lane & 31, h = lane >> 5;
  const int i = base + tid;
  const bool ok = i < hi;
  const T* Ku = K + (size_t)row0 * D;
  const int32_t* srow = seed_rows + (size_t)u * kp.B;
  const uint8_t own_role = role[row0 + min(i, hi - 1)];
  if (tid < H) wband[tid] = band;
  __syncthreads();
  if (tid < 64) {
    float cw = 0.f;
    for (int f = 0; f < 8; ++f) cw += wband[(lane % NCH) * 8 + f];
    int r = 0;  // rank = chunks that come before this lane's
    for (int e = 0; e < NCH; ++e) {
      const float ce = __shfl(cw, e, 64);
      r += (int)(ce > cw) | ((int)(ce == cw) & (int)(e < lane % NCH));
    }
    uint32_t packed = (uint32_t)(lane % NCH) << (4 * r);
#pragma unroll
    for (int m = 1; m < NCH; m *= 2) packed |= (uint32_t)__shfl_xor((int)packed, m, 64);
    if (tid == 0) chunk_order = packed;
  }
  const bool donor = ok && own_role == CASK_ROLE_DONOR;
  const uint64_t donors = __builtin_amdgcn_ballot_w64(donor);

  const float bar = kp.theta * kp.theta * 1.002f;
  auto usable = [](float n2) { return n2 > 1e-26f && n2 < 1e36f; };  // (false for NaN)
  float best = __builtin_inff();
  int best_ord = -1;
  float k[D];
  if (!SCREEN) {
#pragma unroll
    for (int c = 0; c < D; c += 8) load8<T>(Ku + (size_t)(donor ? i : P) * D + c, k + c);
  }
  for (int s0 = 0; s0 < M; s0 += SEEDS) {
    const int lim = min(SEEDS, M - s0);
    float seed[SEEDS * PIECES / 256][8];  // this thread's pieces of the seeds: under way while the rows come in
#pragma unroll
    for (int j = 0; j < SEEDS * PIECES / 256; ++j) {
      const int q = j * 256 + tid, sr = q / PIECES, c = (q % PIECES) * 8;
      load8<T>(Ku + (size_t)srow[s0 + min(sr, lim - 1)] * D + c, seed[j]);  // (places past the last seed: masked below)
    }
    const int seed_at = srow[s0 + min(tid, lim - 1)];
    // W k of the wave's 64 rows as two operand tiles (lane (c32, h): row c32, channels 16 ks + 8 h ...), and
    // each row's half of the bar: a pair is left out where its product < kc + sc.  (Again for each block
    // of seeds: kept beside the rows below they do not fit the registers of two waves.)
    bf16x8 wk[2][NK];
    float kc[2];
#pragma unroll
    for (int t = 0; SCREEN && t < 2; ++t) {
      int at = min(base + (tid & ~63) + t * 32 + c32, hi - 1);
      asm volatile("" : "+v"(at));  // (else all of this is taken out of the loop)
      const T* row = Ku + (size_t)at * D;
      float n2 = 0.f;
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        float v[8];
        load8<T>(row + ks * 16 + h * 8, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = v[e] * wband[(ks * 16 + h * 8) % H + e];
          n2 = __builtin_fmaf(x, x, n2);
          wk[t][ks][e] = (__bf16)x;
        }
      }
      n2 += __shfl_xor(n2, 32, 64);
      kc[t] = usable(n2) ? 0.5f * (n2 * (1.f - kScreen) - bar) : kNegInf;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < SEEDS * PIECES / 256; ++j) {
      const int q = j * 256 + tid, sr = q / PIECES, c = (q % PIECES) * 8;
      const float(&v)[8] = seed[j];
      float n2 = 0.f;
      bf16x8 x8;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sk[sr][c + e] = v[e];
        if (!SCREEN) continue;
        const float x = v[e] * wband[c % H + e];
        n2 = __builtin_fmaf(x, x, n2);
        x8[e] = (__bf16)x;
      }
      if (!SCREEN) continue;
      sw[(q % PIECES) * SEEDS + sr] = x8;
#pragma unroll
      for (int m = 1; m < PIECES; m *= 2) n2 += __shfl_xor(n2, m, 64);  // a row's pieces: neighbouring lanes
      if (c == 0) sc[sr] = usable(n2) ? 0.5f * n2 * (1.f - kScreen) : kNegInf;
    }
    if (tid < SEEDS) spos[tid] = seed_at;
    __syncthreads();
    if (donors == 0) continue;

    // ---- screen: 32 seeds against the wave's 64 rows.  A lane owns one row of a tile and the seeds
    // 8 (r / 4) + 4 h + r % 4: the ballot of register r holds seed s of 32 rows in its lower half and
    // seed s + 4 in its upper.
    uint32_t mine = donor ? 0xffffffffu : 0u;  // seeds left for this lane's row
    if constexpr (SCREEN) {
      f32x16 acc0 = f32x16{0}, acc1 = f32x16{0};
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        const bf16x8 a = sw[(2 * ks + h) * SEEDS + c32];
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, wk[0][ks], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, wk[1][ks], acc1, 0, 0, 0);
      }
      mine = 0;
      const uint64_t d0 = (donors & 0xffffffffull) * 0x100000001ull, d1 = (donors >> 32) * 0x100000001ull;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int s = (r >> 2) * 8 + (r & 3);
        const float bs = sc[s + h * 4];
        const uint64_t m0 = __builtin_amdgcn_ballot_w64(!(acc0[r] < kc[0] + bs)) & d0;
        const uint64_t m1 = __builtin_amdgcn_ballot_w64(!(acc1[r] < kc[1] + bs)) & d1;
        if ((m0 | m1) != 0) {
          const uint64_t own = (h ? m1 : m0) >> c32;
          mine |= (uint32_t)(own & 1u) << s | (uint32_t)((own >> 32) & 1u) << (s + 4);
        }
      }
    }
    if (lim < SEEDS) mine &= (1u << lim) - 1u;
    auto skip_far = [&]() {  // to the lane's next seed within the radius
      if (kp.radius <= 0) return;
      while (mine != 0) {
        const int at = spos[__builtin_ctz(mine)];
        if ((at > i ? at - i : i - at) <= kp.radius) break;
        mine &= mine - 1;
      }
    };
    skip_far();
    if (__builtin_amdgcn_ballot_w64(mine != 0) == 0) continue;

    // ---- the pairs that are left: every lane takes its own next seed, in ascending order
    if constexpr (SCREEN) {
      int from = mine != 0 ? i : P;  // (a row costs its cache lines again with every piece: lanes without a pair share one)
      asm volatile("" : "+v"(from));  // (else the loads are taken out of the loop and spilled)
#pragma unroll
      for (int c = 0; c < D; c += 8) load8<T>(Ku + (size_t)from * D + c, k + c);
    }
    for (; __builtin_amdgcn_ballot_w64(mine != 0) != 0; mine &= mine - 1, skip_far()) {
      const bool in_reach = mine != 0;
      const int sr = in_reach ? __builtin_ctz(mine) : 0;
      const uint32_t order = __builtin_amdgcn_readfirstlane(chunk_order);
      float dist = 0.f;
      bool finished = true;
      for (int ci = 0; ci < NCH; ++ci) {
        const int c = (int)((order >> (4 * ci)) & 15u);
#pragma unroll
        for (int cc = 0; cc < NCH; ++cc) {
          if (c == cc) {
            const float4 a0 = *reinterpret_cast<const float4*>(&sk[sr][cc * 8]);
            const float4 a1 = *reinterpret_cast<const float4*>(&sk[sr][cc * 8 + 4]);
            const float4 b0 = *reinterpret_cast<const float4*>(&sk[sr][H + cc * 8]);
            const float4 b1 = *reinterpret_cast<const float4*>(&sk[sr][H + cc * 8 + 4]);
            const float4 w0 = *reinterpret_cast<const float4*>(&wband[cc * 8]);
            const float4 w1 = *reinterpret_cast<const float4*>(&wband[cc * 8 + 4]);
            const float sa[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
            const float sb[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
            const float ww[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
#pragma unroll
            for (int f = 0; f < 8; ++f) {
              const float a = k[cc * 8 + f] - sa[f];
              const float b = k[H + cc * 8 + f] - sb[f];
              dist = __builtin_fmaf(ww[f], __builtin_amdgcn_sqrtf(__builtin_fmaf(a, a, b * b)), dist);
            }
          }
        }
        const bool alive = in_reach && dist <= kp.theta && dist < best;
        if (ci + 1 < NCH && __builtin_amdgcn_ballot_w64(alive) == 0) {
          finished = false;
          break;
        }
      }
      if (finished && in_reach && dist < best) {
        best = dist;
        best_ord = s0 + sr;
      }
    }
  }
  if (ok) assign_ord[row0 + i] = (donor && best_ord >= 0 && best <= kp.theta) ? best_ord : -1;
}

template <typename T, int D>
hipError_t launch_similarity_kappa(const KParams& kp, const Batch& b, const uint8_t* role,
                                   const int32_t* seed_rows, const int32_t* n_seeds,
                                   int32_t* assign_ord, hipStream_t st) {
  const int tiles = (b.max_decode_len + 255) / 256;
  if (tiles == 0) return hipSuccess;
  auto kern = kp.theta < 1e6f ? &similarity_kappa_kernel<T, D, true> : &similarity_kappa_kernel<T, D, false>;
  kern<<<dim3(mapped_blocks(b.n_units, tiles)), dim3(256), 0, st>>>(kp, b.n_units, tiles, b.row_off, b.prefix_len, static_cast<const T*>(b.K),
                                                                    role, seed_rows, n_seeds, assign_ord);
  return hipGetLastError();
}

// ------------------------------------------------------------------ gather merged donors

constexpr int kGatherThreads = 1024;
constexpr int kGatherPer = 16;  // 64-row groups per wave and chunk, at most (the kernel's instances: 4, 8, 16)
constexpr int kSegLds = 8192;   // seed ordinals whose segment cursors fit in LDS at a time
constexpr int kSmallList = 64;  // donor lists up to this length are split by a single wave

// row groups (of four rows) a copy wave handles one after the other; measured: two beat four
// and one (a long prefix-heavy copy, B = 2048: 64 us against 76 and 74)
constexpr int kCopyRounds = 2;
constexpr int kCopySlots = 4 * kCopyRounds;  // output slots of a copy wave

// Copy of the rows an event keeps as they are (Sections 2.1, 2.4: protected tokens and the kept
// part of the scratch stay untouched; only a seed with donors becomes a folded representative).
// A wave owns 8 consecutive output slots of one unit, sixteen lanes a row (a sixteenth of the
// row each); it puts the loads of its rows of K and V in flight before it touches any of them
// and writes every slot but the seeds' (LEAVE_SEEDS), which the workgroups that fold
// them write beside it; without, the seeds' too: a fold that follows in the stream overwrites
// those whose group has donors.  The copy needs nothing but the ordered walk's output, so it
// shares a launch with the grouping of the donors, whose workgroups leave most of the chip
// idle.  The row pieces are native vectors: with HIP's vector classes the staging arrays end up
// in scratch memory.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <typename Vec, int PIECES, bool LEAVE_SEEDS>
__device__ __forceinline__ void copy_kept_rows(const CopyJob& cj, int B,
                                               const int64_t* __restrict__ row_off,
                                               int u, int t_base, int lane) {
  constexpr int BPL = (int)sizeof(Vec) * PIECES;  // a lane's share of a row: a sixteenth of it
  const int grp = lane >> 4, gl = lane & 15;
  int slot[kCopyRounds], src[kCopyRounds], c0[kCopyRounds], rl[kCopyRounds];
  float a0[kCopyRounds];
  Vec kraw[kCopyRounds][PIECES], vraw[kCopyRounds][PIECES];
  // the slots' sources are read along with the unit's length, which says how many of them mean
  // anything (every unit owns B slots of the array: one round trip instead of two)
#pragma unroll
  for (int j = 0; j < kCopyRounds; ++j) {
    slot[j] = t_base + j * 4 + grp;
    src[j] = slot[j] < B ? cj.out_src[(size_t)u * B + slot[j]] : -1;
  }
  const int len = cj.out_len[u];
  if (t_base >= len) return;
  const int64_t row0 = row_off[u];
  const size_t pitch = (size_t)16 * BPL;
#pragma unroll
  for (int j = 0; j < kCopyRounds; ++j) {
    if (slot[j] >= len) src[j] = -1;
    // a slot past the unit's length reads the unit's first row and writes nothing
    const int64_t row = row0 + max(src[j], 0);
    const size_t at = (size_t)row * pitch + (size_t)gl * BPL;
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
      kraw[j][q] = *reinterpret_cast<const Vec*>(cj.K + at + q * sizeof(Vec));
      vraw[j][q] = *reinterpret_cast<const Vec*>(cj.V + at + q * sizeof(Vec));
    }
    a0[j] = cj.scores[row];
    c0[j] = cj.in_count ? cj.in_count[row] : 1;
    if (LEAVE_SEEDS) rl[j] = cj.role[row];
  }
#pragma unroll
  for (int j = 0; j < kCopyRounds; ++j) {
    if (src[j] < 0 || (LEAVE_SEEDS && rl[j] == CASK_ROLE_SEED)) continue;
    const size_t at = ((size_t)u * cj.out_stride + slot[j]) * pitch + (size_t)gl * BPL;
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
      *reinterpret_cast<Vec*>(cj.K_out + at + q * sizeof(Vec)) = kraw[j][q];
      *reinterpret_cast<Vec*>(cj.V_out + at + q * sizeof(Vec)) = vraw[j][q];
    }
    if (cj.out_mass && gl == 0) cj.out_mass[(size_t)u * B + slot[j]] = a0[j];
    if (cj.out_count && gl == 0) cj.out_count[(size_t)u * B + slot[j]] = c0[j];
  }
}

// Workgroups below `n_gather` group the donors of one unit each; the ones above copy kept rows
// (`cj.K_out` null: there are none).
// assign_mode: 0 none, 1 output slot (whole event), 2 unit-local source row (consolidate API)
template <int PER>
__global__ __launch_bounds__(kGatherThreads) void gather_merged_kernel(
    KParams kp, int n_gather, CopyJob cj,
    const int64_t* __restrict__ row_off, const int32_t* __restrict__ prefix_len,
    const int32_t* __restrict__ assign_ord,
    const int32_t* __restrict__ slot_of, const int32_t* __restrict__ seed_rows,
    int32_t* __restrict__ merged_row, int32_t* __restrict__ merged_ord,
    int32_t* __restrict__ n_merged, int32_t* __restrict__ assign_out, int assign_mode,
    int32_t* __restrict__ status, const int32_t* __restrict__ n_seeds,
    int32_t* __restrict__ seg_row, int32_t* __restrict__ seg_start) {
  __shared__ int wsum[kGatherThreads / 64];
  __shared__ int cursor[kSegLds];
  const int u = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (u >= n_gather) {
    const long long wave = (long long)(u - n_gather) * (kGatherThreads / 64) + wv;
    const int per_unit = (kp.B + kCopySlots - 1) / kCopySlots, cu = (int)(wave / per_unit), first = (int)(wave % per_unit) * kCopySlots;
    if (cu >= cj.n_units) return;
    if (cj.lane_bytes == 16) copy_kept_rows<u32x4, 1, false>(cj, kp.B, row_off, cu, first, lane);
    else if (cj.lane_bytes == 32) copy_kept_rows<u32x4, 2, false>(cj, kp.B, row_off, cu, first, lane);
    else copy_kept_rows<u32x2, 1, false>(cj, kp.B, row_off, cu, first, lane);
    return;
  }
  const int64_t row0 = row_off[u];
  const int N = (int)(row_off[u + 1] - row0);
  const int P = prefix_len[u];
  const UnitPlan pl = make_plan(kp, P, N);
  const int hi = N - pl.r_eff;
  const int32_t* srow = seed_rows + (size_t)u * kp.B;
  // A wave owns PER * 64 consecutive rows of a chunk, touched 64 consecutive rows at a time
  // (coalesced); positions inside the wave come from ballots with a running carry, and one
  // exchange of the wave totals per chunk orders the waves.
  const unsigned long long below = (1ull << lane) - 1ull;
  int count = 0;
  for (int cb = P; cb < hi; cb += kGatherThreads * PER) {
    const int i0 = cb + wv * (64 * PER) + lane;
    int ord[PER], pos[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) ord[e] = i0 + e * 64 < hi ? assign_ord[row0 + i0 + e * 64] : -1;  // (>= 0: a donor that folds)
    int run = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const unsigned long long b = __ballot(ord[e] >= 0);
      pos[e] = run + __popcll(b & below);
      run += __popcll(b);
    }
    if (lane == 0) wsum[wv] = run;
    __syncthreads();
    int before = 0, tot = 0;
    for (int w = 0; w < kGatherThreads / 64; ++w) {
      const int x = wsum[w];
      if (w < wv) before += x;
      tot += x;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int i = i0 + e * 64;
      if (i < hi && ord[e] >= 0) {
        const int at = count + before + pos[e];
        merged_row[row0 + at] = i;
        merged_ord[row0 + at] = ord[e];
        if (at < kSmallList) {  // the head of the list also waits in LDS for the short-list split below
          cursor[at] = ord[e];
          cursor[kSmallList + at] = i;
        }
      }
    }
    if (assign_mode != 0) {
      // A folding donor maps to its seed (all other rows were entered by the ordered walk).  The two
      // dependent lookups (seed's row, then its slot) are taken for all of the thread's rows at a
      // time: one after the other, every row would wait for its own round trip.
      int tgt[PER];
#pragma unroll
      for (int e = 0; e < PER; ++e) tgt[e] = ord[e] >= 0 ? srow[ord[e]] : -1;
      if (assign_mode == 1) {
#pragma unroll
        for (int e = 0; e < PER; ++e)
          if (ord[e] >= 0) tgt[e] = slot_of[row0 + tgt[e]];
      }
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if (ord[e] >= 0) assign_out[row0 + i0 + e * 64] = tgt[e];
    }
    count += tot;
  }
  if (tid == 0) {
    if (n_merged) n_merged[u] = count;
    if (status && count == 0 && !(pl.status & (CASK_ST_IDENTITY | CASK_ST_PREFIX_BUDGET_EXHAUSTED)))
      status[u] = pl.status | CASK_ST_MERGE_INACTIVE;
  }
  if (seg_row == nullptr || count == 0) return;  // count is the same in every thread

  // Second pass: the same donors grouped by seed ordinal, rows still ascending inside a group
  // (a stable split), so that a seed's fold reads one contiguous segment.
  __syncthreads();  // the list written above is read by other threads below
  const int M = n_seeds[u];
  const int32_t* mrow = merged_row + row0;
  const int32_t* mord = merged_ord + row0;
  int32_t* sstart = seg_start + (size_t)u * (kp.B + 1);
  if (count <= kSmallList) {
    // A list of at most 64 donors (the usual case: few donors reach the threshold) is split by
    // one wave from its copy in LDS: an entry's place is the number of entries with a smaller
    // ordinal plus the earlier ones with the same ordinal; a segment starts at the number of
    // entries with a smaller ordinal.
    if (wv == 0) {
      const int o_l = lane < count ? cursor[lane] : 0x7fffffff;
      const int r_l = cursor[kSmallList + lane];
      int place = 0;
      for (int j = 0; j < count; ++j) {
        const int oj = __shfl(o_l, j, 64);
        place += (oj < o_l || (oj == o_l && j < lane)) ? 1 : 0;
      }
      if (lane < count) seg_row[row0 + place] = r_l;
    }
    for (int q = tid; q <= M; q += kGatherThreads) {
      int smaller = 0;
      for (int j = 0; j < count; ++j) smaller += cursor[j] < q ? 1 : 0;
      sstart[q] = smaller;
    }
    return;
  }
  // Longer lists: every wave owns a contiguous run of the list.  Per range of kWaveOrds
  // ordinals: a histogram per wave in LDS, from which every (wave, ordinal) pair gets the place
  // of its first entry (the segment's start plus what the earlier waves hold of that ordinal).
  // Then a wave walks its run 64 entries at a time: an entry's place is its pair's cursor plus
  // the number of earlier lanes with the same ordinal (the lanes that agree in every bit of the
  // ordinal: one ballot per bit), so rows stay ascending inside a segment and no two waves
  // touch the same cursor.
  constexpr int NWV = kGatherThreads / 64;
  constexpr int kWaveOrds = kSegLds / NWV;  // ordinals per range: a cursor per wave and ordinal
  static_assert(kWaveOrds <= kGatherThreads, "a thread per ordinal of a range");
  const int run = (count + NWV * 64 - 1) / (NWV * 64) * 64;
  const int c0 = min(count, wv * run), c1 = min(count, c0 + run);
  int* const my_cursor = cursor + wv * kWaveOrds;
  int base = 0;
  for (int o_lo = 0; o_lo < M; o_lo += kWaveOrds) {
    const int range = min(kWaveOrds, M - o_lo);
    int nbits = 1;
    while ((1 << nbits) < range) ++nbits;
    for (int q = tid; q < kSegLds; q += kGatherThreads) cursor[q] = 0;
    __syncthreads();
    for (int idx = c0 + lane; idx < c1; idx += 64) {
      const int o = mord[idx] - o_lo;
      if (o >= 0 && o < range) atomicAdd(&my_cursor[o], 1);
    }
    __syncthreads();
    // thread q: ordinal o_lo + q.  Its entries per wave become the waves' offsets inside the
    // segment; the segment starts come from a scan of the totals.
    int total = 0;
    if (tid < range) {
      for (int w = 0; w < NWV; ++w) {
        const int t = cursor[w * kWaveOrds + tid];
        cursor[w * kWaveOrds + tid] = total;
        total += t;
      }
    }
    int incl = total;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int before = 0, tot = 0;
    for (int w = 0; w < NWV; ++w) {
      const int x = wsum[w];
      if (w < wv) before += x;
      tot += x;
    }
    if (tid < range) {
      const int start = base + before + (incl - total);
      sstart[o_lo + tid] = start;
      for (int w = 0; w < NWV; ++w) cursor[w * kWaveOrds + tid] += start;
    }
    base += tot;
    __syncthreads();
    constexpr int kAhead = 4;  // 64-entry steps whose loads are in flight together
    for (int i0 = c0; i0 < c1; i0 += 64 * kAhead) {
      int os[kAhead], rs[kAhead];
#pragma unroll
      for (int e = 0; e < kAhead; ++e) {
        const int idx = min(i0 + e * 64 + lane, c1 - 1);  // clamped: no branch around the loads
        os[e] = mord[idx];
        rs[e] = mrow[idx];
      }
#pragma unroll
      for (int e = 0; e < kAhead; ++e) {
        const int idx = i0 + e * 64 + lane;
        const int o = os[e] - o_lo;
        const bool valid = idx < c1 && o >= 0 && o < range;
        unsigned long long same = __ballot(valid);
        for (int bit = 0; bit < nbits; ++bit) {
          const bool one = ((o >> bit) & 1) != 0;
          const unsigned long long ones = __ballot(valid && one);
          same &= one ? ones : ~ones;
        }
        if (valid) {  // `same`: the valid lanes with this lane's ordinal
          const int rank = __popcll(same & below);
          const int cur = my_cursor[o];
          seg_row[row0 + cur + rank] = rs[e];
          if (rank == __popcll(same) - 1) my_cursor[o] = cur + rank + 1;  // (after every lane's read)
        }
      }
    }
    __syncthreads();  // the cursors are cleared for the next range
  }
  if (tid == 0) sstart[M] = count;
}

// ------------------------------------------------------------------ emit (fold)

// Sixteen lanes hold one row (D / 16 elements each).  A seed with up to kWaveFoldMax donors is
// folded by one wave: its four 16-lane groups take the seed's donors (one contiguous segment of
// the grouped donor list, ascending rows) round-robin, four donors' loads in flight per group,
// accumulate in fp32 in ascending order, and the four partial sums are added in a fixed tree.
// A longer group is folded by the four waves of a workgroup together (sixteen groups, the
// waves' sums added in a fixed tree through LDS).  Either way the result depends on the group
// alone, not on timing.  Runs after the launch that copied every kept row, the seeds' own rows
// included, and overwrites the slots of the seeds that have donors.
constexpr int kWaveFoldMax = 64;  // donors of one seed that a single wave folds (four rounds of its four groups)

template <typename T>
struct FoldIo {
  const T* K;
  const T* V;
  const float* scores;
  const int32_t* in_count;
  T* K_out;
  T* V_out;
  float* out_mass;
  int32_t* out_count;
  int out_stride, B;
};
// (kernels take the pointers one by one, as ones that do not alias: from a struct of them the loads of a group
// would be kept behind the stores of the one before)
#define CASK_FOLD_ARGS(T)                                                                                              \
  const T *__restrict__ K, const T *__restrict__ V, const float *__restrict__ scores, const int32_t *__restrict__ in_count, \
      T *__restrict__ K_out, T *__restrict__ V_out, float *__restrict__ out_mass, int32_t *__restrict__ out_count, int out_stride, int B
template <typename T, int D>
struct FoldLane {
  static constexpr int EPL = D / 16;                    // elements per lane
  static constexpr int WORDS = EPL * sizeof(T) / 4;     // 32-bit words per lane
  struct alignas(WORDS * 4 > 16 ? 16 : WORDS * 4) Raw { uint32_t w[WORDS]; };
  typedef uint32_t Words __attribute__((ext_vector_type(WORDS), aligned(WORDS * 4 > 16 ? 16 : WORDS * 4)));
  struct Share {                                        // four waves' sums of a group that they fold together
    float part[4][4 * EPL][16];
    float mass[4];
    int count[4];
  };
};

// Folds donors [s0, s1) of one seed (row `srow` of the unit at row0) into output slot `slot`; donor k is row
// row_at(k).  `NG` 16-lane groups share them round-robin and this one is number `g`: a wave's four, or
// the sixteen of four waves (`all`: wave w4 of four; every thread of the workgroup then has to call it,
// with s0 == s1 and `live` false where there is nothing to fold), whose sums are added through LDS as
// (w0 + w1) + (w2 + w3).
template <typename T, int D, int NG, bool ALL, typename RowAt>
__device__ __forceinline__ void fold_group(const FoldIo<T>& io, int u, int64_t row0, int srow, int slot, int s0, int s1, int g, int w4,
                                           bool live, RowAt row_at, typename FoldLane<T, D>::Share* share) {
  using FL = FoldLane<T, D>;
  constexpr int EPL = FL::EPL;
  typedef typename FL::Raw Raw;
  const int lane = threadIdx.x & 63, grp = lane >> 4, gl = lane & 15;
  float ka[EPL], va[EPL], ku[EPL], vu[EPL];  // score-weighted and count-weighted sums
  float mass = 0.f;
  int count = 0;
#pragma unroll
  for (int e = 0; e < EPL; ++e) ka[e] = va[e] = ku[e] = vu[e] = 0.f;
  if (live && g == 0) {  // the seed's own row opens the first group's sum
    const float a = io.scores[row0 + srow];
    const int c = io.in_count ? io.in_count[row0 + srow] : 1;
    const Raw sk = *reinterpret_cast<const Raw*>(io.K + (size_t)(row0 + srow) * D + gl * EPL);
    const Raw sv = *reinterpret_cast<const Raw*>(io.V + (size_t)(row0 + srow) * D + gl * EPL);
    const T* skp = reinterpret_cast<const T*>(&sk);
    const T* svp = reinterpret_cast<const T*>(&sv);
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      const float kf = Elem<T>::load(skp + e), vf = Elem<T>::load(svp + e);
      ka[e] = a * kf; va[e] = a * vf; ku[e] = (float)c * kf; vu[e] = (float)c * vf;
    }
    mass = a;
    count = c;
  }
  for (int idx = s0 + g; idx < s1; idx += 4 * NG) {
    int drow[4], dc[4];
    float a[4];
    Raw dk[4], dv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) drow[q] = row_at(min(idx + NG * q, s1 - 1));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[q] = io.scores[row0 + drow[q]];
      dc[q] = io.in_count ? io.in_count[row0 + drow[q]] : 1;
      dk[q] = *reinterpret_cast<const Raw*>(io.K + (size_t)(row0 + drow[q]) * D + gl * EPL);
      dv[q] = *reinterpret_cast<const Raw*>(io.V + (size_t)(row0 + drow[q]) * D + gl * EPL);
    }
    __builtin_amdgcn_sched_barrier(0);  // (all four rows on their way before the first is taken)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (idx + NG * q < s1) {
        const float dcf = (float)dc[q];
        const T* dkp = reinterpret_cast<const T*>(&dk[q]);
        const T* dvp = reinterpret_cast<const T*>(&dv[q]);
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          const float kf = Elem<T>::load(dkp + e), vf = Elem<T>::load(dvp + e);
          ka[e] = __builtin_fmaf(a[q], kf, ka[e]);
          va[e] = __builtin_fmaf(a[q], vf, va[e]);
          ku[e] = __builtin_fmaf(dcf, kf, ku[e]);
          vu[e] = __builtin_fmaf(dcf, vf, vu[e]);
        }
        mass += a[q];
        count += dc[q];
      }
    }
  }
  // (g0 + g1) + (g2 + g3): addition commutes, so every lane ends with the same bits
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      ka[e] += __shfl_xor(ka[e], o, 64);
      va[e] += __shfl_xor(va[e], o, 64);
      ku[e] += __shfl_xor(ku[e], o, 64);
      vu[e] += __shfl_xor(vu[e], o, 64);
    }
    mass += __shfl_xor(mass, o, 64);
    count += __shfl_xor(count, o, 64);
  }
  if constexpr (ALL) {
    // The waves' sums meet in LDS.  The first of the four adds them as (w0 + w1) + (w2 + w3), its 16-lane
    // group q taking one of the four sums (score-weighted K, V, count-weighted K, V), and the two
    // groups whose sums the result is made of write it.
    if (grp == 0) {
#pragma unroll
      for (int e = 0; e < EPL; ++e) {
        share->part[w4][e][gl] = ka[e];
        share->part[w4][EPL + e][gl] = va[e];
        share->part[w4][2 * EPL + e][gl] = ku[e];
        share->part[w4][3 * EPL + e][gl] = vu[e];
      }
      if (gl == 0) {
        share->mass[w4] = mass;
        share->count[w4] = count;
      }
    }
    __syncthreads();
    if (live && w4 == 0) {
      const float m = (share->mass[0] + share->mass[1]) + (share->mass[2] + share->mass[3]);
      const int c = (share->count[0] + share->count[1]) + (share->count[2] + share->count[3]);
      const bool uniform = m == 0.f;  // no score mass: average over the original tokens
      const float denom = uniform ? (float)c : m;
      if ((grp >= 2) == uniform) {
        Raw o_;
        T* op = reinterpret_cast<T*>(&o_);
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          const int k = grp * EPL + e;
          Elem<T>::store(op + e, ((share->part[0][k][gl] + share->part[1][k][gl]) + (share->part[2][k][gl] + share->part[3][k][gl])) / denom);
        }
        T* dst = (grp & 1) ? io.V_out : io.K_out;
        *reinterpret_cast<Raw*>(dst + ((size_t)u * io.out_stride + slot) * D + gl * EPL) = o_;
      }
      if (io.out_mass && lane == 0) io.out_mass[(size_t)u * io.B + slot] = m;
      if (io.out_count && lane == 0) io.out_count[(size_t)u * io.B + slot] = c;
    }
    __syncthreads();  // the next group's sums go to the same place
  } else if (grp == 0) {
    const bool uniform = mass == 0.f;  // no score mass: average over the original tokens
    const float denom = uniform ? (float)count : mass;
    Raw ok_, ov_;
    T* okp = reinterpret_cast<T*>(&ok_);
    T* ovp = reinterpret_cast<T*>(&ov_);
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      Elem<T>::store(okp + e, (uniform ? ku[e] : ka[e]) / denom);
      Elem<T>::store(ovp + e, (uniform ? vu[e] : va[e]) / denom);
    }
    *reinterpret_cast<Raw*>(io.K_out + ((size_t)u * io.out_stride + slot) * D + gl * EPL) = ok_;
    *reinterpret_cast<Raw*>(io.V_out + ((size_t)u * io.out_stride + slot) * D + gl * EPL) = ov_;
    if (io.out_mass && gl == 0) io.out_mass[(size_t)u * io.B + slot] = mass;
    if (io.out_count && gl == 0) io.out_count[(size_t)u * io.B + slot] = count;
  }
}

template <typename T, int D>
__global__ __launch_bounds__(256) void emit_kernel(
    int n_units, int fold_per_unit, CASK_FOLD_ARGS(T), const int64_t* __restrict__ row_off, const int32_t* __restrict__ seed_rows,
    const int32_t* __restrict__ n_seeds, const int32_t* __restrict__ slot_of,
    const int32_t* __restrict__ seg_row, const int32_t* __restrict__ seg_start, const int32_t* __restrict__ n_merged) {
  const FoldIo<T> io = {K, V, scores, in_count, K_out, V_out, out_mass, out_count, out_stride, B};
  __shared__ int long_item[256][4];              // (unit, ordinal, segment bounds) of the long groups of a round
  __shared__ int n_long;
  __shared__ typename FoldLane<T, D>::Share share;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, grp = lane >> 4;
  auto fold = [&](int u, int ord, int s0, int s1, auto all_c) {
    constexpr bool kAll = decltype(all_c)::value;
    const int64_t row0 = row_off[u];
    const int32_t* seg = seg_row + row0;
    const int srow = seed_rows[(size_t)u * B + ord], slot = slot_of[row0 + srow];
    fold_group<T, D, kAll ? 16 : 4, kAll>(io, u, row0, srow, slot, s0, s1, kAll ? wv * 4 + grp : grp, wv, true,
                                          [&](int k) { return seg[k]; }, &share);
  };

  // Work items are (unit, seed ordinal) pairs; each lane tests one item of a round
  // (neighbouring ordinals go to different waves).  A wave folds its items that have up to
  // kWaveFoldMax donors one after the other; the longer ones are put on a list and folded by
  // the whole workgroup, one after the other: a seed that gathered a thousand donors is
  // otherwise a chain of sixty dependent round trips in one wave while the chip idles.
  const int NW = (int)gridDim.x * 4;
  const int w = (int)blockIdx.x * 4 + wv;
  const long long items = (long long)n_units * fold_per_unit;
  for (long long base = 0; base < items; base += 64LL * NW) {  // (the same trips in every wave)
    if (threadIdx.x == 0) n_long = 0;
    __syncthreads();
    const long long item = base + (long long)lane * NW + w;
    int my_u = 0, my_ord = 0, my_s0 = 0, my_s1 = 0;
    if (item < items) {
      my_u = (int)(item / fold_per_unit);
      my_ord = (int)(item % fold_per_unit);
      // the segment bounds are read along with the counts that say whether they mean anything
      // (the slots exist for every ordinal below B; one round trip instead of two)
      const int s0 = seg_start[(size_t)my_u * (B + 1) + my_ord];
      const int s1 = seg_start[(size_t)my_u * (B + 1) + my_ord + 1];
      if (my_ord < n_seeds[my_u] && n_merged[my_u] > 0) {
        my_s0 = s0;
        my_s1 = s1;
      }
    }
    if (my_s1 - my_s0 > kWaveFoldMax) {
      const int at = atomicAdd(&n_long, 1);  // (the order on the list does not reach the results)
      long_item[at][0] = my_u;
      long_item[at][1] = my_ord;
      long_item[at][2] = my_s0;
      long_item[at][3] = my_s1;
    }
    unsigned long long todo = __ballot(my_s1 > my_s0 && my_s1 - my_s0 <= kWaveFoldMax);
    while (todo != 0ull) {
      const int src_lane = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
      fold(__shfl(my_u, src_lane, 64), __shfl(my_ord, src_lane, 64), __shfl(my_s0, src_lane, 64),
           __shfl(my_s1, src_lane, 64), std::false_type{});
    }
    __syncthreads();
    const int nl = n_long;
    for (int i = 0; i < nl; ++i)
      fold(long_item[i][0], long_item[i][1], long_item[i][2], long_item[i][3], std::true_type{});
    __syncthreads();  // everyone has read the list's length before it is cleared
  }
}

#define CASK_FOLD_PASS(T)                                                                                            \
  static_cast<const T*>(b.K), static_cast<const T*>(b.V), cj.scores, cj.in_count, reinterpret_cast<T*>(cj.K_out),     \
      reinterpret_cast<T*>(cj.V_out), cj.out_mass, cj.out_count, cj.out_stride, kp.B

template <typename T, int D>
hipError_t launch_emit_t(const KParams& kp, const Batch& b, const int32_t* seed_rows, const int32_t* n_seeds, const int32_t* slot_of,
                         const int32_t* seg_row, const int32_t* seg_start, const int32_t* n_merged, const CopyJob& cj, hipStream_t st) {
  // (unit, seed ordinal) work items; a fold wave tests 64 of them per round
  const int fold_per_unit = plan_seed_bound(kp);
  const long long items = (long long)b.n_units * fold_per_unit;
  long long fold_blocks = (items + 3) / 4;     // an item per wave ...
  if (fold_blocks > 2048) fold_blocks = 2048;  // ... up to 8192 waves
  if (fold_blocks == 0) return hipSuccess;
  emit_kernel<T, D><<<dim3((unsigned)fold_blocks), dim3(256), 0, st>>>(
      b.n_units, fold_per_unit, CASK_FOLD_PASS(T), b.row_off, seed_rows, n_seeds, slot_of, seg_row, seg_start, n_merged);
  return hipGetLastError();
}

// ------------------------------------------------------------------ grouping and fold in one launch

constexpr int kFoldThreads = 512;
constexpr int kFoldWaves = kFoldThreads / 64;
constexpr int kFoldTeams = kFoldWaves / 4;   // four waves fold a long group together
constexpr int kFoldSeeds = 1024;             // most seeds of a unit (rule at launch_group_fold)
constexpr int kFoldList = 1024;              // donors that wait in LDS
constexpr int kFoldAhead = 16;               // rows of a thread in flight

// Grouping, fold and copy of an event in one launch.  `shares` workgroups (a power of two) take a unit
// together without a word between them: each reads the donors' assignments of the whole unit and keeps
// those of its own seeds, ordinals congruent to its number.  What is read several times comes from L2;
// what is saved is a launch and the trips through memory that carried the groups to it.
// A workgroup's donors usually fit a list in LDS (ascending rows, seeds of at most kWaveFoldMax donors):
// a wave takes a seed, picks its rows out of the list by ballots and folds them.  Otherwise the list goes to
// memory and is split by seed there, stably: a histogram per wave gives every (wave, seed) pair its
// first place, and a wave walks its run 64 entries at a time; four waves together fold a long group.
// Either way a seed's donors are summed in the order and the tree of fold_group: the same bits.
// A seed without donors is copied as it is; the copying workgroups leave the seeds out.
// Bound: a chain of about five trips to memory.  Against the two launches (grouping and copy, fold): 112 units of
// 8448 rows 23.2 -> 18.5 us, 8 of 3000 11.8 -> 8.8, 128 of 5378 (d = 64) 15.8 -> 13.6; every donor folding, the
// event on 8 x 3000 rows 79.8 -> 72.6 us.  With the workgroups anywhere on the chip: 19.9, 10.1, 14.7.
template <typename T, int D>
__global__ __launch_bounds__(kFoldThreads, 2) void group_fold_kernel(
    KParams kp, CASK_FOLD_ARGS(T), int n_units, int n_fold, int shares, int seeds, CopyJob cj, const int64_t* __restrict__ row_off,
    const int32_t* __restrict__ prefix_len, const int32_t* __restrict__ assign_ord, const int32_t* __restrict__ slot_of,
    const int32_t* __restrict__ seed_rows, const int32_t* __restrict__ n_seeds, int32_t* merged_row, int32_t* merged_ord,
    int32_t* seg_row, int32_t* __restrict__ assign_out, int32_t* __restrict__ status) {
  using FL = FoldLane<T, D>;
  const FoldIo<T> io = {K, V, scores, in_count, K_out, V_out, out_mass, out_count, out_stride, B};
  // [seeds]: rows, slots, donors per seed, where a group starts, seeds with long groups; behind them
  // kFoldWaves cursors a seed, or the list in LDS
  extern __shared__ __attribute__((aligned(16))) int fold_mem[];
  __shared__ int wave_tot[3][kFoldWaves];
  __shared__ int n_long, longest;
  __shared__ union {
    typename FL::Share share[kFoldTeams];
    int rows[kFoldWaves][kWaveFoldMax];                    // the rows of the seed a wave folds
  } sh;
  int *const seed_row_l = fold_mem, *const slot_l = fold_mem + seeds, *const cnt_l = slot_l + seeds, *const start_l = cnt_l + seeds;
  int *const long_l = start_l + seeds, *const cursor = long_l + seeds;
  int* const list_row = cursor;
  int* const list_ord = cursor + kFoldList;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // (both kinds of workgroup run where their unit's selection and similarity did: what those wrote is in that L2)
  int u, f;
  if ((int)blockIdx.x >= n_fold) {
    const int wgs = (kp.B + kFoldWaves * kCopySlots - 1) / (kFoldWaves * kCopySlots);
    if (!map_block(n_units, wgs, u, f, (int)blockIdx.x - n_fold)) return;
    const int first = (f * kFoldWaves + wv) * kCopySlots;
    if (cj.lane_bytes == 16) copy_kept_rows<u32x4, 1, true>(cj, kp.B, row_off, u, first, lane);
    else if (cj.lane_bytes == 32) copy_kept_rows<u32x4, 2, true>(cj, kp.B, row_off, u, first, lane);
    else copy_kept_rows<u32x2, 1, true>(cj, kp.B, row_off, u, first, lane);
    return;
  }
  if (!map_block(n_units, shares, u, f)) return;
  const int lg = 31 - __clz(shares);
  const int64_t row0 = row_off[u];
  const int N = (int)(row_off[u + 1] - row0);
  const int P = prefix_len[u];
  const UnitPlan pl = make_plan(kp, P, N);
  const int hi = N - pl.r_eff;
  const int M = n_seeds[u], mine_n = M > f ? (M - f + shares - 1) >> lg : 0;  // own seeds: ordinals f, f + shares, ...
  const int32_t* ord_u = assign_ord + row0;

  const int first_row = P + wv * (64 * kFoldAhead) + lane;  // the thread's rows: 64 apart (the host checked that they cover the unit)
  int ord[kFoldAhead];
#pragma unroll
  for (int e = 0; e < kFoldAhead; ++e) ord[e] = first_row + e * 64 < hi ? ord_u[first_row + e * 64] : -1;  // (>= 0: a donor that folds)
  for (int l = tid; l < mine_n; l += kFoldThreads) {
    const int r = seed_rows[(size_t)u * kp.B + (l << lg) + f];
    seed_row_l[l] = r;
    slot_l[l] = slot_of[row0 + r];
    cnt_l[l] = 0;
  }
  if (tid == 0) n_long = longest = 0;

  // ---- the unit's donors: all that fold, those of the shares before this one (their entries come first in
  // the lists in memory), and this share's own
  const unsigned long long below = (1ull << lane) - 1ull;
  auto is_own = [&](int o) { return o >= 0 && (o & (shares - 1)) == f; };
  int all = 0, before = 0, own = 0, own_before = 0;
  int pos[kFoldAhead];
  {
    int a = 0, b = 0, c = 0;
#pragma unroll
    for (int e = 0; e < kFoldAhead; ++e) {
      const unsigned long long m = __ballot(is_own(ord[e]));
      pos[e] = c + __popcll(m & below);
      c += __popcll(m);
      a += __popcll(__ballot(ord[e] >= 0));
      b += __popcll(__ballot(ord[e] >= 0 && (ord[e] & (shares - 1)) < f));
      asm volatile("" : "+v"(pos[e]), "+v"(ord[e]));  // (final here: no ballots held across the barrier)
    }
    if (lane == 0) {
      wave_tot[0][wv] = a;
      wave_tot[1][wv] = b;
      wave_tot[2][wv] = c;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kFoldWaves; ++w) {
      all += wave_tot[0][w];
      before += wave_tot[1][w];
      own_before += w < wv ? wave_tot[2][w] : 0;
      own += wave_tot[2][w];
    }
  }
  if (f == 0 && tid == 0 && status && all == 0 && !(pl.status & (CASK_ST_IDENTITY | CASK_ST_PREFIX_BUDGET_EXHAUSTED)))
    status[u] = pl.status | CASK_ST_MERGE_INACTIVE;
  if (mine_n == 0) return;  // (the same in every thread)

  // ---- the share's list, ascending rows
  int32_t* const mrow = merged_row + row0 + before;
  int32_t* const mord = merged_ord + row0 + before;
  const bool in_lds = own <= kFoldList;
#pragma unroll
  for (int e = 0; e < kFoldAhead; ++e) {
    asm volatile("" : "+v"(ord[e]));
    if (!is_own(ord[e])) continue;
    const int i = first_row + e * 64, at = own_before + pos[e], l = ord[e] >> lg;
    if (in_lds) {
      list_row[at] = i;
      list_ord[at] = l;
    } else {
      mrow[at] = i;
      mord[at] = l;
    }
    atomicAdd(&cnt_l[l], 1);
  }
  __syncthreads();
  if (own > kWaveFoldMax) {
    for (int l = tid; l < mine_n; l += kFoldThreads)
      if (cnt_l[l] > kWaveFoldMax) atomicMax(&longest, cnt_l[l]);
    __syncthreads();
  }
  // What is left to do behind the folds (its stores would be waited for at their barriers): the donors'
  // assignments, and the seeds without donors, which pass through, sixteen lanes a row.
  auto rest = [&]() {
#pragma unroll
    for (int e = 0; e < kFoldAhead; ++e) {
      asm volatile("" : "+v"(ord[e]));
      if (assign_out && is_own(ord[e])) assign_out[row0 + first_row + e * 64] = slot_l[ord[e] >> lg];
    }
    const int gl = lane & 15;
    for (int l = tid >> 4; l < mine_n; l += kFoldThreads / 16) {
      if (cnt_l[l] != 0) continue;
      const int64_t row = row0 + seed_row_l[l];
      const int slot = slot_l[l];
      const size_t from = (size_t)row * D + gl * FL::EPL, to = ((size_t)u * io.out_stride + slot) * D + gl * FL::EPL;
      const typename FL::Words k = *reinterpret_cast<const typename FL::Words*>(io.K + from);
      const typename FL::Words v = *reinterpret_cast<const typename FL::Words*>(io.V + from);
      *reinterpret_cast<typename FL::Words*>(io.K_out + to) = k;
      *reinterpret_cast<typename FL::Words*>(io.V_out + to) = v;
      if (gl == 0 && io.out_mass) io.out_mass[(size_t)u * io.B + slot] = io.scores[row];
      if (gl == 0 && io.out_count) io.out_count[(size_t)u * io.B + slot] = io.in_count ? io.in_count[row] : 1;
    }
  };
  if (own == 0) {
    rest();
    return;
  }
  auto fold_by_wave = [&](int l, int s0, int s1, auto row_at) {
    fold_group<T, D, 4, false>(io, u, row0, seed_row_l[l], slot_l[l], s0, s1, lane >> 4, 0, true, row_at, nullptr);
  };
  if (in_lds && longest == 0) {
    for (int l = wv; l < mine_n; l += kFoldWaves) {
      const int n = cnt_l[l];
      if (n == 0) continue;
      int have = 0;
      for (int k = 0; k < own && have < n; k += 64) {
        const bool m = k + lane < own && list_ord[k + lane] == l;
        const unsigned long long b = __ballot(m);
        if (m) sh.rows[wv][have + __popcll(b & ((1ull << lane) - 1ull))] = list_row[k + lane];
        have += __popcll(b);
      }
      asm volatile("" ::: "memory");  // (the wave's own LDS accesses stay in order)
      fold_by_wave(l, 0, n, [&](int k) { return sh.rows[wv][k]; });
      asm volatile("" ::: "memory");
    }
    rest();
    return;
  }

  // ---- a long list, or a seed with many donors: split by seed in memory
  int32_t* const seg = seg_row + row0 + before;
  if (in_lds) {  // (the cursors take the list's place)
    int r[kFoldList / kFoldThreads], o[kFoldList / kFoldThreads];
#pragma unroll
    for (int q = 0; q < kFoldList / kFoldThreads; ++q) {
      const int k = q * kFoldThreads + tid;
      r[q] = k < own ? list_row[k] : 0;
      o[q] = k < own ? list_ord[k] : 0;
    }
#pragma unroll
    for (int q = 0; q < kFoldList / kFoldThreads; ++q) {
      const int k = q * kFoldThreads + tid;
      if (k < own) {
        mrow[k] = r[q];
        mord[k] = o[q];
      }
    }
    __syncthreads();
  }
  for (int k = tid; k < kFoldWaves * seeds; k += kFoldThreads) cursor[k] = 0;
  __syncthreads();  // (also: the list in memory is read by other threads below)
  const int run = (own + kFoldThreads - 1) / kFoldThreads * 64;
  const int c0 = min(own, wv * run), c1 = min(own, c0 + run);
  int* const my_cursor = cursor + wv * seeds;
  for (int k = c0 + lane; k < c1; k += 64) atomicAdd(&my_cursor[mord[k]], 1);
  if (wv == 0) {  // starts of the groups
    int carry = 0;
    for (int l0 = 0; l0 < mine_n; l0 += 64) {
      const int v = l0 + lane < mine_n ? cnt_l[l0 + lane] : 0;
      int incl = v;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      if (l0 + lane < mine_n) start_l[l0 + lane] = carry + incl - v;
      carry += __shfl(incl, 63, 64);
    }
  }
  __syncthreads();
  for (int l = tid; l < mine_n; l += kFoldThreads) {
    int at = start_l[l];
    for (int w = 0; w < kFoldWaves; ++w) {
      const int t = cursor[w * seeds + l];
      cursor[w * seeds + l] = at;
      at += t;
    }
    if (cnt_l[l] > kWaveFoldMax) long_l[atomicAdd(&n_long, 1)] = l;  // (their order does not reach the results)
  }
  __syncthreads();
  int nbits = 1;
  while ((1 << nbits) < mine_n) ++nbits;
  constexpr int kAhead = 4;  // 64-entry steps whose loads are in flight together
  for (int i0 = c0; i0 < c1; i0 += 64 * kAhead) {
    int os[kAhead], rs[kAhead];
#pragma unroll
    for (int e = 0; e < kAhead; ++e) {
      const int idx = min(i0 + e * 64 + lane, c1 - 1);  // clamped: no branch around the loads
      os[e] = mord[idx];
      rs[e] = mrow[idx];
    }
#pragma unroll
    for (int e = 0; e < kAhead; ++e) {
      const bool valid = i0 + e * 64 + lane < c1;
      unsigned long long same = __ballot(valid);
      for (int bit = 0; bit < nbits; ++bit) {
        const bool one = ((os[e] >> bit) & 1) != 0;
        const unsigned long long ones = __ballot(valid && one);
        same &= one ? ones : ~ones;
      }
      if (valid) {  // `same`: the valid lanes with this lane's seed
        const int rank = __popcll(same & ((1ull << lane) - 1ull));
        const int cur = my_cursor[os[e]];
        seg[cur + rank] = rs[e];
        if (rank == __popcll(same) - 1) my_cursor[os[e]] = cur + rank + 1;  // (after every lane's read)
      }
    }
  }
  __syncthreads();  // the groups in memory are read by other threads below
  for (int l = wv; l < mine_n; l += kFoldWaves)
    if (cnt_l[l] > 0 && cnt_l[l] <= kWaveFoldMax) fold_by_wave(l, start_l[l], start_l[l] + cnt_l[l], [&](int k) { return seg[k]; });
  __syncthreads();
  const int nl = n_long, team = wv >> 2, w4 = wv & 3;
  for (int k0 = 0; k0 < nl; k0 += kFoldTeams) {
    const bool live = k0 + team < nl;
    const int l = long_l[live ? k0 + team : k0];
    const int s0 = start_l[l], s1 = live ? s0 + cnt_l[l] : s0;
    fold_group<T, D, 16, true>(io, u, row0, seed_row_l[l], slot_l[l], s0, s1, w4 * 4 + (lane >> 4), w4, live,
                               [&](int k) { return seg[k]; }, &sh.share[team]);
  }
  rest();
}

// ------------------------------------------------------------------ dispersion and lost mass

// Perturbation diagnostics of a finished event (Section 2.6, Appendix B).  One workgroup per
// unit; sixteen lanes per row (lanes 0-7 hold the first half of the channels, lanes 8-15 the
// second, so a band's two channels sit eight lanes apart).  The sums are kept in double; the 64
// group sums are added in order by one thread.
// Bound: round trips to memory.  A thread takes the assignment and score of kDiagRows rows at once
// (1024 apart); the rows that went to a slot are listed in LDS in ascending order, and the 64 groups take
// the list in turn, several rows in flight each.  With a group per row, one row at a time, the walk
// was a chain of N / 64 x 2 trips: 46 us on 56 units of 6256 rows, 12.6 on 27 of 735; with every
// wave handing its own 64 rows to its four groups, whose longest chain is the always-kept tail's, 26.6 and
// 17.0; with the list 13.8 and 12.0.
constexpr int kDiagRows = 8;
template <typename T, int D>
__global__ __launch_bounds__(1024) void group_diag_kernel(
    KParams kp, const int64_t* __restrict__ row_off, const T* __restrict__ K,
    const float* __restrict__ scores, const int32_t* __restrict__ assign,
    const T* __restrict__ K_out, int out_stride, float* __restrict__ dispersion,
    float* __restrict__ lost_mass) {
  constexpr int EPL = D / 16;
  constexpr int WORDS = EPL * sizeof(T) / 4;
  struct alignas(WORDS * 4 > 16 ? 16 : WORDS * 4) Raw { uint32_t w[WORDS]; };
  constexpr int kAhead = sizeof(T) == 2 ? 4 : 2;  // rows of a group in flight
  __shared__ double part_d[64], part_l[64];
  __shared__ int slot_l[1024 * kDiagRows];         // the listed rows' slots
  __shared__ uint16_t row_l[1024 * kDiagRows];     // their rows, from the round's first
  __shared__ int count_l[16 * kDiagRows];          // rows listed per 64 of the round
  const int u = blockIdx.x, tid = threadIdx.x, grp = tid >> 4, gl = tid & 15;
  const int64_t row0 = row_off[u];
  const int N = (int)(row_off[u + 1] - row0);
  float w[EPL];
#pragma unroll
  for (int e = 0; e < EPL; ++e) w[e] = kp.band_w ? kp.band_w[(gl & 7) * EPL + e] : 1.f;
  double disp = 0.0, lost = 0.0;
  const int lane = tid & 63, wv = tid >> 6;
  int t[kDiagRows];
  float a[kDiagRows];
  auto fetch = [&](int c0) {
#pragma unroll
    for (int q = 0; q < kDiagRows; ++q) {
      const int i = c0 + q * 1024 + tid;
      t[q] = i < N ? assign[row0 + i] : kp.B;
      a[q] = i < N ? scores[row0 + i] : 0.f;
    }
  };
  fetch(0);
  for (int c0 = 0; c0 < N; c0 += 1024 * kDiagRows) {
    unsigned long long listed[kDiagRows];
#pragma unroll
    for (int q = 0; q < kDiagRows; ++q) {
      if (t[q] < 0) lost += (double)a[q];
      listed[q] = __ballot(t[q] >= 0 && t[q] < kp.B);
      if (lane == 0) count_l[q * 16 + wv] = __popcll(listed[q]);
    }
    __syncthreads();  // (also: the list of the round before has been read)
    static_assert(kDiagRows == 8, "two counts per lane");
    int c_lo = count_l[lane], c_hi = count_l[64 + lane];
    const int own_lo = c_lo, own_hi = c_hi;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_up(c_lo, o, 64), y = __shfl_up(c_hi, o, 64);
      if (lane >= o) c_lo += x, c_hi += y;
    }
    const int half = __shfl(c_lo, 63, 64), total = half + __shfl(c_hi, 63, 64);
    c_lo -= own_lo;
    c_hi += half - own_hi;
#pragma unroll
    for (int q = 0; q < kDiagRows; ++q) {
      const int first = __shfl(q < 4 ? c_lo : c_hi, (q & 3) * 16 + wv, 64);
      if ((listed[q] >> lane) & 1ull) {
        const int at = first + __popcll(listed[q] & ((1ull << lane) - 1ull));
        slot_l[at] = t[q];
        row_l[at] = (uint16_t)(q * 1024 + tid);
      }
    }
    if (c0 + 1024 * kDiagRows < N) fetch(c0 + 1024 * kDiagRows);  // on its way while the list is taken
    __syncthreads();
    for (int e0 = grp; e0 < total; e0 += 64 * kAhead) {
      Raw kr[kAhead], rr[kAhead];
      float ar[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {  // (past the end the last row is read again)
        const int e = min(e0 + k * 64, total - 1);
        const int64_t row = row0 + c0 + row_l[e];
        kr[k] = *reinterpret_cast<const Raw*>(K + (size_t)row * D + gl * EPL);
        rr[k] = *reinterpret_cast<const Raw*>(K_out + ((size_t)u * out_stride + slot_l[e]) * D + gl * EPL);
        ar[k] = scores[row];
      }
#pragma unroll
      for (int k = 0; k < kAhead; ++k) {
        const T* kp_ = reinterpret_cast<const T*>(&kr[k]);
        const T* rp_ = reinterpret_cast<const T*>(&rr[k]);
        float r = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) {
          const float x = Elem<T>::load(kp_ + e) - Elem<T>::load(rp_ + e);
          const float sq = x * x;
          const float other = __shfl_xor(sq, 8, 64);  // the band's other channel
          r = __builtin_fmaf(w[e], __builtin_amdgcn_sqrtf(sq + other), r);
        }
        if (gl >= 8) r = 0.f;  // both halves computed the same bands
#pragma unroll
        for (int o = 4; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
        if (e0 + k * 64 < total) disp += (double)ar[k] * (double)r;
      }
    }
  }
  // a thread's own share of the lost mass -> its group
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) lost += __shfl_xor(lost, o, 64);
  if (gl == 0) {
    part_d[grp] = disp;
    part_l[grp] = lost;
  }
  __syncthreads();
  if (tid == 0) {
    double sd = 0.0, sl = 0.0;
    for (int g = 0; g < 64; ++g) {
      sd += part_d[g];
      sl += part_l[g];
    }
    dispersion[u] = (float)sd;
    lost_mass[u] = (float)sl;
  }
}

template <int D>
hipError_t launch_similarity_f32(const KParams& kp, const Batch& b, const uint8_t* role,
                                 const int32_t* seed_rows, const int32_t* n_seeds, int32_t* assign_ord,
                                 bool roles_follow_plan, hipStream_t st) {
  using SG = SimF32Geom<D>;
  const int tiles = (b.max_decode_len + SG::kDonorTile - 1) / SG::kDonorTile;
  if (tiles == 0) return hipSuccess;
  // chunks of a unit as for bf16 caches; beyond kF32Slots units pieces of about 32 tiles
  int chunks = b.n_units > 0 ? kF32Slots / b.n_units : 1;
  if (chunks < 1) chunks = (tiles + 31) / 32;
  if (chunks > tiles) chunks = tiles;
  const bool one = roles_follow_plan && plan_seed_bound(kp) <= SG::kSeeds;
  int tiles_per_wg = (tiles + chunks - 1) / chunks;
  if (!one && tiles_per_wg > kMultiTiles) tiles_per_wg = kMultiTiles;
  chunks = (tiles + tiles_per_wg - 1) / tiles_per_wg;
  auto kern = kp.radius > 0 ? (one ? &similarity_f32_kernel<D, true, true> : &similarity_f32_kernel<D, false, true>)
                            : (one ? &similarity_f32_kernel<D, true, false> : &similarity_f32_kernel<D, false, false>);
  kern<<<dim3(mapped_blocks(b.n_units, chunks)), dim3(256), 0, st>>>(kp, b.n_units, chunks, tiles_per_wg, b.row_off, b.prefix_len,
                                                    static_cast<const float*>(b.K), role, seed_rows, n_seeds, assign_ord);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_similarity(const KParams& kp, const Batch& b, const uint8_t* role,
                             const int32_t* seed_rows, const int32_t* n_seeds,
                             int32_t* assign_ord, bool roles_follow_plan, hipStream_t st) {
  if (kp.geometry == 1) {
    if (kp.dtype == CASK_F32)
      return kp.d == 64 ? launch_similarity_kappa<float, 64>(kp, b, role, seed_rows, n_seeds, assign_ord, st)
                        : launch_similarity_kappa<float, 128>(kp, b, role, seed_rows, n_seeds, assign_ord, st);
    return kp.d == 64 ? launch_similarity_kappa<uint16_t, 64>(kp, b, role, seed_rows, n_seeds, assign_ord, st)
                      : launch_similarity_kappa<uint16_t, 128>(kp, b, role, seed_rows, n_seeds, assign_ord, st);
  }
  if (kp.dtype == CASK_BF16) {
    // a few workgroups per unit, about two per compute unit in all, each walking its share of
    // the unit's donor tiles
    const int tiles = (b.max_decode_len + kDonorTile - 1) / kDonorTile;
    if (tiles == 0) return hipSuccess;
    // (with more units than workgroup slots, units of different length would leave the longest
    // ones running alone at the end: cut them into pieces of about 32 tiles instead)
    int chunks = b.n_units > 0 ? 512 / b.n_units : 1;
    if (chunks < 1) chunks = (tiles + 31) / 32;
    if (chunks < 1) chunks = 1;
    if (chunks > tiles) chunks = tiles;
    const int seed_bound = plan_seed_bound(kp);
    // (a caller-supplied role array may name any number of seeds: general kernel then)
    const bool one = roles_follow_plan && seed_bound <= kSeedBlock;
    int tiles_per_wg = (tiles + chunks - 1) / chunks;
    if (!one && tiles_per_wg > kMultiTiles) tiles_per_wg = kMultiTiles;  // its tiles' results wait in registers
    chunks = (tiles + tiles_per_wg - 1) / tiles_per_wg;
#define CASK_SIM(D, ONE, RAD)                                                          \
  similarity_mfma_kernel<D, ONE, RAD><<<dim3(mapped_blocks(b.n_units, chunks)), dim3(256), 0, st>>>(    \
      kp, b.n_units, chunks, tiles_per_wg, b.row_off, b.prefix_len,                    \
      static_cast<const uint16_t*>(b.K), role, seed_rows, n_seeds, assign_ord)
#define CASK_SIM_D(D)                                                        \
  if (kp.radius > 0) {                                                       \
    if (one) CASK_SIM(D, true, true); else CASK_SIM(D, false, true);         \
  } else {                                                                   \
    if (one) CASK_SIM(D, true, false); else CASK_SIM(D, false, false);       \
  }
    if (kp.d == 64) { CASK_SIM_D(64) } else { CASK_SIM_D(128) }
#undef CASK_SIM_D
#undef CASK_SIM
    return hipGetLastError();
  }
  return kp.d == 64 ? launch_similarity_f32<64>(kp, b, role, seed_rows, n_seeds, assign_ord, roles_follow_plan, st)
                    : launch_similarity_f32<128>(kp, b, role, seed_rows, n_seeds, assign_ord, roles_follow_plan, st);
}

hipError_t launch_gather_merged(const KParams& kp, const Batch& b,
                                const int32_t* assign_ord, const int32_t* slot_of,
                                const int32_t* seed_rows, int32_t* merged_row, int32_t* merged_ord,
                                int32_t* n_merged, int32_t* assign_out, int assign_mode,
                                int32_t* status, const int32_t* n_seeds, int32_t* seg_row,
                                int32_t* seg_start, const CopyJob* copy, hipStream_t st) {
  static_assert((kGatherThreads / 64 & (kGatherThreads / 64 - 1)) == 0, "waves per block: a power of two");
  CopyJob cj{};
  long long copy_blocks = 0;
  if (copy && copy->K_out) {
    cj = *copy;
    cj.n_units = b.n_units;
    cj.lane_bytes = kp.d * (kp.dtype == CASK_F32 ? 4 : 2) / 16;
    const long long waves = (long long)b.n_units * ((kp.B + kCopySlots - 1) / kCopySlots);
    copy_blocks = (waves + kGatherThreads / 64 - 1) / (kGatherThreads / 64);
    if (b.n_units + copy_blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  }
  // the smallest instance whose chunk covers the longest decode trace: a unit that fits one chunk
  // is then shared by all of the workgroup's waves, not by the first few
  const int per_need = (b.max_decode_len + kGatherThreads - 1) / kGatherThreads;
  auto kern = per_need <= 4 ? &gather_merged_kernel<4>
                            : (per_need <= 8 ? &gather_merged_kernel<8> : &gather_merged_kernel<kGatherPer>);
  kern<<<dim3((unsigned)(b.n_units + copy_blocks)), dim3(kGatherThreads), 0, st>>>(
      kp, b.n_units, cj, b.row_off, b.prefix_len, assign_ord, slot_of, seed_rows, merged_row, merged_ord,
      n_merged, assign_out, assign_mode, status, n_seeds, seg_row, seg_start);
  return hipGetLastError();
}

hipError_t launch_group_diag(const KParams& kp, const Batch& b, const float* scores,
                             const int32_t* assign, const void* K_out, int out_stride,
                             float* dispersion, float* lost_mass, hipStream_t st) {
#define CASK_GD(T, D)                                                                     \
  group_diag_kernel<T, D><<<dim3(b.n_units), dim3(1024), 0, st>>>(                        \
      kp, b.row_off, static_cast<const T*>(b.K), scores, assign, static_cast<const T*>(K_out), \
      out_stride, dispersion, lost_mass)
  if (kp.dtype == CASK_F32) {
    if (kp.d == 64) CASK_GD(float, 64); else CASK_GD(float, 128);
  } else {
    if (kp.d == 64) CASK_GD(uint16_t, 64); else CASK_GD(uint16_t, 128);
  }
#undef CASK_GD
  return hipGetLastError();
}

hipError_t launch_emit(const KParams& kp, const Batch& b, const int32_t* seed_rows, const int32_t* n_seeds,
                       const int32_t* slot_of, const int32_t* seg_row, const int32_t* seg_start,
                       const int32_t* n_merged, const CopyJob& cj, hipStream_t st) {
#define CASK_EMIT(T, D) launch_emit_t<T, D>(kp, b, seed_rows, n_seeds, slot_of, seg_row, seg_start, n_merged, cj, st)
  if (kp.dtype == CASK_F32) return kp.d == 64 ? CASK_EMIT(float, 64) : CASK_EMIT(float, 128);
  return kp.d == 64 ? CASK_EMIT(uint16_t, 64) : CASK_EMIT(uint16_t, 128);
#undef CASK_EMIT
}

// A workgroup reads a whole unit's assignments: one chunk of them (8192 rows) is one trip to memory, two
// would be four, counted and then listed (event on 112 units of 33 024 rows 0.5 % slower than in two launches).
// Beyond 256 units the two launches fill the chip by themselves: one share a unit is 2 % faster on 600 units of
// 2000 rows but 3 % slower where every donor folds, two shares are up to 3 % slower.
bool group_fold_fits(const KParams& kp, const Batch& b) {
  return b.n_units <= 256 && plan_seed_bound(kp) <= kFoldSeeds && b.max_decode_len <= kFoldThreads * kFoldAhead;
}

hipError_t launch_group_fold(const KParams& kp, const Batch& b, const uint8_t* role, const int32_t* assign_ord,
                             const int32_t* slot_of, const int32_t* seed_rows, const int32_t* n_seeds, int32_t* merged_row,
                             int32_t* merged_ord, int32_t* seg_row, int32_t* assign_out, int32_t* status, const CopyJob& copy,
                             hipStream_t st) {
  if (!group_fold_fits(kp, b)) return hipErrorInvalidValue;
  int shares = 2;  // of a unit: about two workgroups to a compute unit in all, two to eight
  while (shares < 8 && (long long)b.n_units * shares * 2 <= 512) shares *= 2;
  CopyJob cj = copy;
  cj.role = role;
  cj.lane_bytes = kp.d * (kp.dtype == CASK_F32 ? 4 : 2) / 16;
  const int wgs = (kp.B + kFoldWaves * kCopySlots - 1) / (kFoldWaves * kCopySlots);  // a unit's copying workgroups
  if ((long long)b.n_units * (wgs + shares) + 16 > 0x7fffffffLL) return hipErrorInvalidValue;
  const int folds = mapped_blocks(b.n_units, shares), blocks = folds + mapped_blocks(b.n_units, wgs);
  const int seeds = (plan_seed_bound(kp) + shares - 1) / shares;  // of a share
  // at most 512 seeds a share, 27 KB: with the 17 KB of the other arrays well below the 64 KB that any launch may take
  const size_t lds = ((size_t)5 * seeds + (kFoldWaves * seeds > 2 * kFoldList ? kFoldWaves * seeds : 2 * kFoldList)) * sizeof(int);
  auto go = [&](auto t, auto d) {
    using T = decltype(t);
    group_fold_kernel<T, decltype(d)::value><<<dim3((unsigned)blocks), dim3(kFoldThreads), lds, st>>>(
        kp, CASK_FOLD_PASS(T), b.n_units, (int)folds, shares, seeds, cj, b.row_off, b.prefix_len, assign_ord, slot_of, seed_rows, n_seeds,
        merged_row, merged_ord, seg_row, assign_out, status);
    return hipGetLastError();
  };
  const std::integral_constant<int, 64> d64;
  const std::integral_constant<int, 128> d128;
  if (kp.dtype == CASK_F32) return kp.d == 64 ? go(float(), d64) : go(float(), d128);
  return kp.d == 64 ? go(uint16_t(), d64) : go(uint16_t(), d128);
}

}  // namespace cask
