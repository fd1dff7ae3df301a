// Scoring: s_j = mean over the W*G window rows of softmax_j(scale <q, k_j>), the scalar
// importance used as local score mass a_i (Sections 1 and 2.4 of the paper).
//
// The softmax normaliser of a row needs all keys before any column can be summed, so the
// score takes two sweeps of Q.K^T:
//   sweep A (row statistics)  per window row and key split: a reference logit and the sum of
//                             exp2 against it (pairs of splits combine exactly);
//   sweep B (column mass)     per key: sum over window rows of exp2(logit - L_row).
// Logits are never stored: recomputing the contraction on the matrix cores is cheaper than
// writing and re-reading a W*G x N fp32 matrix through HBM.
//
// bf16: both sweeps use one MFMA kernel (32x32x16 bf16 tiles, fp32 accumulation).
// One operand ("resident") stays in registers for the whole loop, the other ("stream") is
// staged through LDS.  The product tile is stream x resident^T, so each lane owns ONE
// resident column and 16 stream rows: the reduction over the stream dimension (keys in
// sweep A, window rows in sweep B) stays inside a lane until the very end.
// fp32 caches take a simpler kernel of the same structure, their values split into three bf16 terms.
// Few short bf16 units take one sweep that keeps its logits in registers (score_short_kernel).
#include "cask_common.h"

namespace cask {

#define CASK_INLINE __attribute__((always_inline))

namespace {

constexpr float kNegInf = -__builtin_inff();

// Most a lane's sum against its fixed reference may reach; beyond, the wave takes its share again with a
// running maximum.  Short of the fp32 range by more than the sums of 2 lanes and 64 splits can add up to.
constexpr float kMostSum = 0x1p120f;

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// (m, l) <- combination of two partial softmax statistics in base-2 units.  REF: the m are references that
// a sum may lie far above, not maxima.
template <bool REF>
__device__ inline void ml_combine(float& m, float& l, float m2, float l2) {
  const float M = fmaxf(m, m2);
  float a = (m == kNegInf) ? 0.f : fast_exp2(m - M);
  float b = (m2 == kNegInf) ? 0.f : fast_exp2(m2 - M);
  if (REF) {
    // Far apart, 2^e of the lower one by itself would be zero, and its sum may make up for it (further apart than
    // 2 x 126 octaves nothing is left: a reference is at most 16 above a logit of its own).  (Rare, and out of
    // the chain: event on 6 units of up to 25 900 rows 73.3 -> 71.9 us.)
    const float apart = __builtin_fabsf(m - m2);
    const bool far = apart > 64.f && apart < __builtin_inff();
    if (__builtin_amdgcn_ballot_w64(far) != 0ull) {
      const float half = fast_exp2(-0.5f * apart);
      if (far && m < m2) l *= half, a = half;
      if (far && m2 < m) l2 *= half, b = half;
    }
  }
  l = __builtin_fmaf(l, a, l2 * b);
  m = M;
}

// ------------------------------------------------------------------ MFMA path (bf16)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;                    // waves per workgroup, 1 per SIMD; two workgroups share a CU
constexpr int kThreads = kWaves * 64;
constexpr int kResRows = kWaves * 64;        // resident rows per workgroup (64 per wave)
constexpr int kStageRows = 64;               // stream rows per ring slot
constexpr int kDepth = 4;                    // ring slots: loads run kDepth - 1 stages ahead

// What the head dimension decides about a ring slot (see the stage layout below).
template <int D>
struct StageGeom {
  static constexpr int kRowBytes = D * 2;
  static constexpr int kGroupRows = 1024 / kRowBytes;            // rows one load instruction of a wave lands: 4 or 8
  static constexpr int kGroupPitch = 1024 + kGroupRows * 16;     // LDS pitch of such a group
  static constexpr int kDataBytes = (kStageRows / kGroupRows) * kGroupPitch;
  static constexpr int kStageBytes = kDataBytes + kStageRows * 4;  // + one float per row: -L_row (sweep B)
  static constexpr int kLoadsPerThread = kStageRows * (kRowBytes / 16) / kThreads;  // 16-byte pieces per thread per stage
  static constexpr int kStepBytes = 2 * kGroupRows * 16;         // LDS distance of two k-steps of a row
  static constexpr int kTileBytes = (32 / kGroupRows) * kGroupPitch;  // LDS distance of the two tile rows of a stage
};

// Pad value of -L for window rows past W*G: far enough down that exp2 flushes to zero.
constexpr float kPadNegL = -1.0e30f;

// Per window row of a unit: -L_row, L_row the base-2 log-sum-exp combined over the key splits
// of sweep A.  Sweep B adds it to every logit of the row inside the exponent's fma.
constexpr int kBiasThreads = 1024;  // a thread per window row at W*G <= 1024: every partial of the unit in flight at once
__global__ __launch_bounds__(kBiasThreads) void score_bias_kernel(KParams kp, int n_splits, int mq_pad,
                                                         const float2* __restrict__ rowstat,
                                                         float* __restrict__ bias) {
  const int unit = blockIdx.x;
  const float2* part = rowstat + (size_t)unit * n_splits * mq_pad;
  for (int r = threadIdx.x; r < mq_pad; r += kBiasThreads) {
    float nl = kPadNegL;
    if (r < kp.Mq) {
      float m = kNegInf, l = 0.f;
      for (int s0 = 0; s0 < n_splits; s0 += 8) {  // eight partials in flight, combined in order
        float2 pr[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) pr[e] = part[(size_t)min(s0 + e, n_splits - 1) * mq_pad + r];
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (s0 + e < n_splits) ml_combine<true>(m, l, pr[e].x, pr[e].y);
      }
      nl = -(m + log2f(l));
    }
    bias[(size_t)unit * mq_pad + r] = nl;
  }
}

// Both scoring sweeps.  MODE 0 = sweep A (resident: window rows, stream: keys),
// MODE 1 = sweep B (resident: keys, stream: window rows).
//
// Workgroup: 4 waves, one per SIMD, and two workgroups per compute unit, so a SIMD always has a
// second wave from an independent workgroup to run while the first sits in its prologue or at
// a barrier.  Wave w keeps CT resident tiles of 32 rows (rows [32 CT w, 32 CT (w + 1)) of the
// workgroup's 128 CT) as MFMA B-operands in registers: CT = 2 in the narrow form, CT = 4 in the
// wide form that the two separate sweeps take where the shape fills such blocks (every stream
// operand read from LDS then serves four products instead of two; see pipelined_wide below).
// Stream rows arrive 64 at a time in a ring of LDS slots,
// written by direct global->LDS loads (no register staging, no LDS stores) that run
// kDepth - 1 stages ahead of the stage being consumed; one barrier per stage both publishes a
// slot and frees the one consumed before it.
//
// Stage layout in LDS: each load instruction of a wave lands 1 KB = R = four 256-byte rows (d =
// 128) or eight 128-byte rows (d = 64); lane s fetches 16-byte piece s / R of row s % R, so the
// group holds piece-major data (piece g of row r at (g R + r) * 16).  A wave reading A-operands
// (lane = row) then touches 16 consecutive bytes per row and groups 1024 + 16 R bytes apart: any
// sixteen consecutive lanes cover all banks once, and the k-steps are plain immediate offsets
// (32 R bytes apart).
//
// Per stage a wave runs 2 CT tiles of 32x32, (rt0,ct0) ... (rt0,ct CT-1) (rt1,ct0) ...,
// software-pipelined: the MFMA chain of a tile is issued interleaved, two logits per MFMA, with
// the exp2 epilogue of the tile before it, so the matrix cores and the vector ALU of a wave
// run at the same time; the epilogue of a stage's last tile rides on the next stage's first
// chain.  The epilogue is exactly three vector instructions per logit:
//   sweep A  fma, exp2, add: no running maximum in the loop -- exp2 is taken against a per-lane
//            reference (from the first logits of the lane's row), which is exact as long as the sum
//            stays finite, because (reference, sum) pairs combine exactly.  A sum that left the
//            fp32 range (a logit more than ~128 binary orders above the reference) shows as
//            inf at the end; the wave then recomputes its share with a true running maximum,
//            operands straight from memory (rare, slow, exact);
//   sweep B  fma, exp2, add: the fma adds -L_row, read from LDS next to the stage's rows (a lane's
//            16 rows of a tile are four float4 reads).
// With d = 64 a tile is a chain of four MFMA instead of eight under the same 48 vector instructions:
// the vector issue is the bound there (256 of 288 cycles a tile), and two pieces of the epilogue
// ride on each MFMA.
// Stages that touch masked entries (causal tail, ragged end, keys inside the window) run the same
// pipeline with two more instructions per logit (a compare of the logit's constant row offset
// with a per-lane limit, a select); only a sweep-A workgroup without a single clean stage, which
// has no reference logit yet, takes a plain unpipelined path with a true running maximum.
template <int D, int MODE, int CT = 2, bool RING_RES = false>
__global__ __launch_bounds__(kThreads, 2) void score_mfma_kernel(
    KParams kp, int n_units, int tiles_per_unit, int n_splits, int split_len, int q_splits, int mq_pad,
    const int64_t* __restrict__ row_off, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ Q, float2* __restrict__ rowstat,
    const float* __restrict__ bias, float* __restrict__ bias_out, float* __restrict__ scores,
    float* __restrict__ parts, int part_pitch) {
  using SG = StageGeom<D>;
  constexpr int kRowBytes = SG::kRowBytes, kGroupRows = SG::kGroupRows, kGroupPitch = SG::kGroupPitch;
  constexpr int kDataBytes = SG::kDataBytes, kStageBytes = SG::kStageBytes, kLoadsPerThread = SG::kLoadsPerThread;
  constexpr int kStepBytes = SG::kStepBytes, kTileBytes = SG::kTileBytes;
  constexpr int NK = D / 16;   // k-steps per tile
  constexpr int NP = 8 / NK;   // epilogue pieces (two logits each) that ride on one k-step
  // MODE 2 = both sweeps in one launch for short units (one key split): the first pass is
  // MODE 0; the second keeps the same resident window rows and streams the keys again, leaving
  // one partial column sum per wave.  MODE 3 = the same for units of any length when W*G <= 512
  // (at most two row blocks per unit): the four waves' column sums are added in LDS in wave
  // order and leave the workgroup as one addend per key -- stored when the unit has one row
  // block, added atomically onto scores cleared beforehand when it has two (two addends onto
  // zero: the order cannot change the bits).
  // CT = resident 32-row tiles per wave: 2 (64 rows a wave, 256 a workgroup) or 4 (128 / 512:
  // every stream operand read from LDS then serves four products instead of two)
  constexpr int kWaveRows = CT * 32;
  constexpr int kResRowsT = kWaves * kWaveRows;
  // RING_RES: the resident rows come through the ring as well, in kResStages ring stages ahead
  // of the stream (else they are loaded straight into registers and the ring starts with the stream)
  constexpr int kResStages = RING_RES ? kResRowsT / kStageRows : 0;
  constexpr bool kRowPass = MODE != 1;
  constexpr bool kTwoPass = MODE >= 2;
  constexpr bool kWgReduce = MODE == 3;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* ring = smem;

  int unit, tile;
  if (!map_block(n_units, tiles_per_unit, unit, tile)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c32 = lane & 31, h = lane >> 5;
  const int64_t row0 = row_off[unit];
  const int N = (int)(row_off[unit + 1] - row0);
  const int Mq = kp.Mq, W = kp.W, Gq = kp.G;
  const float c = kp.scale_log2;
  const uint16_t* Ku = K + (size_t)row0 * D;
  const uint16_t* Qu = Q + (size_t)unit * Mq * D;

  // ---- what this workgroup covers
  const uint16_t* res_ptr;
  const uint16_t* str_ptr;
  int res_base, res_limit, s_begin, s_end;  // resident rows [res_base, ..), stream rows [s_begin, s_end)
  int split = 0;
  if (kRowPass) {
    const int qb = tile / n_splits;
    split = turned(unit, tile % n_splits, n_splits);
    res_base = qb * kResRowsT;
    if (res_base >= Mq) return;
    res_ptr = Qu;
    res_limit = Mq;
    str_ptr = Ku;
    s_begin = split * split_len;
    s_end = min(N, s_begin + split_len);
    if (kp.causal) {  // (MODE 2: the keys cut here get zeros as their partial sums at the end)
      const int last_row = min(Mq, res_base + kResRowsT) - 1;
      s_end = min(s_end, N - W + last_row / Gq + 1);
    }
  } else {
    // a unit's last tile first: its waves run the masked path and take longest
    const int key_tiles = tiles_per_unit / q_splits;
    res_base = (key_tiles - 1 - tile / q_splits) * kResRowsT;
    if (res_base >= N) return;
    res_ptr = Ku;
    res_limit = N;
    str_ptr = Qu;
    s_begin = 0;
    s_end = Mq;
    if (q_splits == 2) {  // this workgroup's half of the window rows, whole stages
      const int half = ((Mq + 2 * kStageRows - 1) / (2 * kStageRows)) * kStageRows;
      if (tile & 1) s_begin = half; else s_end = min(Mq, half);
    }
    if (kp.causal && res_base > N - W)
      s_begin = max(s_begin, (((res_base - (N - W)) * Gq) / kStageRows) * kStageRows);
  }
  const int n_stages = s_end > s_begin ? (s_end - s_begin + kStageRows - 1) / kStageRows : 0;
  if (MODE == 0 && q_splits == 2 && tile == 0) {
    // sweep B will add two partial sums per key: clear the unit's scores here
    for (int i = tid; i < N; i += kThreads) scores[row0 + i] = 0.f;
  }

  // ---- ring loads: thread t, piece j covers 16-byte LDS slot t + kThreads * j of the stage:
  //      row = kGroupRows * (slot / 64) + slot % kGroupRows, 16-byte piece = (slot % 64) / kGroupRows
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(str_ptr), 0,
                                        max(s_end, 0) * kRowBytes, 0x00020000);
  // (load j of a wave fills group wv + kWaves * j: the same lane offset, kWaves KB of rows on)
  const int ld_voff = (wv * kGroupRows + lane % kGroupRows) * kRowBytes + (lane / kGroupRows) * 16;
  // sweep B: the -L_row of a stage's 64 rows is one more 256-byte load, taken in turn by the
  // waves (stage % kWaves), so every wave has at most one extra load in flight
  const __amdgpu_buffer_rsrc_t brsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(bias + (size_t)unit * mq_pad), 0, mq_pad * 4, 0x00020000);
  // RING_RES: ring stages [0, kResStages) hold resident rows [res_base + 64 s, ...), each read out
  // of LDS by the wave that owns those rows; ring stage kResStages + s is stream stage s.  Loaded
  // straight into registers, a lane per row, every load instruction touches 32 rows at 32 bytes
  // each: a workgroup of the wide sweep B spends 8 us on its resident keys.  Through the ring the
  // loads are whole rows, but the stream waits behind them: it pays where workgroups are short
  // (W*G <= 512: eight stream stages in sweep B) and costs elsewhere (measured both ways).
  const __amdgpu_buffer_rsrc_t res_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(res_ptr), 0, res_limit * kRowBytes, 0x00020000);
  // (two functions, and the resident phase below unrolled: where one call site could take
  // either descriptor the compiler kept both in scratch memory and fetched one per call)
  auto issue_resident = [&](int stage) {  // rows past the end read as zero through the descriptor
    unsigned char* slot = ring + (stage % kDepth) * kStageBytes;
    const int roff = (res_base + stage * kStageRows) * kRowBytes;
#pragma unroll
    for (int j = 0; j < kLoadsPerThread; ++j) {
      const int grp = wv + kWaves * j;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          res_rsrc, (__attribute__((address_space(3))) void*)(slot + grp * kGroupPitch),
          16, ld_voff, roff + j * (kWaves * 1024), 0, 0);
    }
  };
  auto issue_stage = [&](int stage) {  // ring stage >= kResStages; rows past s_end read as zero
    unsigned char* slot = ring + (stage % kDepth) * kStageBytes;
    const int sstage = stage - kResStages;
    // MODE 2: the stages of the second pass follow those of the first and read the same keys
    const int src_stage = (kTwoPass && sstage >= n_stages) ? sstage - n_stages : sstage;
    const int soff = (s_begin + src_stage * kStageRows) * kRowBytes;
    if (MODE == 1 && (stage & (kWaves - 1)) == wv)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          brsrc, (__attribute__((address_space(3))) void*)(slot + kDataBytes), 4, lane * 4,
          (s_begin + sstage * kStageRows) * 4, 0, 0);
    // Sweep B's last stage, 64 channels: its places past the last window row hold that row again (their
    // bias makes nothing of it).  A zero row times a key with an infinity would be a NaN.
    const int past = s_begin + (src_stage + 1) * kStageRows - s_end;
    if (MODE == 1 && D == 64 && past > 0 && past < kStageRows) {
#pragma unroll
      for (int j = 0; j < kLoadsPerThread; ++j) {
        const int grp = wv + kWaves * j;
        const int over = max(0, grp * kGroupRows + lane % kGroupRows - (kStageRows - 1 - past));
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rsrc, (__attribute__((address_space(3))) void*)(slot + grp * kGroupPitch),
            16, ld_voff + (j * kWaves * kGroupRows - over) * kRowBytes, soff, 0, 0);
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < kLoadsPerThread; ++j) {
      const int grp = wv + kWaves * j;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrc, (__attribute__((address_space(3))) void*)(slot + grp * kGroupPitch),
          16, ld_voff, soff + j * (kWaves * 1024), 0, 0);
    }
  };
  // Once per ring stage g: this thread's pieces of stages g and g + 1 have landed when at most
  // (kDepth - 3) later stages of its loads are still in flight; the barrier extends that to
  // every thread's pieces and tells everyone that the slot consumed before is free, so the next
  // load can go there.  The barrier is bare: a fence here would drain the whole ring.
  auto ring_wait = [&]() {
    __builtin_amdgcn_s_waitcnt(0x0F70 | (((kDepth - 3) * kLoadsPerThread) & 0xF) |
                               ((((kDepth - 3) * kLoadsPerThread) >> 4) << 14));
    __builtin_amdgcn_s_barrier();
  };
  auto ring_sync = [&](int g) {  // g + kDepth - 1 >= kResStages
    ring_wait();
    issue_stage(g + kDepth - 1);
  };

  static_assert(!RING_RES || kResStages >= kDepth - 1, "the ring's first loads are resident rows");
  if (n_stages > 0) {
#pragma unroll
    for (int s = 0; s < kDepth - 1; ++s) {
      if (RING_RES) issue_resident(s);
      else issue_stage(s);
    }
  }

  // Operand rows of this lane inside a stage: row rt * 32 + c32 -> group, row-in-group
  // (lane (c32, h) holds row c32 of a 32-row tile, k-chunk h: the same layout for both operands)
  const int a_off = (c32 / kGroupRows) * kGroupPitch + (c32 % kGroupRows) * 16 + h * (kGroupRows * 16);
  auto load_a = [&](bf16x8(&a)[NK], const unsigned char* slot, int rt) {
    const unsigned char* p = slot + rt * kTileBytes + a_off;
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) a[ks] = *reinterpret_cast<const bf16x8*>(p + ks * kStepBytes);
  };

  // ---- resident fragments: wave w owns ring stages [w CT / 2, (w + 1) CT / 2) of the resident
  // phase, two 32-row tiles each
  bf16x8 bres[CT][NK];
  auto res_row_of = [&](int ct) { return res_base + wv * kWaveRows + ct * 32 + c32; };
  if (!RING_RES) {
    // straight into registers through a bounds-checked descriptor (rows past the end read as
    // zero), after the ring's first loads are on their way so that the two latencies overlap
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      // (one launch for both sweeps: places past the last window row hold that row again, see issue_stage)
      const int r = kTwoPass ? min(res_row_of(ct), res_limit - 1) : res_row_of(ct);
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(res_rsrc, r * kRowBytes + h * 16, ks * 32, 0);
        bres[ct][ks] = __builtin_bit_cast(bf16x8, v);
      }
    }
  } else if (n_stages > 0) {
#pragma unroll
    for (int g = 0; g < kResStages; ++g) {
      ring_wait();
      if (g + kDepth - 1 < kResStages) issue_resident(g + kDepth - 1);
      else issue_stage(g + kDepth - 1);
      const unsigned char* slot = ring + (g % kDepth) * kStageBytes;
#pragma unroll
      for (int q = 0; q < CT / 2; ++q)
        if (g == wv * (CT / 2) + q) {
          load_a(bres[2 * q], slot, 0);
          load_a(bres[2 * q + 1], slot, 1);
          // the rows are in registers before the wave lets the slot go at the next barrier
          __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) alone
        }
    }
  } else {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) bres[ct][ks] = bf16x8{0};
  }
  // a wave whose resident rows are all past the end only helps with loads and barriers
  const bool wave_live = res_base + wv * kWaveRows < res_limit;
  // sweep B: -L of the lane's 16 rows of tile row rt (accumulator order)
  auto load_nl = [&](float (&nl)[16], const unsigned char* slot, int rt) {
    if (MODE == 1) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        // read with the operands' vector type: a differently typed LDS read is taken to alias
        // the ring's loads still in flight and would wait for all of them
        const bf16x8 raw = *reinterpret_cast<const bf16x8*>(slot + kDataBytes + (rt * 32 + g * 8 + h * 4) * 4);
        const f32x4 v = __builtin_bit_cast(f32x4, raw);
        nl[g * 4 + 0] = v[0]; nl[g * 4 + 1] = v[1]; nl[g * 4 + 2] = v[2]; nl[g * 4 + 3] = v[3];
      }
    }
  };

  // per-lane reduction state
  // (vector values, not arrays: an array the optimiser cannot split ends up in scratch memory)
  typedef float fxCT __attribute__((ext_vector_type(CT)));
  fxCT m_ref, l_run;  // sweep A
  fxCT colsum;                 // sweep B
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    m_ref[ct] = kNegInf;
    l_run[ct] = 0.f;
    colsum[ct] = 0.f;
  }
  // sweep A: last key the lane's window row sees; sweep B: the lane's key
  auto vis_limit_of = [&](int ct) {
    return (kRowPass) ? (kp.causal ? N - W + res_row_of(ct) / Gq : N - 1) : res_row_of(ct);
  };
  const int tail_start = kp.causal ? N - W : N;  // keys > tail_start are hidden from some row
  typedef int ixCT __attribute__((ext_vector_type(CT)));
  ixCT first_row;  // sweep B: first window row that sees the lane's key
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
    first_row[ct] = (MODE == 1 && kp.causal) ? max(0, (res_row_of(ct) - (N - W)) * Gq) : 0;

  // ---- epilogues
  // sweep A: a tile's 16 terms are summed on their own and banked into the lane's running sum
  // once per tile, so the long sum over a unit's keys has N / 32 addends, not N / 2 (the rounding
  // error of a single fp32 running sum would grow with the unit's length)
  float tsum = 0.f;
  auto bank_tile = [&](int ct) {
    if (kRowPass) {
      // (static indices only: an index the optimiser does not see through would move the
      // array into scratch memory)
#pragma unroll
      for (int k = 0; k < CT; ++k)
        if (k == ct) l_run[k] += tsum;
      tsum = 0.f;
    }
  };
  // Masked variant (tag true): a logit is dropped by one comparison of its stream-row offset
  // inside the tile (a constant) with `d`, the lane's limit relative to the tile:
  //   sweep A: hidden iff offset > d, d = (last key the lane's row sees) - first row of the tile - 4 h
  //   sweep B: hidden iff offset < d, d = (first row that sees the lane's key) - first row of the tile - 4 h
  // sweep A: last stream row (key) that counts for the lane's window row.  Only masked stages
  // look at it: set_limits() runs in front of them, so the clean stages do not carry the values.
  int lim_a[CT];
  auto set_limits = [&]() {
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) lim_a[ct] = min(s_end - 1, vis_limit_of(ct));
  };
  auto mask_d = [&](int ct, int trow0) { return (kRowPass ? lim_a[ct] : first_row[ct]) - trow0 - h * 4; };
  auto piece = [&](auto masked, const f32x16& acc, const float (&nl)[16], int ct, int i, int d) {  // two logits of the fast epilogue
    constexpr bool kMasked = decltype(masked)::value;
    const int o0 = ((2 * i) >> 2) * 8 + ((2 * i) & 3), o1 = o0 + 1;  // row offsets of logits 2i, 2i + 1
    if (kRowPass) {
      const float nm = -m_ref[ct];
      float x0 = acc[2 * i], x1 = acc[2 * i + 1];
      if (kMasked) {
        x0 = o0 > d ? kNegInf : x0;
        x1 = o1 > d ? kNegInf : x1;
      }
      tsum += fast_exp2(__builtin_fmaf(x0, c, nm));
      tsum += fast_exp2(__builtin_fmaf(x1, c, nm));
      // pin the partial sum here: without it the optimiser is free to sink these pieces out
      // of the MFMA chain they are meant to overlap with
      asm volatile("" : "+v"(tsum));
    } else {
      float y0 = __builtin_fmaf(acc[2 * i], c, nl[2 * i]), y1 = __builtin_fmaf(acc[2 * i + 1], c, nl[2 * i + 1]);
      if (kMasked) {
        y0 = o0 < d ? kNegInf : y0;
        y1 = o1 < d ? kNegInf : y1;
      }
      colsum[ct] += fast_exp2(y0);
      colsum[ct] += fast_exp2(y1);
      asm volatile("" : "+v"(colsum[ct]));
    }
  };
  // exact online-softmax update of (m_ref, l_run) with the 16 logits of `acc` (masked = -inf)
  auto exact_update = [&](const f32x16& acc, int ct) {
    float xm = acc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) xm = fmaxf(xm, acc[r]);
    const float m_new = fmaxf(m_ref[ct], xm * c);
    const float nm = (m_new == kNegInf) ? 0.f : -m_new;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) sum += fast_exp2(__builtin_fmaf(acc[r], c, nm));
    l_run[ct] = l_run[ct] * fast_exp2(m_ref[ct] + nm) + sum;
    m_ref[ct] = m_new;
  };
  auto slow_tile = [&](f32x16& acc, const float (&nl)[16], int ct, int trow0) {
    if (kRowPass) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = trow0 + (r >> 2) * 8 + h * 4 + (r & 3);
        if (!(key <= lim_a[ct])) acc[r] = kNegInf;  // (the limit is already cut at the end of the stream)
      }
      exact_update(acc, ct);
    } else {
      // window row r sits at slot N - W + r / G, so key j is visible to it iff
      // r >= (j - (N - W)) * G: one comparison against a per-lane constant
      float sum = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = trow0 + (r >> 2) * 8 + h * 4 + (r & 3);
        const float y = (row < first_row[ct]) ? kNegInf : __builtin_fmaf(acc[r], c, nl[r]);
        sum += fast_exp2(y);
      }
      colsum[ct] += sum;
    }
  };
  auto chain = [&](f32x16& acc, const bf16x8(&a)[NK], int ct) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], bres[ct][0], f32x16{0}, 0, 0, 0);
#pragma unroll
    for (int ks = 1; ks < NK; ++ks)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], bres[ct][ks], acc, 0, 0, 0);
  };
  // chain of the new tile interleaved with the fast epilogue of the old one
  // (`trow_old`: first stream row of the old tile; only the masked variant looks at it)
  auto fused = [&](auto masked, f32x16& acc_new, const bf16x8(&a)[NK], int ct_new, const f32x16& acc_old,
                   const float (&nl_old)[16], int ct_old, int trow_old) {
    const int d = mask_d(ct_old, trow_old);
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
#pragma unroll
      for (int e = 0; e < NP; ++e) piece(masked, acc_old, nl_old, ct_old, ks * NP + e, d);
      acc_new = (ks == 0)
                    ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], bres[ct_new][0], f32x16{0}, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], bres[ct_new][ks], acc_new, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    bank_tile(ct_old);
  };
  auto drain = [&](auto masked, const f32x16& acc_old, const float (&nl_old)[16], int ct_old, int trow_old) {
    const int d = mask_d(ct_old, trow_old);
#pragma unroll
    for (int i = 0; i < 8; ++i) piece(masked, acc_old, nl_old, ct_old, i, d);
    bank_tile(ct_old);
  };

  // ---- main loop over ring stages
  // Take the wait for the resident operands here, before the first barrier issues more loads:
  // left to the compiler it lands inside the loop prologue as a wait for every load in flight,
  // the ring's newest stage included.
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) asm volatile("" ::"v"(bres[ct][ks]));
  // Stream stage `it` is ring stage kResStages + it.  Being one stage ahead (see ring_sync) lets
  // a wave fetch the next stage's first operands from LDS while it is still busy with this one.
  auto stage_sync = [&](int it) { ring_sync(kResStages + it); };
  auto slot_of = [&](int it) -> const unsigned char* {
    return ring + ((kResStages + it) % kDepth) * kStageBytes;
  };
  f32x16 acc0, acc1;
  bf16x8 a0[NK], a1[NK];
  float nl0[16], nl1[16];  // sweep B: -L of the rows of tile rows 0 and 1 of the stage in flight
  auto slow_stage = [&](int it) {
    const unsigned char* cur = slot_of(it);
    const int stage_base = s_begin + it * kStageRows;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const int trow0 = stage_base + rt * 32;
      if (trow0 >= s_end) continue;
      load_a(a0, cur, rt);
      load_nl(nl0, cur, rt);
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        chain(acc0, a0, ct);
        slow_tile(acc0, nl0, ct, trow0);
      }
    }
    if (kRowPass) {
      // a lane that saw nothing yet takes 0 as its reference: (0, 0) is the empty sum
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        if (m_ref[ct] == kNegInf) m_ref[ct] = 0.f;
    }
  };

  // Stages [f0, f1) run the pipelined path, [sk, f0) and [f1, n_stages) the masked path, and
  // the wave sits out stages [0, sk).
  // Sweep A: the causal tail and the ragged end are masked.
  // Sweep B: window rows come in slot order, so a wave whose keys lie in the window sees
  // nothing in the first stages (every row is older than its oldest key), is partly masked
  // until the rows pass its youngest key, and is clean from there on.
  int sk = 0, f0 = 0, f1;
  if (kRowPass) {
    const int clean_rows = min(tail_start + 1, s_end) - s_begin;  // keys every row sees
    f1 = clean_rows > 0 ? clean_rows / kStageRows : 0;
  } else {
    if (kp.causal) {
      const int k0 = res_base + wv * kWaveRows - (N - W);  // the wave's oldest key, relative to the window
      const int fr_min = max(0, k0 * Gq), fr_max = max(0, (k0 + kWaveRows - 1) * Gq);
      sk = max(0, min(n_stages, (fr_min - s_begin) / kStageRows));
      f0 = max(sk, min(n_stages, (fr_max - s_begin + kStageRows - 1) / kStageRows));
    }
    f1 = n_stages;
  }
  f1 = max(min(f1, n_stages), f0);
  if (!wave_live) sk = f0 = f1 = n_stages;  // only loads and barriers: the first loop below

  // Reference of a resident row from the lane's first 16 logits of it.  A term is as exact as its
  // distance from the reference is small, so with 64 channels it is put near the row's largest logit:
  // at most 16 above the largest one seen, so that the sum stays far from underflow.  (Norm of the
  // scores' error against 64-bit sums, 128 units of 5378 rows: 6.4e-7 with the first logit, 2.2e-7;
  // 200 of 1100: 5.2e-7, 2.1e-7.  A running maximum, as the vector kernel had it: 8.1e-7 and 3.5e-7.)
  auto reference = [&](const f32x16& acc) {
    if constexpr (D == 128) return acc[0] * c;
    float hi = acc[0], lo = acc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) {
      hi = fmaxf(hi, acc[r]);
      lo = fminf(lo, acc[r]);
    }
    return __builtin_fmaf(hi, c, fminf(0.3f * c * (hi - lo), 16.f));
  };
  // stages [from, to), to > from, software-pipelined; does the stage_sync of each of them
  auto pipelined = [&](auto masked, int from, int to) {
    constexpr bool kMasked = decltype(masked)::value;
    stage_sync(from);
    load_a(a0, slot_of(from), 0);
    load_nl(nl0, slot_of(from), 0);
    if (kRowPass && !kMasked && from == 0) {
      // Nothing seen yet: the first logits of the lane's own row give the reference.  Too low shows
      // as a sum out of range at the end and sends the wave through the exact recomputation; too
      // high only means every other term is negligible next to the first ones, which are themselves
      // part of the sum.
      chain(acc1, a0, 1);
      m_ref[1] = reference(acc1);
      chain(acc0, a0, 0);
      m_ref[0] = reference(acc0);
    } else {
      chain(acc0, a0, 0);
    }
    for (int it = from;; ++it) {
      const unsigned char* cur = slot_of(it);
      const int base = s_begin + it * kStageRows;
      load_a(a1, cur, 1);
      load_nl(nl1, cur, 1);
      fused(masked, acc1, a0, 1, acc0, nl0, 0, base);
      load_a(a0, slot_of(it + 1), 0);  // a0 is free: operands of the coming stage
      fused(masked, acc0, a1, 0, acc1, nl0, 1, base);
      load_nl(nl0, slot_of(it + 1), 0);  // the last tile of tile row 0 is through its epilogue
      fused(masked, acc1, a1, 1, acc0, nl1, 0, base + 32);
      if (it + 1 >= to) break;
      stage_sync(it + 1);
      fused(masked, acc0, a0, 0, acc1, nl1, 1, base + 32);
    }
    drain(masked, acc1, nl1, 1, s_begin + (to - 1) * kStageRows + 32);
  };
  // Wide form, four resident tiles per wave (both sweeps): a wave keeps ONE tile row's stream
  // operands; while the last of the tile row's four chains consumes them k-step by k-step, each
  // is replaced in place by the next tile row's (the 32 registers that saves, with the 64 the two
  // more resident tiles cost, still fit two waves per SIMD).  Sweep B's 16 -L values of a tile
  // row change hands the same way during the chain that carries the tile row's last epilogue.
  // Tiles of a stage in the order (tile row, resident tile) = (0,0) (0,1) (0,2) (0,3) (1,0) ...
  // (1,3), accumulators alternating.
  // fused_refill: `refill_a`: the stream operands are replaced by the rows at `next_rows`;
  // `refill_nl` (sweep B): the -L values by those at `next_nl`, four at a time behind the two
  // pieces that used them.
  auto fused_refill = [&](auto masked, auto refill_a, auto refill_nl, f32x16& acc_new, bf16x8(&a)[NK],
                          int ct_new, const f32x16& acc_old, float (&nl)[16], int ct_old, int trow_old,
                          const unsigned char* next_rows, const unsigned char* next_nl) {
    constexpr bool kA = decltype(refill_a)::value, kNl = decltype(refill_nl)::value && MODE == 1;
    const int d = mask_d(ct_old, trow_old);
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
#pragma unroll
      for (int e = 0; e < NP; ++e) piece(masked, acc_old, nl, ct_old, ks * NP + e, d);
      acc_new = (ks == 0)
                    ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], bres[ct_new][0], f32x16{0}, 0, 0, 0)
                    : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[ks], bres[ct_new][ks], acc_new, 0, 0, 0);
      if (kA) a[ks] = *reinterpret_cast<const bf16x8*>(next_rows + ks * kStepBytes);
      if (kNl && ((ks + 1) * NP) % 2 == 0) {
        const int g = (ks + 1) * NP / 2 - 1;
        const bf16x8 raw = *reinterpret_cast<const bf16x8*>(next_nl + (g * 8 + h * 4) * 4);
        const f32x4 v = __builtin_bit_cast(f32x4, raw);
        nl[g * 4 + 0] = v[0]; nl[g * 4 + 1] = v[1]; nl[g * 4 + 2] = v[2]; nl[g * 4 + 3] = v[3];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    bank_tile(ct_old);
  };
  auto pipelined_wide = [&](auto masked, int from, int to) {
    constexpr bool kMasked = decltype(masked)::value;
    constexpr int L = CT - 1;  // the last resident tile
    const std::integral_constant<bool, true> yes;
    const std::integral_constant<bool, false> no;
    stage_sync(from);
    load_a(a0, slot_of(from), 0);
    load_nl(nl0, slot_of(from), 0);
    if (kRowPass && !kMasked && from == 0) {
      // references: from the first logits of every resident row of the lane
#pragma unroll
      for (int ct = L; ct >= 1; --ct) {
        chain(acc1, a0, ct);
        m_ref[ct] = reference(acc1);
      }
      chain(acc0, a0, 0);
      m_ref[0] = reference(acc0);
    } else {
      chain(acc0, a0, 0);
    }
    for (int it = from;; ++it) {
      const unsigned char* cur = slot_of(it);
      const int base = s_begin + it * kStageRows;
      fused(masked, acc1, a0, 1, acc0, nl0, 0, base);
      fused(masked, acc0, a0, 2, acc1, nl0, 1, base);
      // a0 <- tile row 1 behind the last chain of tile row 0
      fused_refill(masked, yes, no, acc1, a0, 3, acc0, nl0, 2, base, cur + kTileBytes + a_off, nullptr);
      // the last epilogue of tile row 0 hands its -L registers over to tile row 1
      fused_refill(masked, no, yes, acc0, a0, 0, acc1, nl0, 3, base, nullptr, cur + kDataBytes + 32 * 4);
      fused(masked, acc1, a0, 1, acc0, nl0, 0, base + 32);
      fused(masked, acc0, a0, 2, acc1, nl0, 1, base + 32);
      if (it + 1 >= to) {
        fused(masked, acc1, a0, 3, acc0, nl0, 2, base + 32);
        break;
      }
      const unsigned char* nxt = slot_of(it + 1);
      fused_refill(masked, yes, no, acc1, a0, 3, acc0, nl0, 2, base + 32, nxt + a_off, nullptr);  // a0 <- next stage
      stage_sync(it + 1);
      fused_refill(masked, no, yes, acc0, a0, 0, acc1, nl0, 3, base + 32, nullptr, nxt + kDataBytes);
    }
    drain(masked, acc1, nl0, L, s_begin + (to - 1) * kStageRows + 32);
  };
  const std::integral_constant<bool, false> clean_tag;
  const std::integral_constant<bool, true> masked_tag;

  int it = 0;
  if (kRowPass && f0 < f1) {
    // (placeholder values while the clean stages run: nothing reads them there)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) lim_a[ct] = 0;
  } else if (kRowPass) {
    set_limits();
  }
  for (; it < sk; ++it) stage_sync(it);
  if (MODE == 1) {
    // the partly visible stages run pipelined as well, with the mask in the epilogue
    if (f0 > sk) {
      if (CT == 4) pipelined_wide(masked_tag, sk, f0);
      else pipelined(masked_tag, sk, f0);
    }
  } else {
    for (; it < f0; ++it) {
      stage_sync(it);
      slow_stage(it);
    }
  }
  if (f1 > f0) {
    if (CT == 4) pipelined_wide(clean_tag, f0, f1);
    else pipelined(clean_tag, f0, f1);
  }
  it = f1;
  if (kRowPass) set_limits();
  if (kRowPass && f1 > 0 && n_stages > f1) {
    // the tail (causal, ragged end) after at least one clean stage: the reference is set, so
    // the masked epilogue can take it
    if (CT == 4) pipelined_wide(masked_tag, f1, n_stages);
    else pipelined(masked_tag, f1, n_stages);
    it = n_stages;
  }
  for (; it < n_stages; ++it) {
    stage_sync(it);
    slow_stage(it);
  }
  if (kRowPass && wave_live) {
    // Range check of the fast epilogue, once per wave: a sum in range is exact.
    bool bad = false;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) bad = bad || !(l_run[ct] < kMostSum);
    if (__builtin_amdgcn_ballot_w64(bad) != 0ull) {
      // Recompute this wave's statistics with a true running maximum.  The ring belongs to the
      // whole workgroup, so the stream rows come straight from memory (same bounds-checked
      // descriptor: rows past the end read as zero and are masked).
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        m_ref[ct] = kNegInf;
        l_run[ct] = 0.f;
      }
      for (int stg = 0; stg < n_stages; ++stg) {
        for (int rt = 0; rt < 2; ++rt) {
          const int trow0 = s_begin + stg * kStageRows + rt * 32;
          if (trow0 >= s_end) continue;
#pragma unroll
          for (int ks = 0; ks < NK; ++ks) {
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (trow0 + c32) * kRowBytes + h * 16, ks * 32, 0);
            a0[ks] = __builtin_bit_cast(bf16x8, v);
          }
#pragma unroll
          for (int ct = 0; ct < CT; ++ct) {
            chain(acc0, a0, ct);
            slow_tile(acc0, nl0, ct, trow0);
          }
        }
      }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct)
        if (m_ref[ct] == kNegInf) m_ref[ct] = 0.f;
    }
  }
  // loads issued past the last stage may still be landing in LDS: let them finish before the
  // workgroup's LDS can be handed to another one
  if (!kTwoPass) __builtin_amdgcn_s_waitcnt(0x0F70);

  // ---- finish
  if (kTwoPass) {
    // ---- second pass: the same resident window rows are now the A operand and the keys
    // stream through the ring once more (their stages were requested while the first pass
    // finished), so a lane owns one key column of a tile and 16 window rows.  exp2(c x - L_row)
    // summed over the rows of this wave is one partial column sum per key; the waves write
    // theirs side by side (`parts[unit][16-row-block wave][key]`) and whoever reads the scores
    // adds them in wave order: no atomics, the same bits every run.
    float* negl_s = reinterpret_cast<float*>(smem + kDepth * kStageBytes);  // -L of the workgroup's 256 rows
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      const float m2 = __shfl_xor(m_ref[ct], 32, 64);
      const float l2 = __shfl_xor(l_run[ct], 32, 64);
      float mc = m_ref[ct], lc = l_run[ct];
      ml_combine<true>(mc, lc, m2, l2);
      m_ref[ct] = mc;
      l_run[ct] = lc;
      if (h == 0)
        negl_s[wv * 64 + ct * 32 + c32] = res_row_of(ct) < Mq ? -(m_ref[ct] + log2f(l_run[ct])) : kPadNegL;
    }
    // the wave reads back only what it wrote itself (LDS operations of a wave stay in order);
    // the empty asm keeps the compiler from moving the differently typed reads above the writes
    asm volatile("" ::: "memory");
    float nlq[2][16];
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const bf16x8 raw = *reinterpret_cast<const bf16x8*>(
            reinterpret_cast<const unsigned char*>(negl_s) + (wv * 64 + ct * 32 + g * 8 + h * 4) * 4);
        const f32x4 v = __builtin_bit_cast(f32x4, raw);
        nlq[ct][g * 4 + 0] = v[0]; nlq[ct][g * 4 + 1] = v[1]; nlq[ct][g * 4 + 2] = v[2]; nlq[ct][g * 4 + 3] = v[3];
      }
    float* part_out = parts + ((size_t)unit * ((Mq + 63) / 64) + (res_base >> 6) + wv) * part_pitch;
    float ksum = 0.f;
    auto chain2 = [&](f32x16& acc, const bf16x8(&a)[NK], int ct) {
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bres[ct][0], a[0], f32x16{0}, 0, 0, 0);
#pragma unroll
      for (int ks = 1; ks < NK; ++ks)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bres[ct][ks], a[ks], acc, 0, 0, 0);
    };
    // hidden iff the row's offset inside the resident tile is < d,
    // d = (first window row that sees the lane's key) - first row of the tile - 4 h
    auto mask_d2 = [&](int ct, int key) {
      const int first = kp.causal ? max(0, (key - (N - W)) * Gq) : 0;
      return first - (res_base + wv * 64 + ct * 32 + h * 4);
    };
    auto piece2 = [&](auto masked, const f32x16& acc, int ct, int i, int d) {
      constexpr bool kMasked = decltype(masked)::value;
      const int o0 = ((2 * i) >> 2) * 8 + ((2 * i) & 3), o1 = o0 + 1;
      float y0 = __builtin_fmaf(acc[2 * i], c, nlq[ct][2 * i]), y1 = __builtin_fmaf(acc[2 * i + 1], c, nlq[ct][2 * i + 1]);
      if (kMasked) {
        y0 = o0 < d ? kNegInf : y0;
        y1 = o1 < d ? kNegInf : y1;
      }
      ksum += fast_exp2(y0);
      ksum += fast_exp2(y1);
      asm volatile("" : "+v"(ksum));
    };
    auto fused2 = [&](auto masked, f32x16& acc_new, const bf16x8(&a)[NK], int ct_new, const f32x16& acc_old,
                      int ct_old, int key_old) {
      const int d = mask_d2(ct_old, key_old);
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
#pragma unroll
        for (int e = 0; e < NP; ++e) piece2(masked, acc_old, ct_old, ks * NP + e, d);
        acc_new = (ks == 0)
                      ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(bres[ct_new][0], a[0], f32x16{0}, 0, 0, 0)
                      : __builtin_amdgcn_mfma_f32_32x32x16_bf16(bres[ct_new][ks], a[ks], acc_new, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // MODE 3: per stage and wave 64 partial column sums go to LDS (a ring of four stages behind
    // the -L table), and two barriers later the wave whose turn it is adds the four waves' sums
    // in wave order.  The LDS traffic is written out as instructions: accesses the compiler
    // generates here would be taken to alias the ring's loads in flight and wait for all of them.
    const unsigned xs_base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)(
        smem + kDepth * kStageBytes + kResRows * sizeof(float));
    const int two_blocks = Mq > kResRows;
    const float inv_mq = 1.0f / (float)Mq;
    auto reduce_stage = [&](int st) {  // all four waves' sums of pass-2 stage `st` are in LDS
      float v0, v1, v2, v3;
      const unsigned addr = xs_base + (unsigned)(((st & 3) * kWaves * 64 + lane) * 4);
      asm volatile(
          "ds_read_b32 %0, %4\n\tds_read_b32 %1, %4 offset:256\n\tds_read_b32 %2, %4 offset:512\n\t"
          "ds_read_b32 %3, %4 offset:768\n\ts_waitcnt lgkmcnt(0)"
          : "=&v"(v0), "=&v"(v1), "=&v"(v2), "=&v"(v3)
          : "v"(addr));
      float v = v0;  // wave 0 always has rows
      if (res_base + 64 < res_limit) v += v1;
      if (res_base + 128 < res_limit) v += v2;
      if (res_base + 192 < res_limit) v += v3;
      const int key = s_begin + st * kStageRows + lane;
      if (key < N) {
        if (two_blocks) atomicAdd(&scores[row0 + key], v * inv_mq);
        else scores[row0 + key] = v * inv_mq;
      }
    };
    auto flush = [&](int key, int st, int kt) {  // both resident tiles of this key tile are through their epilogue
      const float tot = ksum + __shfl_xor(ksum, 32, 64);
      if (kWgReduce) {
        if (h == 0) {
          const unsigned addr = xs_base + (unsigned)((((st & 3) * kWaves + wv) * 64 + kt * 32 + c32) * 4);
          asm volatile("ds_write_b32 %0, %1" ::"v"(addr), "v"(tot));
        }
      } else {
        if (h == 0 && key < N) part_out[key] = tot;
      }
      ksum = 0.f;
    };
    // barrier of pass-2 stage it2; MODE 3: the waves' LDS writes are complete before it, and the
    // sums of stage it2 - 2 (complete since the barrier before this one) are added by one wave
    auto sync2 = [&](int it2) {
      if (kWgReduce) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0) alone; vmcnt is stage_sync's business
      stage_sync(n_stages + it2);
      if (kWgReduce && it2 >= 2 && ((it2 - 2) & 3) == wv) reduce_stage(it2 - 2);
    };
    // stages [from, to) of the second pass (ring stages n_stages + from ...), software-pipelined
    auto pipelined2 = [&](auto masked, int from, int to) {
      sync2(from);
      load_a(a0, slot_of(n_stages + from), 0);
      chain2(acc0, a0, 0);
      for (int it = from;; ++it) {
        const unsigned char* cur = slot_of(n_stages + it);
        const int key0 = s_begin + it * kStageRows + c32;  // the lane's key in key tile 0 of the stage
        load_a(a1, cur, 1);
        fused2(masked, acc1, a0, 1, acc0, 0, key0);
        load_a(a0, slot_of(n_stages + it + 1), 0);
        fused2(masked, acc0, a1, 0, acc1, 1, key0);
        flush(key0, it, 0);
        fused2(masked, acc1, a1, 1, acc0, 0, key0 + 32);
        if (it + 1 >= to) break;
        sync2(it + 1);
        fused2(masked, acc0, a0, 0, acc1, 1, key0 + 32);
        flush(key0 + 32, it, 1);
      }
      const int key1 = s_begin + (to - 1) * kStageRows + 32 + c32;
      const int d = mask_d2(1, key1);
#pragma unroll
      for (int i = 0; i < 8; ++i) piece2(masked, acc1, 1, i, d);
      flush(key1, to - 1, 1);
    };
    if (wave_live) {
      const int clean = min(f1, n_stages);  // stages whose keys every window row sees
      if (clean > 0) pipelined2(clean_tag, 0, clean);
      if (n_stages > clean) pipelined2(masked_tag, clean, n_stages);
      // keys past the stages that ran are hidden from every row of this workgroup
      if (!kWgReduce)
        for (int key = s_begin + n_stages * kStageRows + lane; key < N; key += 64) part_out[key] = 0.f;
    } else {
      for (int it2 = 0; it2 < n_stages; ++it2) sync2(it2);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    if (kWgReduce) {
      // the last two stages' sums: complete once every wave is here
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_s_barrier();
      if (n_stages >= 2 && ((n_stages - 2) & 3) == wv) reduce_stage(n_stages - 2);
      if (n_stages >= 1 && ((n_stages - 1) & 3) == wv) reduce_stage(n_stages - 1);
      // a single row block stores its scores: keys past its stages are hidden from every row
      if (!two_blocks && wv == 0)
        for (int key = s_begin + n_stages * kStageRows + lane; key < N; key += 64) scores[row0 + key] = 0.f;
    }
  } else if (MODE == 0) {
    float2* part = rowstat + (size_t)unit * n_splits * mq_pad;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const float m2 = __shfl_xor(m_ref[ct], 32, 64);
      const float l2 = __shfl_xor(l_run[ct], 32, 64);
      float mc = m_ref[ct], lc = l_run[ct];
      ml_combine<true>(mc, lc, m2, l2);
      m_ref[ct] = mc;
      l_run[ct] = lc;
      if (h == 0 && res_row_of(ct) < Mq)
        part[(size_t)split * mq_pad + res_row_of(ct)] = make_float2(m_ref[ct], l_run[ct]);
      // a single split is the whole row: -L goes out here and no combining kernel runs
      if (n_splits == 1 && h == 0 && res_row_of(ct) < mq_pad)
        bias_out[(size_t)unit * mq_pad + res_row_of(ct)] =
            res_row_of(ct) < Mq ? -(m_ref[ct] + log2f(l_run[ct])) : kPadNegL;
    }
  } else if (MODE == 1) {
    const float inv = 1.0f / (float)Mq;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      const float tot = colsum[ct] + __shfl_xor(colsum[ct], 32, 64);
      if (h == 0 && res_row_of(ct) < N) {
        if (q_splits == 2) atomicAdd(&scores[row0 + res_row_of(ct)], tot * inv);
        else scores[row0 + res_row_of(ct)] = tot * inv;
      }
    }
  }
}

// ------------------------------------------------------------------ short units, one sweep

// Scores of units of at most 1024 rows with the contraction and the exponentials done once: a
// workgroup takes 64 window rows of a unit and ALL its keys, and the logits stay in registers (fp32)
// between the row statistics and the column sums.  It leaves one partial column sum per key,
// `parts[unit][block of 64 rows][key]`; whoever reads the scores adds them in order (no atomics: the
// same bits every run).
//
// Wave w of NW holds the key tiles w, w + NW, ... (KT of 32 keys) against both 32-row tiles: KT x 2
// accumulators of 16 registers, 64 more for the window rows' operands (read from LDS once), so two
// waves per SIMD at KT <= 5.  Keys reach LDS by direct loads into two slots of the wave's own: no
// barrier in the loop.  A lane owns one key of a tile and 16 rows of each row tile, so column sums
// stay in the lane; a row's maximum and sum cross the 32 lanes once per wave (reduce32), and the
// waves exchange (maximum, sum) pairs through LDS: the one barrier behind the window rows'.
//
// Operand rows lie in LDS in groups of 1 KB (four rows of 256 bytes, eight of 128): piece p of
// row r of group g at ((p ^ g) x rows + r) x 16, which spreads any 16 lanes of an operand read over
// all banks without padding (two workgroups take exactly the 160 KB of a compute unit).
//
// Bound: a workgroup's chain (window rows and first keys 3 us, loop, exponentials, exchange, column
// sums: 8 - 13 us); in a full chip the loop runs at the keys' rate from L2 (14 TB/s over all
// compute units) and the rest at the vector pipes', one after the other, where the two sweeps below
// overlap them.  So it is for batches that leave the sweeps' 256-row workgroups too few (rule at
// launch_score_parts).  4 units x 512 rows, 896 window rows: 22.4 -> 10.1 us; 112 x 640 rows: 48.4 ->
// 47.  Several blocks per workgroup, walking the tiles back and forth so that two need not be read
// again, took 51 - 62 us there.
template <typename Op>
__device__ __forceinline__ float reduce32(float (&v)[32], int c32, Op op) {
  // v[i] of the 32 lanes of a half wave combined over the lanes; lane c32 gets value c32
  float a[16], b[8], c[4], d[2];
#pragma unroll
  for (int j = 0; j < 16; ++j) {  // (swaps the odd rows of 16 lanes of the first with the even ones of the second)
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[j]), __float_as_uint(v[j + 16]), false, false);
    a[j] = op(__uint_as_float(s[0]), __uint_as_float(s[1]));
  }
  auto halve = [&](bool up, float lo, float hi, auto ctrl) {
    const float keep = up ? hi : lo, send = up ? lo : hi;
    const int got = __builtin_amdgcn_update_dpp(0, __float_as_int(send), decltype(ctrl)::value, 0xF, 0xF, true);
    return op(keep, __int_as_float(got));
  };
#pragma unroll
  for (int j = 0; j < 8; ++j) b[j] = halve(c32 & 8, a[j], a[j + 8], std::integral_constant<int, 0x128>());  // row_ror:8
#pragma unroll
  for (int j = 0; j < 4; ++j) c[j] = halve(c32 & 4, b[j], b[j + 4], std::integral_constant<int, 0x141>());  // row_half_mirror
#pragma unroll
  for (int j = 0; j < 2; ++j) d[j] = halve(c32 & 2, c[j], c[j + 2], std::integral_constant<int, 0x4E>());   // lanes ^ 2
  return halve(c32 & 1, d[0], d[1], std::integral_constant<int, 0xB1>());                                    // lanes ^ 1
}

template <int D, int KT, int NW>
__global__ __launch_bounds__(NW * 64, 2) void score_short_kernel(
    KParams kp, int n_units, int blocks, const int64_t* __restrict__ row_off, const uint16_t* __restrict__ K,
    const uint16_t* __restrict__ Q, float* __restrict__ parts, int part_pitch) {
  constexpr int RB = D * 2, GR = 1024 / RB, NK = D / 16;
  constexpr int TL = 32 / GR;               // loads (groups) of a 32-row tile
  constexpr int kTile = 32 * RB;
  constexpr int kStep = 2 * GR * 16;        // two pieces of a group
  static_assert(KT >= 2 && (2 * TL) % NW == 0, "two slots are filled ahead; the waves share the window rows' loads");
  static_assert(NW * 768 <= 2 * kTile, "the exchange lies over the window rows");
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * kTile + NW * 2 * kTile];
  int unit, blk;
  if (!map_block(n_units, blocks, unit, blk)) return;
  const int lane = threadIdx.x & 63, c32 = lane & 31, h = lane >> 5;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row0 = row_off[unit];
  const int N = (int)(row_off[unit + 1] - row0);  // <= KT * NW * 32: the host checked
  const int Mq = kp.Mq, Gq = kp.G, row_base = blk * 64;
  const int tail = kp.causal ? N - kp.W : N - 1;  // keys beyond are hidden from some row
  const float c = kp.scale_log2;
  unsigned char* const own = smem + 2 * kTile + wv * (2 * kTile);

  const __amdgpu_buffer_rsrc_t krsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(K + (size_t)row0 * D), 0, N * RB, 0x00020000);
  const __amdgpu_buffer_rsrc_t qrsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(Q + (size_t)unit * Mq * D), 0, Mq * RB, 0x00020000);
  const int ld_voff = (lane % GR) * RB + (lane / GR) * 16;  // group 0; group g takes piece ^ g
  auto load_group = [&](const __amdgpu_buffer_rsrc_t& rsrc, unsigned char* dst, int g, int row) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(dst + g * 1024), 16,
                                             ld_voff ^ (g * 16), row * RB, 0, 0);
  };
  auto load_keys = [&](int kt) {  // rows past the unit's end read as zero
#pragma unroll
    for (int g = 0; g < TL; ++g) load_group(krsrc, own + (kt & 1) * kTile, g, (kt * NW + wv) * 32 + g * GR);
  };
#pragma unroll
  for (int j = 0; j < 2 * TL / NW; ++j) {  // rows past W*G read as zero
    const int g = wv * (2 * TL / NW) + j;
    load_group(qrsrc, smem, g, row_base + g * GR);
  }
  load_keys(0);
  load_keys(1);
  // operand of lane (c32, h), k-step ks: piece 2 ks + h of row c32
  const int rd = (c32 / GR) * 1024 + (c32 % GR) * 16 + ((h ^ (c32 / GR)) * (GR * 16));
  const int my_row = (c32 >> 4) * 32 + ((c32 >> 2) & 3) * 8 + h * 4 + (c32 & 3);  // where reduce32 leaves value c32
  float* const bcast = reinterpret_cast<float*>(smem + wv * 768);  // one value per row, for the wave itself
  auto stat_of = [&](int w) { return reinterpret_cast<float2*>(smem + w * 768 + 256); };  // (maximum, sum) per row, for all
  // (one instruction; fmaxf, which this becomes if the bound is a known constant, would first quiet
  // a NaN in either operand: one more each)
  float bound = __builtin_inff();
  asm("" : "+s"(bound));
  auto larger = [&](float x, float y) { return __builtin_amdgcn_fmed3f(x, y, bound); };

  __builtin_amdgcn_s_waitcnt(0x0F70 | ((2 * TL) & 0xF) | (((2 * TL) >> 4) << 14));  // the window rows are here
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  bf16x8 q[2][NK];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    // (the second tile's groups are TL .. 2 TL - 1: their number reaches into the piece as well)
    const int rq = rd ^ (rt * TL * (GR * 16));
#pragma unroll
    for (int ks = 0; ks < NK; ++ks)
      q[rt][ks] = *reinterpret_cast<const bf16x8*>(smem + rt * kTile + (rq ^ (ks * kStep)));
  }
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) asm volatile("" ::"v"(q[rt][ks]));
  // every wave has its operands: the exchange below may overwrite the window rows
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  // ---- logits; a tile that no row of the block sees is left out, here and below
  const int last_row = min(Mq, row_base + 64) - 1;
  const int last_key = kp.causal ? N - kp.W + last_row / Gq : N - 1;  // < N
  auto tile0 = [&](int kt) { return (kt * NW + wv) * 32; };  // first key
  auto seen = [&](int kt) { return tile0(kt) <= last_key; };
  const bool ragged = row_base + 64 > Mq;  // (a zero row past the last times a key with an infinity: a NaN)
  auto masked = [&](int kt) { return tile0(kt) + 31 > tail || ragged; };
  // Bit r: the lane's key of tile kt is hidden from row r of the 16 the lane holds in row tile rt.
  // (Bit fields, not compares: a compare and its select wait for each other.)
  auto hidden_bits = [&](int kt, int rt) {
    const int key = tile0(kt) + c32;
    const int first = key < N ? (kp.causal ? (key - (N - kp.W)) * Gq : 0) : 0x40000000;  // first row that sees the key
    const int d = min(max(first - row_base - rt * 32 - h * 4, 0), 32);                    // hidden: row offset < d
    const int rows = min(max(Mq - row_base - rt * 32 - h * 4, 0), 32);                    // hidden: row offset >= rows
    const unsigned below = (unsigned)((1ull << d) - 1ull) | ~(unsigned)((1ull << rows) - 1ull);  // offsets 0 .. 31; the lane's are 8 g + 0 .. 3
    return (below & 0xFu) | ((below >> 4) & 0xF0u) | ((below >> 8) & 0xF00u) | ((below >> 12) & 0xF000u);
  };
  auto where_hidden = [&](unsigned bits, int r, unsigned then, float x) {  // x, or the bit pattern `then` where hidden
    unsigned t;  // (written out: the compiler makes a shift, a compare and a select of it)
    asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(t) : "v"(bits), "n"(r));
    return __uint_as_float((t & then) | (~t & __float_as_uint(x)));
  };
  f32x16 acc[KT][2];
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    if (kt + 1 < KT) __builtin_amdgcn_s_waitcnt(0x0F70 | TL);  // the next tile may still be in flight
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");
    if (seen(kt)) {
      const unsigned char* slot = own + (kt & 1) * kTile;
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(slot + (rd ^ (ks * kStep)));
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
          acc[kt][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[rt][ks], b, ks == 0 ? f32x16{0} : acc[kt][rt], 0, 0, 0);
      }
      if (masked(kt)) {
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
          const unsigned bits = hidden_bits(kt, rt);
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[kt][rt][r] = where_hidden(bits, r, 0xFF800000u, acc[kt][rt][r]);
        }
      }
    }
    if (kt + 2 < KT) {
      __builtin_amdgcn_s_waitcnt(0xC07F);  // the slot's operands are in registers
      asm volatile("" ::: "memory");
      load_keys(kt + 2);
    }
  }

  // ---- row statistics of the wave's keys
  auto publish = [&](float x) {
    asm volatile("" ::: "memory");  // (the wave's LDS accesses stay in order; the compiler's of other types must too)
    bcast[my_row] = x;
    asm volatile("" ::: "memory");
  };
  auto published = [&](int rt, float (&v)[16]) {  // v[r] <- x of the lane that holds row r of the lane's 16 in row tile rt
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 t = *reinterpret_cast<const f32x4*>(bcast + rt * 32 + g * 8 + h * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[g * 4 + e] = t[e];
    }
  };
  float v[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) v[i] = kNegInf;
#pragma unroll
  for (int kt = 0; kt < KT; ++kt)
    if (seen(kt)) {
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = larger(v[i], acc[kt][i >> 4][i & 15]);
    }
  const float m = reduce32(v, c32, larger) * c;
  publish(m == kNegInf ? 0.f : -m);
  float sum[32];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {  // (a row tile at a time: fewer registers)
    float nm[16];
    published(rt, nm);
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[rt * 16 + r] = 0.f;
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
      if (seen(kt)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float e = fast_exp2(__builtin_fmaf(acc[kt][rt][r], c, nm[r]));
          acc[kt][rt][r] = e;
          sum[rt * 16 + r] += e;
        }
      }
  }
  const float l = reduce32(sum, c32, [](float x, float y) { return x + y; });
  stat_of(wv)[my_row] = make_float2(m, l);
  __syncthreads();

  // ---- the rows' weights 2^(m - L) of this wave's terms, then the column sums
  {
    float M = kNegInf, l_all = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float2 o = stat_of(w)[my_row];
      ml_combine<false>(M, l_all, o.x, o.y);
    }
    publish(row_base + my_row < Mq ? fast_exp2(m - (M + log2f(l_all))) : 0.f);
  }
  float w[2][16];
  published(0, w[0]);
  published(1, w[1]);
  float* const out = parts + ((size_t)unit * blocks + blk) * part_pitch;
#pragma unroll
  for (int kt = 0; kt < KT; ++kt) {
    float s[2] = {0.f, 0.f};
    if (seen(kt)) {
      if (masked(kt)) {  // (a hidden term is 0 whatever the row's weight, a NaN included)
        const unsigned bits[2] = {hidden_bits(kt, 0), hidden_bits(kt, 1)};
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
            s[rt] = __builtin_fmaf(acc[kt][rt][r], where_hidden(bits[rt], r, 0u, w[rt][r]), s[rt]);
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int rt = 0; rt < 2; ++rt) s[rt] = __builtin_fmaf(acc[kt][rt][r], w[rt][r], s[rt]);
      }
    }
    const float mine = s[0] + s[1], tot = mine + __shfl_xor(mine, 32, 64);
    const int key = tile0(kt) + c32;
    if (h == 0 && key < N) out[key] = tot;
  }
}

// ------------------------------------------------------------------ fp32 caches

// What the head dimension decides about a stage (32 stream rows) of the fp32 sweeps.
template <int D>
struct F32Geom {
  static constexpr int kStageRows = 32;
  static constexpr int kPieces = D / 8;                      // 16-byte pieces (eight terms) of a row of a plane
  static constexpr int kPlaneBytes = kStageRows * D * 2;
  static constexpr int kStageBytes = 3 * kPlaneBytes;
  static constexpr int kItems = kStageRows * kPieces / kThreads;  // pieces a thread splits per stage
};

// x = hi + mid + lo, each rounded to bf16: 24 bits, so the three terms are x itself up to 2^-25 of it, or up
// to 2^-125 where that is more (bf16 ends where fp32's normal numbers do: below 2^-109 the third term, below
// 2^-117 the second loses bits).  (A value that rounds past the bf16 range gives an infinity and a NaN,
// like an infinity itself.)
struct Split3 {
  bf16x8 hi, mid, lo;
};
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split_pair(float x0, float x1, Split3& o, int q) {  // terms 2 q and 2 q + 1
  auto round2 = [](float a, float b) { return __builtin_convertvector(f32x2{a, b}, bf16x2); };
  auto first = [](bf16x2 v) { return __uint_as_float(__builtin_bit_cast(uint32_t, v) << 16); };
  auto second = [](bf16x2 v) { return __uint_as_float(__builtin_bit_cast(uint32_t, v) & 0xffff0000u); };
  const bf16x2 hi = round2(x0, x1);
  const float r0 = x0 - first(hi), r1 = x1 - second(hi);
  const bf16x2 mid = round2(r0, r1), lo = round2(r0 - first(mid), r1 - second(mid));
  o.hi[2 * q] = hi[0], o.hi[2 * q + 1] = hi[1];
  o.mid[2 * q] = mid[0], o.mid[2 * q + 1] = mid[1];
  o.lo[2 * q] = lo[0], o.lo[2 * q + 1] = lo[1];
}
__device__ __forceinline__ Split3 split3(const f32x4& a, const f32x4& b) {
  Split3 o;
#pragma unroll
  for (int q = 0; q < 4; ++q) split_pair(q < 2 ? a[2 * q] : b[2 * q - 4], q < 2 ? a[2 * q + 1] : b[2 * q - 3], o, q);
  return o;
}

// Both scoring sweeps of an fp32 cache.  MODE 0 = sweep A (resident: window rows, stream: keys),
// MODE 1 = sweep B (resident: keys, stream: window rows), as for bf16 above: a wave keeps 32 resident
// rows as B operands in registers, and a lane owns one resident row and 16 stream rows of a tile.
//
// The products are bf16 matrix tiles over terms of the operands: with x = hi + mid + lo the product of
// two values is hi hi + (hi mid + mid hi) + (mid mid + hi lo + lo hi) up to 2^-24 of it, products of
// bf16 terms are exact in fp32, and six of them take 6 x 32 cycles for sixteen channels where the
// fp32 tiles (32x32x2) take 8 x 64.  The five small ones have an accumulator of their own, so that the
// large one is rounded once per sixteen channels, not once per two: the result is closer to 64-bit sums
// than the fp32 tiles' was.  The waves of a workgroup that meets a value past the bf16 range, or so large that what its
// partner lost below 2^-125 could show in a logit, take their share again on the fp32 tiles, operands
// straight from memory (rare, slow, exact).
//
// Stream rows are split once per workgroup: a thread loads eight channels three stages ahead, splits them
// and leaves the terms in LDS as three planes, one stage ahead; one barrier a stage.  The 16-byte piece p
// of row r lies at slot p ^ r of its row (d = 64: p ^ r / 2, two rows to 256 bytes), which spreads any
// 16 lanes of an operand read, and of a store, over all banks.
//
// Bound: the matrix pipe (1536 cycles a tile of d = 128).  The clean stages are software-pipelined: the six products
// of a k-step carry two logits of the tile before (fma, exp2, add: the reference is taken once, as in
// the bf16 sweeps, and a sum out of range is taken again) and two channels of the split of the
// stage after.  32 units of 4096 rows, 256 window rows, d = 128: 50 + 53 us, 1.0 PFLOP/s of bf16 products, which
// is what the bf16 sweeps reach (the clock under matrix load is 1.8 GHz); the fp32 tiles took 81 + 94.  Norm
// of the scores' error against 64-bit sums over nine shapes: 1.7e-7 - 3.1e-7, with fp32 products 2.2e-7 - 6.8e-7.
// The resident rows a lane per row from memory, the stream one stage ahead: 64 + 55 us.
template <int D, int MODE>
__global__ __launch_bounds__(kThreads, D == 128 ? 2 : 3) void score_f32_kernel(
    KParams kp, int n_units, int tiles_per_unit, int n_splits, int split_len, int mq_pad,
    const int64_t* __restrict__ row_off, const float* __restrict__ K, const float* __restrict__ Q,
    float2* __restrict__ rowstat, const float* __restrict__ bias, float* __restrict__ bias_out,
    float* __restrict__ scores) {
  using SG = F32Geom<D>;
  constexpr int kStageRows = SG::kStageRows, kPieces = SG::kPieces, kPlane = SG::kPlaneBytes, kItems = SG::kItems;
  constexpr int kRes = kWaves * 32;  // resident rows per workgroup
  constexpr int NK = D / 16;
  __shared__ __attribute__((aligned(16))) unsigned char stage_mem[2 * SG::kStageBytes];
  __shared__ __attribute__((aligned(16))) float negl[4][kStageRows];  // sweep B: -L of the rows of four stages
  __shared__ int too_large;
  int unit, tile;
  if (!map_block(n_units, tiles_per_unit, unit, tile)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c32 = lane & 31, h = lane >> 5;
  const int64_t row0 = row_off[unit];
  const int N = (int)(row_off[unit + 1] - row0);
  const int Mq = kp.Mq, W = kp.W, Gq = kp.G;
  const float c = kp.scale_log2;
  const float* Ku = K + (size_t)row0 * D;
  const float* Qu = Q + (size_t)unit * Mq * D;

  // ---- what this workgroup covers: resident rows [res_base, ..), stream rows [s_begin, s_end)
  const float *res_ptr, *str_ptr;
  int res_base, res_limit, s_begin, s_end, split = 0;
  if (MODE == 0) {
    res_base = tile / n_splits * kRes;
    split = tile % n_splits;
    if (res_base >= Mq) return;
    res_ptr = Qu;
    res_limit = Mq;
    str_ptr = Ku;
    s_begin = split * split_len;
    s_end = min(N, s_begin + split_len);
    if (kp.causal) s_end = min(s_end, N - W + (min(Mq, res_base + kRes) - 1) / Gq + 1);
  } else {
    res_base = tile * kRes;
    if (res_base >= N) return;
    res_ptr = Ku;
    res_limit = N;
    str_ptr = Qu;
    s_begin = 0;
    s_end = Mq;
    if (kp.causal && res_base > N - W) s_begin = ((res_base - (N - W)) * Gq) / kStageRows * kStageRows;
  }
  const int n_stages = s_end > s_begin ? (s_end - s_begin + kStageRows - 1) / kStageRows : 0;
  const int res_row = res_base + wv * 32 + c32;  // the lane's resident row
  const bool wave_live = res_base + wv * 32 < res_limit;

  // ---- rows on their way: 32 at a time, a thread taking eight channels of one (two rows of d = 128) as they
  // lie in memory.  Places past the last row hold that row again: of the stream, sweep A masks them and
  // sweep B's bias makes nothing of them (a zero row times an infinity would be a NaN); resident ones
  // are not stored.
  struct Raw {
    f32x4 v[kItems][2];
    float nl;
  };
  const __amdgpu_buffer_rsrc_t str_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(str_ptr), 0, (int)((unsigned)max(s_end, 0) * (unsigned)(D * 4)), 0x00020000);
  const __amdgpu_buffer_rsrc_t res_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(res_ptr), 0, (int)((unsigned)res_limit * (unsigned)(D * 4)), 0x00020000);
  auto load_rows = [&](Raw& raw, const __amdgpu_buffer_rsrc_t& rsrc, int first, int last) CASK_INLINE {
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const int item = tid + j * kThreads;
      const unsigned at = (unsigned)min(first + item / kPieces, last) * (unsigned)(D * 4) + (item % kPieces) * 32;
      raw.v[j][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, 0, 0));
      raw.v[j][1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, 16, 0));
    }
  };
  auto load_stage = [&](Raw& raw, int st) CASK_INLINE {  // (past the last stage: its last row again)
    load_rows(raw, str_rsrc, s_begin + st * kStageRows, s_end - 1);
    if (MODE == 1 && tid < kStageRows) raw.nl = bias[(size_t)unit * mq_pad + min(s_begin + st * kStageRows + tid, mq_pad - 1)];
  };
  auto swizzle = [](int row, int piece) CASK_INLINE { return row * (D * 2) + ((piece ^ (D == 128 ? row & 15 : (row >> 1) & 7)) * 16); };
  auto slot_of = [&](int st) -> unsigned char* { return stage_mem + (st & 1) * SG::kStageBytes; };
  auto store_item = [&](int st, int j, const Split3& t) CASK_INLINE {
    const int item = tid + j * kThreads;
    unsigned char* p = slot_of(st) + swizzle(item / kPieces, item % kPieces);
    *reinterpret_cast<bf16x8*>(p) = t.hi;
    *reinterpret_cast<bf16x8*>(p + kPlane) = t.mid;
    *reinterpret_cast<bf16x8*>(p + 2 * kPlane) = t.lo;
  };
  auto store_negl = [&](const Raw& raw, int st) CASK_INLINE {
    if (MODE == 1 && tid < kStageRows) negl[st & 3][tid] = raw.nl;
  };
  // the largest value this thread has split: 2^90 / c times 2^-125, over 128 channels and both operands, is
  // 2^-27 of a logit in base 2
  float largest = 0.f;
  auto note_pair = [&](float x0, float x1) CASK_INLINE {
    // (written out: fmaxf would first quiet a NaN in either value, an instruction each)
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(largest) : "v"(x0), "v"(x1));
  };
  auto store_rows = [&](const Raw& raw, int st) CASK_INLINE {
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
#pragma unroll
      for (int q = 0; q < 4; ++q) note_pair(raw.v[j][q >> 1][(q & 1) * 2], raw.v[j][q >> 1][(q & 1) * 2 + 1]);
      store_item(st, j, split3(raw.v[j][0], raw.v[j][1]));
    }
  };
  const int rd = swizzle(c32, h);  // the lane's piece of k-step 0; k-step ks: 32 ks further in the row's order
  auto read_terms = [&](int st, int ks) CASK_INLINE {
    const unsigned char* p = slot_of(st) + (rd ^ (ks * 32));
    Split3 t;
    t.hi = *reinterpret_cast<const bf16x8*>(p);
    t.mid = *reinterpret_cast<const bf16x8*>(p + kPlane);
    t.lo = *reinterpret_cast<const bf16x8*>(p + 2 * kPlane);
    return t;
  };
  auto stage_barrier = [&]() CASK_INLINE {  // this wave's LDS accesses are done; its loads stay in flight
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // Stream stage st waits in even or odd (st & 1) until it is split, loaded three stages ahead of its use.
  // The resident rows come the same way, whole rows at a time (a lane per row, each load would touch
  // 32 rows at 32 bytes each), two waves' at a time.
  Split3 res[NK];
  Raw even, odd;
  if (tid == 0) too_large = 0;  // (a barrier follows wherever there are stages)
  if (n_stages > 0) {
    Raw mine[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) load_rows(mine[w], res_rsrc, res_base + w * 32, res_limit - 1);
    load_stage(even, 0);
    load_stage(odd, 1);
#pragma unroll
    for (int w = 0; w < kWaves; w += 2) {
      store_rows(mine[w], 0);
      store_rows(mine[w + 1], 1);
      stage_barrier();
      if ((wv & 2) == w) {
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) res[ks] = read_terms(wv, ks);
      }
      stage_barrier();
    }
    store_rows(even, 0);
    store_negl(even, 0);
    load_stage(even, 2);
  }

  // stages [0, sk) show the wave nothing, [sk, f0) and [f1, n_stages) are partly masked
  int sk = 0, f0 = 0, f1 = n_stages;
  int lim = 0, first_row = 0;
  if (MODE == 0) {
    lim = min(s_end - 1, kp.causal ? N - W + res_row / Gq : N - 1);  // last key the lane's row sees
    const int clean_rows = min((kp.causal ? N - W : N) + 1, s_end) - s_begin;
    f1 = clean_rows > 0 ? min(n_stages, clean_rows / kStageRows) : 0;
  } else if (kp.causal) {
    const int k0 = res_base + wv * 32 - (N - W);  // the wave's oldest key, relative to the window
    first_row = max(0, (res_row - (N - W)) * Gq);  // first window row that sees the lane's key
    sk = max(0, min(n_stages, (max(0, k0 * Gq) - s_begin) / kStageRows));
    f0 = max(sk, min(n_stages, (max(0, (k0 + 31) * Gq) - s_begin + kStageRows - 1) / kStageRows));
  }
  if (!wave_live) sk = n_stages;  // only loads, splits and barriers

  float m_ref = kNegInf, l_run = 0.f, colsum = 0.f;
  // a finished tile of stage `it` into the sums; nl: -L of the lane's sixteen rows (sweep B)
  auto tally = [&](f32x16& acc, const float (&nl)[16], int it) {
    const int trow = s_begin + it * kStageRows + h * 4;  // first stream row of the lane
    if (MODE == 0) {
      if (it >= f1) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (trow + (r >> 2) * 8 + (r & 3) > lim) acc[r] = kNegInf;
      }
      float xm = acc[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) xm = fmaxf(xm, acc[r]);
      const float m_new = fmaxf(m_ref, xm * c);
      const float nm = (m_new == kNegInf) ? 0.f : -m_new;
      float sum = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) sum += fast_exp2(__builtin_fmaf(acc[r], c, nm));
      l_run = l_run * fast_exp2(m_ref + nm) + sum;
      m_ref = m_new;
    } else {
      float sum = 0.f;
      if (it < f0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float y = __builtin_fmaf(acc[r], c, nl[r]);
          sum += fast_exp2(trow + (r >> 2) * 8 + (r & 3) < first_row ? kNegInf : y);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += fast_exp2(__builtin_fmaf(acc[r], c, nl[r]));
      }
      colsum += sum;
    }
  };
  f32x16 acc, small;
  auto products = [&](const Split3& a, int ks) CASK_INLINE {
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.lo, res[ks].hi, ks == 0 ? f32x16{0} : small, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi, res[ks].hi, ks == 0 ? f32x16{0} : acc, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi, res[ks].lo, small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.mid, res[ks].mid, small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.mid, res[ks].hi, small, 0, 0, 0);
    small = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.hi, res[ks].mid, small, 0, 0, 0);
  };
  auto load_nl = [&](float (&nl)[16], int it) {
    if (MODE == 1) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(&negl[it & 3][g * 8 + h * 4]);
        nl[g * 4 + 0] = v[0]; nl[g * 4 + 1] = v[1]; nl[g * 4 + 2] = v[2]; nl[g * 4 + 3] = v[3];
      }
    }
  };
  // one stage, nothing overlapped; leaves the tile's logits in acc
  auto plain_chain = [&](int it) CASK_INLINE {
    Split3 a = read_terms(it, 0);
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
      products(a, ks);
      if (ks + 1 < NK) a = read_terms(it, ks + 1);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] += small[r];
  };
  // Stage `it` is whole behind the barrier, and stage it - 1 has been read by everyone.  `raw` holds stage
  // it + 1: even behind an odd stage.  (Named at every call, and the loops run two stages at a time: chosen
  // by a branch, the loads go to other registers, and the copy waits for them.)
  auto next_stage = [&](int it, Raw& raw) CASK_INLINE {
    stage_barrier();
    store_rows(raw, it + 1);
    store_negl(raw, it + 1);
    load_stage(raw, it + 3);
  };
  auto plain_stage = [&](int it, Raw& raw) CASK_INLINE {
    next_stage(it, raw);
    if (it < sk) return;
    plain_chain(it);
    float nl[16];
    load_nl(nl, it);
    tally(acc, nl, it);
  };
  auto plain = [&](int from, int to) CASK_INLINE {
    if ((from & 1) && from < to) plain_stage(from++, even);
    for (; from + 1 < to; from += 2) {
      plain_stage(from, odd);
      plain_stage(from + 1, even);
    }
    if (from < to) plain_stage(from, odd);
  };
  auto pipelined = [&](int from, int to) CASK_INLINE {  // clean stages, to > from, from even
    next_stage(from, odd);
    plain_chain(from);
    if (MODE == 0) {  // (always the first stages of the workgroup) at most 16 above the row's largest logit so far
      float top = acc[0], low = acc[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) {
        top = fmaxf(top, acc[r]);
        low = fminf(low, acc[r]);
      }
      m_ref = __builtin_fmaf(top, c, fminf(0.3f * c * (top - low), 16.f));
    }
    f32x16 old = acc;
    float sum = 0.f;
    auto bank = [&]() CASK_INLINE {
      if (MODE == 0) l_run += sum;
      else colsum += sum;
      sum = 0.f;
    };
    auto body = [&](int it, Raw& raw) CASK_INLINE {
      stage_barrier();
      Split3 a = read_terms(it, 0);
      Split3 t;
      store_negl(raw, it + 1);
#pragma unroll
      for (int ks = 0; ks < NK; ++ks) {
        constexpr int kTerms = 16 / NK;  // 2 or 4 logits of the old tile
        float nl[4];
        if (MODE == 1) {
          const int r0 = ks * kTerms;
          const f32x4 v = *reinterpret_cast<const f32x4*>(&negl[(it - 1) & 3][(r0 >> 2) * 8 + h * 4]);
#pragma unroll
          for (int e = 0; e < kTerms; ++e) nl[e] = v[(r0 & 3) + e];
        }
        Split3 next = a;
        if (ks + 1 < NK) next = read_terms(it, ks + 1);
        products(a, ks);
#pragma unroll
        for (int e = 0; e < kTerms; ++e) sum += fast_exp2(__builtin_fmaf(old[ks * kTerms + e], c, MODE == 0 ? -m_ref : nl[e]));
        const int j = ks / 4, q = ks % 4;
        split_pair(raw.v[j][q >> 1][(q & 1) * 2], raw.v[j][q >> 1][(q & 1) * 2 + 1], t, q);
        note_pair(raw.v[j][q >> 1][(q & 1) * 2], raw.v[j][q >> 1][(q & 1) * 2 + 1]);
        if (q == 3) store_item(it + 1, j, t);
        // (pinned: the optimiser would sink the sum out of the products it is meant to overlap with)
        asm volatile("" : "+v"(sum));
        __builtin_amdgcn_sched_barrier(0);
        a = next;
      }
      bank();
      load_stage(raw, it + 3);
#pragma unroll
      for (int r = 0; r < 16; ++r) old[r] = acc[r] + small[r];
    };
    int it = from + 1;
    for (; it + 1 < to; it += 2) {
      body(it, even);
      body(it + 1, odd);
    }
    if (it < to) body(it, even);
    float nl[16];
    load_nl(nl, to - 1);
#pragma unroll
    for (int r = 0; r < 16; ++r) sum += fast_exp2(__builtin_fmaf(old[r], c, MODE == 0 ? -m_ref : nl[r]));
    bank();
  };
  if (!wave_live || MODE == 1) {
    const int from = (f0 + 1) & ~1;
    plain(0, wave_live ? min(from, n_stages) : n_stages);
    if (wave_live && from < n_stages) pipelined(from, n_stages);
  } else {
    int first = 0;
    asm volatile("" : "+s"(first));
    if (f1 > 0) pipelined(first, f1);
    plain(f1, n_stages);
  }

  // ---- out of range somewhere: the wave's share again with a running maximum, operands from memory.  The products
  // are the same, so that a logit has the same bits in both sweeps (its rounding then cancels against that of
  // the row's sum, which is most of it where one key has the row's mass); fp32 ones where a value is too large.
  const float total = MODE == 0 ? l_run : colsum;
  if (n_stages > 0 && !(largest * c < 0x1p90f && largest < 0x1.fep127f)) too_large = 1;
  __syncthreads();
  const bool fp32_tiles = too_large != 0;
  if (fp32_tiles || __builtin_amdgcn_ballot_w64(wave_live && !(total < kMostSum)) != 0ull) {
    m_ref = kNegInf;
    l_run = colsum = 0.f;
    const float* bp = res_ptr + (size_t)min(res_row, res_limit - 1) * D;
    for (int it = sk; it < n_stages; ++it) {
      const int srow = s_begin + it * kStageRows;
      const float* ap = str_ptr + (size_t)min(srow + c32, s_end - 1) * D;
      if (fp32_tiles) {
        acc = f32x16{0};
        for (int p = 0; p < D / 8; ++p) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(ap + p * 8 + h * 4), y = *reinterpret_cast<const f32x4*>(bp + p * 8 + h * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], y[e], acc, 0, 0, 0);
        }
      } else {
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
          const float* p = ap + ks * 16 + h * 8;
          products(split3(*reinterpret_cast<const f32x4*>(p), *reinterpret_cast<const f32x4*>(p + 4)), ks);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] += small[r];
      }
      float nl[16];
      if (MODE == 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          nl[r] = bias[(size_t)unit * mq_pad + min(srow + (r >> 2) * 8 + h * 4 + (r & 3), mq_pad - 1)];
      }
      tally(acc, nl, it);
    }
  }

  if (MODE == 0) {
    const float m2 = __shfl_xor(m_ref, 32, 64), l2 = __shfl_xor(l_run, 32, 64);
    ml_combine<true>(m_ref, l_run, m2, l2);
    if (h == 0 && res_row < Mq)
      rowstat[((size_t)unit * n_splits + split) * mq_pad + res_row] = make_float2(m_ref, l_run);
    if (n_splits == 1 && h == 0 && res_row < mq_pad)  // a single split is the whole row
      bias_out[(size_t)unit * mq_pad + res_row] = res_row < Mq ? -(m_ref + log2f(l_run)) : kPadNegL;
  } else {
    const float tot = colsum + __shfl_xor(colsum, 32, 64);
    if (h == 0 && res_row < N) scores[row0 + res_row] = tot * (1.0f / (float)Mq);
  }
}

template <int D>
hipError_t launch_score_f32(const KParams& kp, const Batch& b, const Workspace& wl, char* ws,
                            float* scores, hipStream_t st, hipEvent_t between) {
  float2* rowstat = reinterpret_cast<float2*>(ws + wl.rowstat);
  float* bias = reinterpret_cast<float*>(ws + wl.bias);
  const float *K = static_cast<const float*>(b.K), *Q = static_cast<const float*>(b.Q);
  const int tilesA = (kp.Mq + kWaves * 32 - 1) / (kWaves * 32) * wl.n_splits;
  score_f32_kernel<D, 0><<<dim3(mapped_blocks(b.n_units, tilesA)), dim3(kThreads), 0, st>>>(
      kp, b.n_units, tilesA, wl.n_splits, wl.split_len, wl.mq_pad, b.row_off, K, Q, rowstat, nullptr, bias, scores);
  if (between) (void)hipEventRecord(between, st);
  if (wl.n_splits > 1)
    score_bias_kernel<<<dim3(b.n_units), dim3(kBiasThreads), 0, st>>>(kp, wl.n_splits, wl.mq_pad, rowstat, bias);
  const int tilesB = (b.max_unit_len + kWaves * 32 - 1) / (kWaves * 32);
  score_f32_kernel<D, 1><<<dim3(mapped_blocks(b.n_units, tilesB)), dim3(kThreads), 0, st>>>(
      kp, b.n_units, tilesB, wl.n_splits, wl.split_len, wl.mq_pad, b.row_off, K, Q, rowstat, bias, nullptr, scores);
  return hipGetLastError();
}

}  // namespace

bool score_uses_mfma(const KParams& kp) { return kp.dtype == CASK_BF16; }

namespace {
// One instance of the scoring kernel on a stream; raises its LDS limit on the first launch.
template <int D, int MODE, int CT, bool RING_RES>
hipError_t launch_sweep(int blocks, size_t lds, hipStream_t st, const KParams& kp, int n_units, int tiles,
                        int n_splits, int split_len, int q_splits, int mq_pad, const int64_t* row_off,
                        const void* K, const void* Q, float2* rowstat, const float* bias, float* bias_out,
                        float* scores, float* parts, int parts_pitch) {
  static LdsLimitOnce lim;
  const hipError_t e = lim.ensure(reinterpret_cast<const void*>(&score_mfma_kernel<D, MODE, CT, RING_RES>), 160 * 1024);
  if (e != hipSuccess) return e;
  score_mfma_kernel<D, MODE, CT, RING_RES><<<dim3(blocks), dim3(kThreads), lds, st>>>(
      kp, n_units, tiles, n_splits, split_len, q_splits, mq_pad, row_off, static_cast<const uint16_t*>(K),
      static_cast<const uint16_t*>(Q), rowstat, bias, bias_out, scores, parts, parts_pitch);
  return hipSuccess;
}

template <int D>
hipError_t launch_score_mfma(const KParams& kp, const Batch& b, const Workspace& wl, char* ws, float* scores,
                             hipStream_t st, hipEvent_t between) {
  float2* rowstat = reinterpret_cast<float2*>(ws + wl.rowstat);
  float* bias = reinterpret_cast<float*>(ws + wl.bias);
  const size_t lds = (size_t)kDepth * StageGeom<D>::kStageBytes;
  // W*G <= 512 (one wide row block per unit, eight stream stages per workgroup of sweep B): the
  // resident rows come through the ring (measured: both sweeps 3 - 4 % faster on the Llama-shaped
  // batch, up to 4 % slower at W*G = 896)
  const bool ring_res = kp.Mq <= 2 * kResRows;
  auto sweep_a = [&](auto kern, int block_rows) {
    const int tiles = (kp.Mq + block_rows - 1) / block_rows * wl.n_splits;
    return kern(mapped_blocks(b.n_units, tiles), lds, st, kp, b.n_units, tiles, wl.n_splits, wl.split_len, wl.q_splits, wl.mq_pad,
                b.row_off, b.K, b.Q, rowstat, nullptr, bias, scores, nullptr, 0);
  };
  auto sweep_b = [&](auto kern, int block_rows) {
    const int tiles = (b.max_unit_len + block_rows - 1) / block_rows * wl.q_splits;
    return kern(mapped_blocks(b.n_units, tiles), lds, st, kp, b.n_units, tiles, wl.n_splits, wl.split_len, wl.q_splits, wl.mq_pad,
                b.row_off, b.K, b.Q, rowstat, bias, nullptr, scores, nullptr, 0);
  };
  hipError_t e;
  if (!wl.wide_rows) e = sweep_a(&launch_sweep<D, 0, 2, false>, kResRows);
  else if (ring_res) e = sweep_a(&launch_sweep<D, 0, 4, true>, 2 * kResRows);
  else e = sweep_a(&launch_sweep<D, 0, 4, false>, 2 * kResRows);
  if (e != hipSuccess) return e;
  if (between) (void)hipEventRecord(between, st);  // right behind sweep A: the stage is that kernel alone
  if (wl.n_splits > 1)  // with one split sweep A has written -L itself
    score_bias_kernel<<<dim3(b.n_units), dim3(kBiasThreads), 0, st>>>(kp, wl.n_splits, wl.mq_pad, rowstat, bias);
  if (!wl.wide_cols) e = sweep_b(&launch_sweep<D, 1, 2, false>, kResRows);
  else if (ring_res) e = sweep_b(&launch_sweep<D, 1, 4, true>, 2 * kResRows);
  else e = sweep_b(&launch_sweep<D, 1, 4, false>, 2 * kResRows);
  return e != hipSuccess ? e : hipGetLastError();
}
}  // namespace

hipError_t launch_score(const KParams& kp, const Batch& b, const Workspace& wl, char* ws,
                        float* scores, hipStream_t st, hipEvent_t between) {
  if (kp.dtype == CASK_F32)
    return kp.d == 64 ? launch_score_f32<64>(kp, b, wl, ws, scores, st, between)
                      : launch_score_f32<128>(kp, b, wl, ws, scores, st, between);
  return kp.d == 64 ? launch_score_mfma<64>(kp, b, wl, ws, scores, st, between)
                    : launch_score_mfma<128>(kp, b, wl, ws, scores, st, between);
}

namespace {
__global__ __launch_bounds__(256) void clear_scores_kernel(float* __restrict__ scores, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * 256 * 4;
  for (int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4; i < n; i += stride) {
    if (i + 3 < n) {
      *reinterpret_cast<float4*>(scores + i) = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
      for (int64_t j = i; j < n; ++j) scores[j] = 0.f;
    }
  }
}
}  // namespace

// Both sweeps in one launch for units of any length: pays when a workgroup of the second sweep
// would stream few window rows (at most eight stages behind a full prologue) and there are
// enough (unit, row block) pairs to fill the chip several times over.  Its waves hold 64 window
// rows each; with 256 < W*G <= 512 the two separate sweeps in their wide form (128 resident rows
// per wave) are faster (a Llama-shaped ragged batch: 10.7 against 11.4 ms), so the one launch is
// left to W*G <= 256 unless the caller asks for it.
bool score_fused_fits(const KParams& kp, const Batch& b) {
  const int row_blocks = (kp.Mq + kResRows - 1) / kResRows;
  if (!score_uses_mfma(kp) || kp.Mq > 2 * kResRows || (kp.path_flags & CASK_PATH_NO_FUSED_SWEEPS)) return false;
  if (kp.path_flags & CASK_PATH_FORCE_FUSED_SWEEPS) return true;
  if (kp.Mq > kResRows && !(kp.path_flags & CASK_PATH_NARROW_ROWS)) return false;
  return (int64_t)b.n_units * row_blocks >= 1024;
}

namespace {
template <int D>
hipError_t launch_fused_sweeps(const KParams& kp, const Batch& b, const Workspace& wl, float* scores, hipStream_t st) {
  const size_t lds = (size_t)kDepth * StageGeom<D>::kStageBytes + kResRows * sizeof(float) + 4 * kWaves * 64 * sizeof(float);
  const int qblocks = (kp.Mq + kResRows - 1) / kResRows;
  const int whole = (b.max_unit_len + kStageRows - 1) / kStageRows * kStageRows;
  return launch_sweep<D, 3, 2, false>(mapped_blocks(b.n_units, qblocks), lds, st, kp, b.n_units, qblocks, 1, whole, 1,
                                      wl.mq_pad, b.row_off, b.K, b.Q, nullptr, nullptr, nullptr, scores, nullptr, 0);
}

template <int D>
hipError_t launch_sweeps_to_parts(const KParams& kp, const Batch& b, const Workspace& wl, float* parts, hipStream_t st) {
  const size_t lds = (size_t)kDepth * StageGeom<D>::kStageBytes + kResRows * sizeof(float);
  const int qblocks = (kp.Mq + kResRows - 1) / kResRows;
  return launch_sweep<D, 2, 2, false>(mapped_blocks(b.n_units, qblocks), lds, st, kp, b.n_units, qblocks, 1, wl.split_len,
                                      1, wl.mq_pad, b.row_off, b.K, b.Q, nullptr, nullptr, nullptr, nullptr, parts,
                                      wl.parts_pitch);
}

template <int D>
hipError_t launch_short(const KParams& kp, const Batch& b, float* parts, int pitch, hipStream_t st) {
  const int blocks = (kp.Mq + 63) / 64, grid = mapped_blocks(b.n_units, blocks);
  auto go = [&](auto kt, auto nw) {
    score_short_kernel<D, decltype(kt)::value, decltype(nw)::value><<<dim3(grid), dim3(decltype(nw)::value * 64), 0, st>>>(
        kp, b.n_units, blocks, b.row_off, static_cast<const uint16_t*>(b.K), static_cast<const uint16_t*>(b.Q), parts, pitch);
    return hipGetLastError();
  };
  using std::integral_constant;
  const integral_constant<int, 4> four;
  const integral_constant<int, 8> eight;
  const int tiles = (b.max_unit_len + 31) / 32;
  // Two workgroups of four waves share a compute unit up to 640 rows.  Where a workgroup has the
  // compute unit to itself anyway, and beyond 640 rows, it takes eight waves.
  if (grid > 256 && tiles <= 20) {
    if (tiles <= 8) return go(integral_constant<int, 2>(), four);
    if (tiles <= 12) return go(integral_constant<int, 3>(), four);
    if (tiles <= 16) return go(four, four);
    return go(integral_constant<int, 5>(), four);
  }
  if (tiles <= 16) return go(integral_constant<int, 2>(), eight);
  if (tiles <= 24) return go(integral_constant<int, 3>(), eight);
  return go(four, eight);
}
}  // namespace

hipError_t launch_score_fused(const KParams& kp, const Batch& b, const Workspace& wl, float* scores,
                              hipStream_t st) {
  if (!score_fused_fits(kp, b)) return hipErrorInvalidValue;
  if (kp.Mq > kResRows) {
    // two workgroups add onto each key's score; scores is 4-byte aligned only: float4 stores need 16
    const bool al16 = (reinterpret_cast<uintptr_t>(scores) & 15u) == 0;
    if (al16) {
      const int64_t n = b.total_rows;
      const int blocks = (int)((n / 4 + 255) / 256 < 8192 ? (n / 4 + 255) / 256 + 1 : 8192);
      clear_scores_kernel<<<dim3(blocks), dim3(256), 0, st>>>(scores, n);
    } else {
      return hipErrorInvalidValue;
    }
  }
  const hipError_t e = kp.d == 64 ? launch_fused_sweeps<64>(kp, b, wl, scores, st)
                                  : launch_fused_sweeps<128>(kp, b, wl, scores, st);
  return e != hipSuccess ? e : hipGetLastError();
}

bool score_parts_fits(const KParams& kp, const Batch& b, const Workspace& wl) {
  return score_uses_mfma(kp) && wl.n_splits == 1 && wl.parts_pitch > 0 && b.max_unit_len <= wl.parts_pitch;
}

// Scores of short units in one launch: writes, for every unit, ceil(W*G / 64) partial column
// sums per key, `parts[unit][part][key]` with row pitch wl.parts_pitch; score[key] = (sum of the
// parts in order) / (W*G).
// Two sweeps with 256 window rows to a workgroup overlap matrix and vector work and are the better
// form once they fill the chip several times; one sweep, with its 64 rows to a workgroup, is before
// that.  The line is where it was measured: up to 512 workgroups of 64 rows one sweep wins at every
// length, also where its eight-wave form (one workgroup to a compute unit) needs a second turn of the
// chip, and at 896 it no longer does.  Events, two sweeps against one, d = 128: 56 workgroups (4 units
// of 512) 40 / 28 us, 112 (8 of 1024) 89 / 66, 280 (20 of 1024) 75 / 64, 504 (36 of 1024) 77 / 66, 504 (36
// of 700) 55 / 48, 512 (64 of 1024) 76 / 65, 512 (128 of 500) 45 / 37, 512 (512 of 1024) 192 / 179; 896 (64 of 512)
// 44 / 45, 896 (64 of 1024) 100 / 112, 1568 (112 of 1024) 138 / 163, 8192 (512 of 900) 380 / 531.
// d = 64: 504 (36 of 1024) 68 / 56, 504 (36 of 700) 50 / 43, 512 (512 of 1024) 133 / 124.
hipError_t launch_score_parts(const KParams& kp, const Batch& b, const Workspace& wl, char* ws,
                              hipStream_t st) {
  if (!score_parts_fits(kp, b, wl)) return hipErrorInvalidValue;
  float* parts = reinterpret_cast<float*>(ws + wl.parts);
  if ((int64_t)b.n_units * ((kp.Mq + 63) / 64) <= 512)
    return kp.d == 64 ? launch_short<64>(kp, b, parts, wl.parts_pitch, st) : launch_short<128>(kp, b, parts, wl.parts_pitch, st);
  const hipError_t e = kp.d == 64 ? launch_sweeps_to_parts<64>(kp, b, wl, parts, st)
                                  : launch_sweeps_to_parts<128>(kp, b, wl, parts, st);
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace cask
