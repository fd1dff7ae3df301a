// Consumer side: one decode step's attention over a compressed cache, with the proportional
// bias ln(count) for rows that stand for several original tokens (the paper's folds preserve
// group mass, Section 2.4; how attention uses it is left open there: this is the rule under
// which a fold of identical tokens is lossless).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "cask.h"
#include "cask_common.h"

namespace cask {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kNegInf = -__builtin_inff();
constexpr int kAttHeads = 16;  // query heads per pass over the cache: the columns of a 16x16 product

// Sizes that follow from the cache's element type and head dimension.
template <typename T, int D>
struct AttGeom {
  static constexpr bool kBf16 = sizeof(T) == 2;
  static constexpr int kTileRows = kBf16 ? 32 : 16;          // cache rows a wave takes at a time
  static constexpr int kKeys = kTileRows / 4;                // of them per lane group (16 lanes)
  static constexpr int kSub = kTileRows / 16;                // 16-row subtiles of the logit product
  static constexpr int kSteps = D * (int)sizeof(T) / 64;     // 16-byte pieces of a key row per lane
  static constexpr int EPV = (kBf16 && D == 128) ? 8 : 4;    // elements of a value row per lane and load
  static constexpr int kValLoads = D / (16 * EPV);           // loads per value row
  static constexpr int kBlocks = D / 16;                     // 16-channel blocks of the value product
  typedef typename std::conditional<EPV * sizeof(T) == 16, u32x4, u32x2>::type ValVec;
  // channel of row m of block b of the value product
  __device__ static int channel(int b, int m) { return (b / EPV) * (16 * EPV) + m * EPV + b % EPV; }
};

// A workgroup takes the tiles of one unit (or, with `splits` > 1, every splits-th round of them),
// dealt to its waves round robin.  Per tile two products on 16x16 matrix tiles:
//   logits   S[key][head]     = K_tile . Q^T       (lane: key or head = lane % 16, 16 bytes of channels)
//   values   O[channel][head] += V_tile^T . P      (lane: channel or head = lane % 16, keys of group lane / 16)
// A lane ends the first product with one head's logits of the kKeys keys 16 t + 4 (lane / 16) + r,
// takes the online-softmax step on them and holds its weights as the second product's operand as
// they stand.  The values need no turning round either: lane (m, group) loads its 16-channel-wide
// share of the value rows of its group's own keys, and the product's channel rows are numbered so
// that row m of block b is the channel the lane already holds (AttGeom::channel): an 8-key operand
// is put together from two rows' words by one byte permutation per word.  Nothing but a tile's 32
// biases passes through LDS inside the loop, and nothing there is a workgroup barrier.
// (The former kernel wrote the value rows transposed to LDS two bytes at a time, 64 stores per
// lane and tile, and used 8 columns of 32x32 products.)
// bf16 weights enter as two terms, p = hi + lo (lo the rounded remainder: 2^-17 in all).
// fp32: a logit's D products are summed in chains of eight, the chains in pairs; the scaled logit meets
// its reference inside one rounding; a tile's weighted values are summed on their own before they
// join the long sum over the unit's rows.  Against 64-bit sums, norm of the error over norm of the
// result: 128 units x 2000 rows, d = 128 9.9e-7 with one chain throughout, 3.3e-7 (a thread group per
// row on the vector units: 4.1e-7); 4 x 100 6.5e-7, 2.0e-7 (3.1e-7).
//
// The first tile's rows are requested before the unit's length arrives (any row below `stride`
// is readable; rows past the end get weight zero and zeroed values); after that the next tile's keys are requested behind the first product, its values behind the second.
// At the end the waves' states are merged in wave order (with splits: written out unnormalised for
// attend_combine_kernel, which adds them in split order): the same bits every run.
template <typename T, int D, int WAVES, bool NT>
__global__ __launch_bounds__(WAVES * 64, 8 / WAVES) void attend_kernel(
    KParams kp, const T* __restrict__ Q, const T* __restrict__ Kc, const T* __restrict__ Vc, int stride,
    const int32_t* __restrict__ len, const int32_t* __restrict__ count, int count_pitch, T* __restrict__ out,
    int splits, float* __restrict__ part) {
  using A = AttGeom<T, D>;
  typedef typename A::ValVec ValVec;
  constexpr int TR = A::kTileRows, KEYS = A::kKeys, SUB = A::kSub, KS = A::kSteps, NB = A::kBlocks, EPV = A::EPV, NV = A::kValLoads;
  constexpr int kAccPitch = D + 4;
  constexpr int ROWB = D * (int)sizeof(T);
  constexpr int kAux = NT ? 2 : 0;  // cache policy of the row loads: non-temporal or default
  extern __shared__ __align__(16) unsigned char att_lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int u = blockIdx.x / splits, sp = blockIdx.x % splits;
  const int G = kp.G;
  const int heads = G < kAttHeads ? G : kAttHeads;
  float* bias_s = reinterpret_cast<float*>(att_lds) + wv * 32;
  float* st_m = reinterpret_cast<float*>(att_lds) + WAVES * 32;  // [WAVES][16]
  float* st_l = st_m + WAVES * kAttHeads;
  float* st_acc = st_l + WAVES * kAttHeads;                      // [WAVES][heads][kAccPitch]
  const T* Ku = Kc + (size_t)u * stride * D;
  const T* Vu = Vc + (size_t)u * stride * D;
  const int32_t* cu = count ? count + (size_t)u * count_pitch : nullptr;
  const float c = kp.scale_log2;  // softmax scale * log2(e)
  const int step = splits * WAVES;
  const int first = sp * WAVES + wv;  // the wave's first tile

  u32x4 ka[SUB][KS];
  ValVec va[KEYS][NV];
  int cn = 1;
  // A tile's rows through a descriptor of their own that ends with the unit (`rows` of it): rows past
  // the end read as zero, tiles past the end touch no memory, and a lane needs one 32-bit offset
  // for all of its loads, however long the unit.
  auto tile_rsrc = [&](const T* base, int t, int rows) {
    const int left = rows - t * TR;
    // (the clamp is one vector instruction: a descriptor made of its result as it stands is taken to
    // differ between lanes, and every load becomes a loop.  256 units of 512 rows 15.0 -> 14.3 us)
    const int bytes = __builtin_amdgcn_readfirstlane((left > TR ? TR : (left > 0 ? left : 0)) * ROWB);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(base + (size_t)(left > 0 ? t * TR : 0) * D), 0, bytes, 0x00020000);
  };
  const int k_off = l16 * ROWB + g * 16, v_off = g * 4 * ROWB + l16 * (EPV * (int)sizeof(T));
  auto load_keys = [&](int t, int rows) {
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(Ku, t, rows);
#pragma unroll
    for (int y = 0; y < SUB; ++y)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        ka[y][ks] = __builtin_amdgcn_raw_buffer_load_b128(rs, k_off + ks * 64, y * 16 * ROWB, kAux);
    if (cu) {
      const int r = t * TR + (lane & (TR - 1));
      cn = cu[min(r, count_pitch - 1)];
      if (r >= count_pitch) cn = 1;  // rows behind the counted ones stand for themselves
    }
  };
  auto load_values = [&](int t, int rows) {
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(Vu, t, rows);
#pragma unroll
    for (int j = 0; j < KEYS; ++j)
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int at = (j & 3) * ROWB + q * (16 * EPV * (int)sizeof(T)), sub = (j >> 2) * 16 * ROWB;
        if constexpr (sizeof(ValVec) == 16) va[j][q] = __builtin_amdgcn_raw_buffer_load_b128(rs, v_off + at, sub, kAux);
        else va[j][q] = __builtin_amdgcn_raw_buffer_load_b64(rs, v_off + at, sub, kAux);
      }
  };

  for (int g0 = 0; g0 < G; g0 += kAttHeads) {
    load_keys(first, stride);
    load_values(first, stride);
    // the query operand: head l16, the same channels in the same order as the keys
    u32x4 q[KS];
    {
      const bool head = g0 + l16 < G;
      const T* qp = Q + ((size_t)u * G + (head ? g0 + l16 : 0)) * D;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        q[ks] = *reinterpret_cast<const u32x4*>(qp + (ks * 4 + g) * (16 / sizeof(T)));
        if (!head) q[ks] = u32x4{0u, 0u, 0u, 0u};
      }
    }
    int L = len[u];
    L = L < 0 ? 0 : (L > stride ? stride : L);
    const int n_tiles = (L + TR - 1) / TR;

    float m_run = kNegInf, l_run = 0.f;  // of head l16, l_run over the keys of this lane
    f32x4 acc[NB];                       // acc[b][r] = O[channel(b, 4 g + r)][head l16]
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};

    for (int t = first; t < n_tiles; t += step) {
      const bool partial = t * TR + TR > L;
      if (cu || partial) {  // bias of a row of the tile: log2(count), or -inf past the end of the unit
        const int r = lane & (TR - 1);
        const float b = t * TR + r < L ? (cn > 1 ? __log2f((float)cn) : 0.f) : kNegInf;
        if (lane < TR) bias_s[r] = b;
      }
      f32x4 s[SUB];
#pragma unroll
      for (int y = 0; y < SUB; ++y) {
        s[y] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (A::kBf16) {
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            s[y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ka[y][ks]),
                                                           __builtin_bit_cast(bf16x8, q[ks]), s[y], 0, 0, 0);
        } else {
          f32x4 part[KS / 2];
#pragma unroll
          for (int pair = 0; pair < KS / 2; ++pair) {
            f32x4 a[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const f32x4 kf = __builtin_bit_cast(f32x4, ka[y][2 * pair + (e >> 1)]), qf = __builtin_bit_cast(f32x4, q[2 * pair + (e >> 1)]);
              a[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[2 * (e & 1)], qf[2 * (e & 1)], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
              a[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[2 * (e & 1) + 1], qf[2 * (e & 1) + 1], a[e], 0, 0, 0);
            }
            part[pair] = (a[0] + a[1]) + (a[2] + a[3]);
            asm volatile("" : "+v"(part[pair]));  // (the compiler would put the additions off and hold all sixteen sums)
          }
#pragma unroll
          for (int o = KS / 4; o > 0; o >>= 1)
#pragma unroll
            for (int h = 0; h < o; ++h) part[h] += part[h + o];
          s[y] = part[0];
        }
      }
      load_keys(t + step, L);  // the product is done with this tile's key rows
      // s[y][r] = <key 16 y + 4 g + r, head l16>
      float p[KEYS], mx = kNegInf;
      f32x4 bias4[SUB];
#pragma unroll
      for (int y = 0; y < SUB; ++y) bias4[y] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (cu || partial) {
#pragma unroll
        for (int y = 0; y < SUB; ++y) {
          bias4[y] = *reinterpret_cast<const f32x4*>(&bias_s[y * 16 + g * 4]);
#pragma unroll
          for (int r = 0; r < 4; ++r)  // (a row past the end may hold anything)
            p[y * 4 + r] = bias4[y][r] == kNegInf ? kNegInf : __builtin_fmaf(s[y][r], c, bias4[y][r]);
        }
        if (partial && t == first) {  // (later tiles were read with the unit's length known)
#pragma unroll
          for (int j = 0; j < KEYS; ++j)
            if (t * TR + (j >> 2) * 16 + g * 4 + (j & 3) >= L)
#pragma unroll
              for (int y = 0; y < NV; ++y) va[j][y] = ValVec(0u);
        }
      } else {
#pragma unroll
        for (int j = 0; j < KEYS; ++j) p[j] = s[j >> 2][j & 3] * c;
      }
#pragma unroll
      for (int j = 0; j < KEYS; ++j) mx = fmaxf(mx, p[j]);
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      // (fp32: the logit meets its reference inside one rounding)
      auto shifted = [&](int j, float reference) {
        if constexpr (A::kBf16) return p[j] - reference;
        const float b = bias4[j >> 2][j & 3];
        return b == kNegInf ? kNegInf : __builtin_fmaf(s[j >> 2][j & 3], c, b - reference);
      };
      const float mn = fmaxf(m_run, mx);  // finite: row 0 of a tile in range is in range
      const float corr = __builtin_amdgcn_exp2f(m_run - mn);  // exp2(-inf) = 0 on the first tile
      float ps = 0.f;
#pragma unroll
      for (int j = 0; j < KEYS; ++j) {
        p[j] = __builtin_amdgcn_exp2f(shifted(j, mn));
        ps += p[j];
      }
      l_run = __builtin_fmaf(l_run, corr, ps);
      m_run = mn;
      if (__any(corr != 1.f)) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[b][r] *= corr;
      }
      if constexpr (A::kBf16) {
        bf16x8 ph, pl;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const __bf16 hi = (__bf16)p[j];
          ph[j] = hi;
          pl[j] = (__bf16)(p[j] - (float)hi);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int w = (b % EPV) >> 1;
          u32x4 v;
#pragma unroll
          for (int k2 = 0; k2 < 4; ++k2)  // the halves of two keys' words that hold the block's channel
            v[k2] = __builtin_amdgcn_perm(va[2 * k2 + 1][b / EPV][w], va[2 * k2][b / EPV][w],
                                          (b & 1) ? 0x07060302u : 0x05040100u);
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), ph, acc[b], 0, 0, 0);
          acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), pl, acc[b], 0, 0, 0);
        }
      } else {
        // (a tile's products are summed on their own: the long sum over a unit's rows has as many addends as it has tiles)
#pragma unroll
        for (int b0 = 0; b0 < NB; b0 += 4) {
          f32x4 a[4];
#pragma unroll
          for (int j = 0; j < KEYS; ++j)
#pragma unroll
            for (int b = 0; b < 4; ++b)
              a[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(va[j][(b0 + b) / EPV][(b0 + b) % EPV]), p[j],
                                                          j ? a[b] : f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
          for (int b = 0; b < 4; ++b) acc[b0 + b] += a[b];
        }
      }
      load_values(t + step, L);
    }
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    if (l16 < heads) {
      if (g == 0) {
        st_m[wv * kAttHeads + l16] = m_run;
        st_l[wv * kAttHeads + l16] = l_run;
      }
#pragma unroll
      for (int b = 0; b < NB; ++b)
        *reinterpret_cast<f32x4*>(&st_acc[(wv * heads + l16) * kAccPitch + b * 16 + g * 4]) = acc[b];
    }
    __syncthreads();
    const int pass_heads = min(heads, G - g0);
    int o0 = tid;
    asm volatile("" : "+v"(o0));  // (or the addresses below are formed before the tile loop and held through it)
    for (int o = o0; o < pass_heads * D; o += WAVES * 64) {
      const int h = o / D, ch = o % D;
      // where channel `ch` waits: block b, row m with AttGeom::channel(b, m) == ch
      const int at = ((ch / (16 * EPV)) * EPV + ch % EPV) * 16 + (ch % (16 * EPV)) / EPV;
      float top = kNegInf;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) top = fmaxf(top, st_m[w * kAttHeads + h]);
      float num = 0.f, den = 0.f;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {  // wave order: the same bits every run
        const float mw = st_m[w * kAttHeads + h];
        const float f = mw == kNegInf ? 0.f : __builtin_amdgcn_exp2f(mw - top);
        den = __builtin_fmaf(st_l[w * kAttHeads + h], f, den);
        num = __builtin_fmaf(st_acc[(w * heads + h) * kAccPitch + at], f, num);
      }
      if (splits == 1) {
        Elem<T>::store(out + ((size_t)u * G + g0 + h) * D + ch, den > 0.f ? num / den : 0.f);
      } else {  // [unit][split][head]: D sums, then the reference and the denominator
        float* pp = part + (((size_t)u * splits + sp) * G + g0 + h) * (D + 2);
        pp[ch] = num;
        if (ch == 0) {
          pp[D] = top;
          pp[D + 1] = den;
        }
      }
    }
    __syncthreads();
  }
}

// Adds the splits of attend_kernel in split order.  A thread per (head, channel) of a unit.
template <typename T, int D>
__global__ __launch_bounds__(256) void attend_combine_kernel(int rows, int splits, int G, const float* __restrict__ part,
                                                             T* __restrict__ out) {
  const int o = blockIdx.x * 256 + threadIdx.x;
  if (o >= rows * D) return;
  const int row = o / D, ch = o % D, u = row / G, h = row % G;
  const float* pp = part + ((size_t)u * splits * G + h) * (D + 2);
  const size_t pitch = (size_t)G * (D + 2);
  float m = kNegInf, num = 0.f, den = 0.f;
  for (int s0 = 0; s0 < splits; s0 += 8) {  // eight partials in flight
    float pm[8], pd[8], pn[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float* ps = pp + min(s0 + e, splits - 1) * pitch;
      pn[e] = ps[ch];
      pm[e] = ps[D];
      pd[e] = ps[D + 1];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (s0 + e >= splits || pm[e] == kNegInf) continue;
      const float mn = fmaxf(m, pm[e]);
      const float fa = __builtin_amdgcn_exp2f(m - mn), fb = __builtin_amdgcn_exp2f(pm[e] - mn);
      den = __builtin_fmaf(den, fa, pd[e] * fb);
      num = __builtin_fmaf(num, fa, pn[e] * fb);
      m = mn;
    }
  }
  Elem<T>::store(out + o, den > 0.f ? num / den : 0.f);
}

template <typename T, int D, int WAVES, bool NT>
hipError_t launch_attend_as(const KParams& kp, int n_units, const void* Q, const void* Kc, const void* Vc, int stride,
                            const int32_t* len, const int32_t* count, int count_pitch, void* out, int splits,
                            float* part, hipStream_t st) {
  const int heads = kp.G < kAttHeads ? kp.G : kAttHeads;
  const int lds = WAVES * (32 + 2 * kAttHeads + heads * (D + 4)) * (int)sizeof(float);
  static LdsLimitOnce lim;  // one per instantiation
  const hipError_t e = lim.ensure(reinterpret_cast<const void*>(&attend_kernel<T, D, WAVES, NT>), 160 * 1024);
  if (e != hipSuccess) return e;
  attend_kernel<T, D, WAVES, NT><<<dim3(n_units * splits), dim3(WAVES * 64), lds, st>>>(
      kp, static_cast<const T*>(Q), static_cast<const T*>(Kc), static_cast<const T*>(Vc), stride, len, count, count_pitch,
      static_cast<T*>(out), splits, part);
  if (splits > 1)
    attend_combine_kernel<T, D><<<dim3((n_units * kp.G * D + 255) / 256), dim3(256), 0, st>>>(
        n_units * kp.G, splits, kp.G, part, static_cast<T*>(out));
  return hipSuccess;
}

// Waves per workgroup.  As long as every workgroup has a compute unit to itself: eight (more rows of a
// unit in flight); with more workgroups than compute units four, so that several share one and
// one's merge overlaps the others' loads (eight / four: 300 units x 500 rows bf16, d = 128 21.4 / 19.2 us, d = 64 x 2000
// 40.8 / 35.7; 294 units of 3800 - 4750 rows 74.3 / 73.0).  Long fp32 units are the exception where it was
// measured: 64 channels from 512 workgroups on (600 x 3000 four 174, eight 166; 600 x 1000 62 / 58; 4000 x
// 1000 320 / 309; but 2000 x 250 46 / 48 and 400 x 2000 77 / 82), 128 channels up to 511 (400 x 4000 298 / 284).
// Non-temporal loads where the caches of the call exceed the 256 MB last-level cache, so that no
// call can find them there (554 MB: 102 -> 91 us; 1 GB of fp32: 185 -> 169 us); below that a
// call that repeats finds its rows there and the hint costs up to a quarter.
template <typename T, int D>
hipError_t launch_attend_t(const KParams& kp, int n_units, const void* Q, const void* Kc, const void* Vc, int stride,
                           const int32_t* len, const int32_t* count, int count_pitch, void* out, int splits,
                           float* part, hipStream_t st) {
  const bool nt = (int64_t)n_units * stride * (2 * D * (int)sizeof(T)) > (256ll << 20);
  const int64_t groups = (int64_t)n_units * splits;
  const int rounds = (stride - 1) / (8 * AttGeom<T, D>::kTileRows) + 1;  // of eight waves
  const bool eight_f32 = sizeof(T) == 4 && (D == 64 ? groups >= 512 && rounds > 6 : groups < 512 && rounds > 24);
  const bool four = groups > 256 && !eight_f32;
  auto go = [&](auto f) { return f(kp, n_units, Q, Kc, Vc, stride, len, count, count_pitch, out, splits, part, st); };
  if (four) return nt ? go(&launch_attend_as<T, D, 4, true>) : go(&launch_attend_as<T, D, 4, false>);
  return nt ? go(&launch_attend_as<T, D, 8, true>) : go(&launch_attend_as<T, D, 8, false>);
}

}  // namespace

// Workgroups that share a unit.  Without a workspace one; with it enough to fill the chip's compute
// units, of which a workgroup of eight waves takes one (the row loads in flight need the registers),
// as long as each still has two rounds of tiles and the unit at least six (the combining launch behind
// them costs about 4 us, a round of eight waves about 2.5 us).  A few workgroups more than compute
// units make a second turn of the chip that is nearly empty, so it is as many as fit at once; twice
// as many (the form with four waves) only where that fills the chip exactly and they stay long enough,
// or where one turn would leave a fifth of the chip idle and the units are long.
// Measured, one workgroup per unit -> split (bf16, d = 128): 8 units x 16 000 rows 159 -> 21 us,
// 16 x 4000 45 -> 14, 4 x 1500 21 -> 12, 100 x 2000 34 -> 25, 128 x 2000 36 -> 30; with 384 and
// 400 workgroups the last two took 37 and 29.  Two workgroups a unit and six rounds: 128 x 1281 19.6 ->
// 20.6, so a bf16 unit has to have seven then (seven: 29.7 -> 24.5; fp32, whose rounds are longer, six: 27.2 ->
// 22.9).  256 x 2000 (two each) 43 -> 47, so not beyond 128 units, but for one case: fp32 with 128 channels,
// two workgroups of four waves to a compute unit, where a few units more than compute units leave most
// of the chip half empty (300 x 1500 109 -> 87 us, 260 x 3000 200 -> 152, 350 x 1500 115 -> 105; 300 x 600 47.8 ->
// 46.5; 400 x 600 52 -> 60).
int attend_splits(const KParams& kp, int n_units, int stride) {
  if (n_units <= 0 || n_units > 380) return 1;
  const int tile = kp.dtype == CASK_BF16 ? 32 : 16;
  const int rounds = (stride + tile * 8 - 1) / (tile * 8);  // of eight waves, all rows used
  if (rounds < 6 || (int64_t)n_units * kp.G * kp.d > (1 << 30)) return 1;  // (the combining launch counts elements in 32 bits)
  if (n_units > 128) return n_units > 256 && rounds >= 9 && kp.dtype == CASK_F32 && kp.d == 128 ? 3 : 1;
  int s = 256 / n_units;
  const int twice = 512 / n_units;
  // (96 units: 6000 rows, two and five workgroups each 59.6 / 58.7 us; 16 000 rows 141 / 132)
  if ((twice * n_units == 512 && rounds >= 2 * twice) || (10 * twice > 23 * s && rounds >= 4 * twice)) s = twice;
  if (s > rounds / 2) s = rounds / 2;
  if (s == 2 && rounds < 7 && kp.dtype == CASK_BF16) return 1;
  return s > 64 ? 64 : s;
}

size_t attend_part_bytes(const KParams& kp, int n_units, int splits) {
  return splits <= 1 ? 0 : (size_t)n_units * splits * kp.G * (kp.d + 2) * sizeof(float);
}

hipError_t launch_attend(const KParams& kp, int n_units, const void* Q, const void* Kc, const void* Vc,
                         int stride, const int32_t* len, const int32_t* count, int count_pitch,
                         void* out, int splits, float* part, hipStream_t st) {
  if (n_units == 0) return hipSuccess;
  hipError_t e;
#define CASK_ATT(T, D) e = launch_attend_t<T, D>(kp, n_units, Q, Kc, Vc, stride, len, count, count_pitch, out, splits, part, st)
  if (kp.dtype == CASK_F32) {
    if (kp.d == 64) CASK_ATT(float, 64); else CASK_ATT(float, 128);
  } else {
    if (kp.d == 64) CASK_ATT(uint16_t, 64); else CASK_ATT(uint16_t, 128);
  }
#undef CASK_ATT
  return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace cask
