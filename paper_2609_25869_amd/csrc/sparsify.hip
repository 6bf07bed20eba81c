// Mean-pooled top-k block sparsifier on gfx950 (the step that supplies the
// logical mask M and its geometry B, Section 2.1), so that sparsify -> plan ->
// forward runs on the device.
//
// For every (b, h) and query block qb the score of KV block kb is the dot
// product of the mean query row of qb and the mean key row of kb; the k
// largest scores of each row are active (ties to the lower kb), and
// optionally every block the token diagonal passes through.  The selection
// is an integer decided by floating point, so the arithmetic is pinned:
// block sums of bf16 values in IEEE double in token order, the mean as one
// double division, and each score accumulated over the head dimension in
// increasing order with one rounding per multiply and per add (contraction
// into fused multiply-adds is switched off).  Any implementation that follows
// the same steps selects the same blocks.
//
// The pinned scores decide, but few of them have to be formed: the matrix
// units give every score within a proven distance of the pinned one, the
// selection finds the k-th largest of those, and only columns closer to it
// than that distance allows to tell apart are scored again in the pinned
// arithmetic.
//
// Kernels, at 115200 tokens, 24 heads, (64, 64) blocks, k = 216 of 1800 in
// parentheses, in a trace of whole requests (fp64 scores of every pair on the
// vector units and a radix select of 64-bit keys per workgroup took 335 + 1109 +
// 481 us on another run; the calls alone, repeated, 1.91 and 0.82 ms):
//   block_mean_kernel    (354 us, 4.0 TB/s) HBM-bound: the tensors once, 16
//                        bytes per lane and row where the layout allows
//   block_score_kernel   (313 us, 64 TFLOP/s) fp32 matrix instructions on the
//                        means rounded to fp32, 128 x 64 or 64 x 64 score
//                        tiles; the means are converted on the way into LDS.
//                        128 x 128 tiles need 256 registers: 474 us with two
//                        waves a SIMD forced, 355 with one
//   topk_select_kernel   (235 us) one wave per score row with the row's keys
//                        in registers, counted against a threshold that
//                        interpolation and bisection move (VALU-bound; no
//                        LDS, no barrier).  Rows that fp32 leaves undecided
//                        (most of a row's columns tied, non-finite or extreme
//                        values, one block thousands of times the others)
//                        cost more: 3.5 ms in all with every row such a row
#include "bsa_internal.h"

namespace bsa {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline double bf16_to_f64(uint32_t b) { return (double)__uint_as_float(b << 16); }

// Block means of Q and K in one launch.  A thread sums COLS columns of one
// block over its tokens in order, eight rows' loads in flight: COLS = 8 reads
// 16 bytes a row (16 lanes a block), COLS = 2 reads 4 bytes (one wave a
// block), COLS = 1 takes any stride and alignment.
template <int COLS>
__device__ inline void load_cols(const uint16_t* p, uint32_t (&v)[COLS]) {
  if constexpr (COLS == 8) {
    const u32x4 x = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (x[j / 2] >> (16 * (j % 2))) & 0xFFFFu;
  } else if constexpr (COLS == 2) {
    const uint32_t x = *reinterpret_cast<const uint32_t*>(p);
    v[0] = x & 0xFFFFu;
    v[1] = x >> 16;
  } else {
    v[0] = *p;
  }
}

template <int COLS>
__global__ __launch_bounds__(256) void block_mean_kernel(MeanArgs a) {
  constexpr int kLanes = kHeadDim / COLS;  // threads per block
  const int64_t w = (int64_t)blockIdx.x * (256 / kLanes) + threadIdx.x / kLanes;
  const int64_t nq = (int64_t)a.nbh * a.nb[0];
  if (w >= nq + (int64_t)a.nbh * a.nb[1]) return;
  const int t = w < nq ? 0 : 1;  // Q blocks first, then K blocks
  const int64_t wi = t ? w - nq : w;
  const int32_t nb = a.nb[t], blk = a.blk[t], n = a.n[t];
  // tensors that keep a token's heads together are walked head by head inside
  // a block of tokens, so that a workgroup's 256-byte rows are neighbours
  const bool by_head = a.s1[t] < a.s2[t];
  const int32_t i = (int32_t)(by_head ? wi / a.nbh : wi % nb), bhl = (int32_t)(by_head ? wi % a.nbh : wi / nb);
  const int32_t bh = a.bh0 + bhl;
  const int32_t b = bh / a.H, h = bh - b * a.H;
  const int c = (threadIdx.x % kLanes) * COLS;
  const int64_t s2 = a.s2[t];
  const int32_t r0 = i * blk, r1 = min(n, r0 + blk);
  const uint16_t* p = a.x[t] + b * a.s0[t] + h * a.s1[t] + c + r0 * s2;
  double s[COLS];
#pragma unroll
  for (int j = 0; j < COLS; ++j) s[j] = 0.0;
  int32_t r = r0;
  for (; r + 8 <= r1; r += 8, p += 8 * s2) {
    uint32_t v[8][COLS];
#pragma unroll
    for (int k = 0; k < 8; ++k) load_cols<COLS>(p + k * s2, v[k]);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
#pragma unroll
      for (int j = 0; j < COLS; ++j) s[j] += bf16_to_f64(v[k][j]);
    }
  }
  for (; r < r1; ++r, p += s2) {
    uint32_t v[COLS];
    load_cols<COLS>(p, v);
#pragma unroll
    for (int j = 0; j < COLS; ++j) s[j] += bf16_to_f64(v[j]);
  }
  double* out = a.out[t] + ((int64_t)bhl * nb + i) * kHeadDim + c;
#pragma unroll
  for (int j = 0; j < COLS; ++j) out[j] = s[j] / (double)(r1 - r0);
}

// ---------------------------------------------------------------------------
// Scores in fp32 on the matrix units.
//
// Their distance from the pinned score of a pair is at most kScoreEps * |q|
// |k| (2-norms of the means): both operands are rounded to fp32 (2^-24 each),
// 32 products are accumulated at a time (at most 2^-23 of the sum of
// magnitudes per accumulation, whichever way the unit rounds), and the four
// partial sums are added (2^-24 each): 70 * 2^-24 in all, and the pinned
// score itself is within 2^-45.  The sum of magnitudes is at most |q| |k|.
// Underflow adds nothing that matters while both norms lie in
// [kNormMin, kNormMax]; other rows take the pinned scores throughout.
constexpr float kScoreEps = 0x1p-17f;
constexpr float kNormMin = 0x1p-40f, kNormMax = 0x1p40f;

constexpr int kSC = 32;  // head-dim chunk staged per step
constexpr int kSP = kSC + 4;  // padded LDS row: 16 rows' 16-byte reads on distinct banks

// RQ x RK matrix tiles of 32 x 32 scores per wave, 2 x 2 waves per workgroup.
template <int RQ, int RK>
__global__ __launch_bounds__(256) void block_score_kernel(const double* pq, const double* pk, int32_t nqb,
                                                          int32_t nkb, float* scores, float* knorm, int32_t nx,
                                                          int32_t ny, int64_t ntiles) {
  constexpr int kTQ = 64 * RQ, kTK = 64 * RK;
  constexpr int kLQ = kTQ * kSC / 2 / 256, kLK = kTK * kSC / 2 / 256;  // pairs per thread and chunk
  __shared__ __attribute__((aligned(16))) float sq[kTQ * kSP];
  __shared__ __attribute__((aligned(16))) float sk[kTK * kSP];
  __shared__ float wave_max[4];
  // Workgroup i runs on XCD i % 8: each XCD takes a contiguous eighth of the
  // tiles (k tile fastest, head slowest), so that a head's means are read into
  // one L2 or two instead of all eight.
  const int64_t per = (ntiles + 7) / 8, ti = (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if ((blockIdx.x >> 3) >= per || ti >= ntiles) return;
  const int32_t tx = (int32_t)(ti % nx), ty = (int32_t)(ti / nx % ny);
  const int64_t bhl = ti / nx / ny;
  const int32_t q0 = ty * kTQ, k0 = tx * kTK;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int n = lane & 31, hh = lane >> 5;
  const int wr = (w >> 1) * 32 * RQ, wc = (w & 1) * 32 * RK;
  const double* gq = pq + bhl * nqb * kHeadDim;
  const double* gk = pk + bhl * nkb * kHeadDim;
  f64x2 lq[kLQ], lk[kLK];
  auto fetch = [&](int c0) {
    const int rr = tid / (kSC / 2), cc = c0 + 2 * (tid % (kSC / 2));
#pragma unroll
    for (int i = 0; i < kLQ; ++i) {
      const int32_t r = q0 + rr + 16 * i;
      lq[i] = r < nqb ? *reinterpret_cast<const f64x2*>(gq + (int64_t)r * kHeadDim + cc) : f64x2{0.0, 0.0};
    }
#pragma unroll
    for (int i = 0; i < kLK; ++i) {
      const int32_t r = k0 + rr + 16 * i;
      lk[i] = r < nkb ? *reinterpret_cast<const f64x2*>(gk + (int64_t)r * kHeadDim + cc) : f64x2{0.0, 0.0};
    }
  };
  const bool norms = ty == 0;  // the first row of tiles also reports the key norms
  float sumsq[kLK];
#pragma unroll
  for (int i = 0; i < kLK; ++i) sumsq[i] = 0.f;
  f32x16 tot[RQ][RK];
#pragma unroll
  for (int i = 0; i < RQ; ++i) {
#pragma unroll
    for (int j = 0; j < RK; ++j) tot[i][j] = f32x16{};
  }
  fetch(0);
  for (int c0 = 0; c0 < kHeadDim; c0 += kSC) {
    float* dst = sq + (tid / (kSC / 2)) * kSP + 2 * (tid % (kSC / 2));
#pragma unroll
    for (int i = 0; i < kLQ; ++i)
      *reinterpret_cast<f32x2*>(dst + 16 * i * kSP) = f32x2{(float)lq[i][0], (float)lq[i][1]};
    dst += sk - sq;
#pragma unroll
    for (int i = 0; i < kLK; ++i) {
      const f32x2 f = {(float)lk[i][0], (float)lk[i][1]};
      *reinterpret_cast<f32x2*>(dst + 16 * i * kSP) = f;
      if (norms) sumsq[i] += f[0] * f[0] + f[1] * f[1];
    }
    __syncthreads();
    if (c0 + kSC < kHeadDim) fetch(c0 + kSC);
    f32x16 acc[RQ][RK];
#pragma unroll
    for (int i = 0; i < RQ; ++i) {
#pragma unroll
      for (int j = 0; j < RK; ++j) acc[i][j] = f32x16{};
    }
    // eight head-dim columns per step: the lane halves take four each, one
    // per matrix instruction (the order inside a chunk is free)
#pragma unroll
    for (int g = 0; g < kSC / 8; ++g) {
      f32x4 av[RQ], bv[RK];
#pragma unroll
      for (int i = 0; i < RQ; ++i) av[i] = *reinterpret_cast<const f32x4*>(sq + (wr + 32 * i + n) * kSP + 8 * g + 4 * hh);
#pragma unroll
      for (int i = 0; i < RK; ++i) bv[i] = *reinterpret_cast<const f32x4*>(sk + (wc + 32 * i + n) * kSP + 8 * g + 4 * hh);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int i = 0; i < RQ; ++i) {
#pragma unroll
          for (int j = 0; j < RK; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i][e], bv[j][e], acc[i][j], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int i = 0; i < RQ; ++i) {
#pragma unroll
      for (int j = 0; j < RK; ++j) tot[i][j] += acc[i][j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < RQ; ++i) {
#pragma unroll
    for (int j = 0; j < RK; ++j) {
      const int32_t kb = k0 + wc + 32 * j + n;
      if (kb >= nkb) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int32_t qb = q0 + wr + 32 * i + 8 * (e / 4) + 4 * hh + e % 4;
        if (qb < nqb) scores[(bhl * nqb + qb) * nkb + kb] = tot[i][j][e];
      }
    }
  }
  if (norms) {
    // the largest 2-norm of the tile's mean keys
    float mx = 0.f;
#pragma unroll
    for (int i = 0; i < kLK; ++i) {
      float v = sumsq[i];
#pragma unroll
      for (int o = 1; o < kSC / 2; o <<= 1) v += __shfl_xor(v, o, 64);
      mx = fmaxf(mx, v);
    }
    for (int o = kSC / 2; o < 64; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
    if (lane == 0) wave_max[w] = mx;
    __syncthreads();
    if (tid == 0) {
      mx = fmaxf(fmaxf(wave_max[0], wave_max[1]), fmaxf(wave_max[2], wave_max[3]));
      knorm[bhl * nx + tx] = sqrtf(mx) * 1.0001f;
    }
  }
}

// Order-preserving map of a double to an unsigned key (larger score, larger
// key); -0 and +0 map to the same key, as they compare equal.
__device__ inline uint64_t order_key(double x) {
  if (x == 0.0) x = 0.0;
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ inline uint32_t wave_inclusive_scan(uint32_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  return x;
}

// The same for a float (adding 0 turns -0 into +0 and changes nothing else).
__device__ inline uint32_t order_key32(float x) {
  const uint32_t u = __float_as_uint(x + 0.f);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ inline float key32_value(uint32_t k) { return __uint_as_float((k >> 31) ? (k & 0x7FFFFFFFu) : ~k); }

// A mean query row that is the same for the whole wave, read through the
// scalar cache.
typedef const __attribute__((address_space(4))) double* UniformRow;
__device__ inline UniformRow uniform_row(const double* p) {
  const uint64_t u = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)u), hi = __builtin_amdgcn_readfirstlane((int)(u >> 32));
  return (UniformRow)((uint64_t)hi << 32 | lo);
}

// The pinned score of (mean query row q, mean key row k), by one thread.
__device__ inline double pinned_score(UniformRow q, const double* k) {
#pragma clang fp contract(off)
  double acc = 0.0;
#pragma unroll 1
  for (int c = 0; c < kHeadDim; c += 8) {
    f64x2 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const f64x2*>(k + c + 2 * j);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const double prod = q[c + j] * v[j / 2][j % 2];
      acc = acc + prod;
    }
  }
  return acc;
}

constexpr int kSelWaves = 4;
constexpr int kMaxCand = 64;

// x, but addresses formed from it are formed where they are used: kept across
// the loops around, they would cost the whole kernel registers.
__device__ inline int not_hoisted(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Rows in the pinned arithmetic throughout, by the whole workgroup, two rows
// of one head at a time.
//
// Scores: a wave takes 64 columns at a time, eight head-dim columns per step.
// Its lanes read the mean keys as whole 64-byte pieces, pass them on through
// LDS (kPinStage bytes per wave, 16-byte chunks of row r permuted by
// (r / 2) % 4, so that neither side conflicts), and lane l accumulates its
// column's two scores in order.  Bound by the latency of those steps.  (A
// thread that walked a mean key row by itself, one row of scores at a time,
// read 64 lines per instruction: with every row undecided, 115200 tokens x 24
// heads in (64, 64) blocks took 14.9 ms with it and 3.5 so, 0.87 with none.)
constexpr int kPinDims = 8;

constexpr int kPinStage = 64 * kPinDims * 8;

__device__ inline void pinned_keys(UniformRow q0, UniformRow q1, const double* pk, int32_t nkb, uint64_t* key0,
                                   uint64_t* key1, uint8_t* smem) {
#pragma clang fp contract(off)
  const int wv = threadIdx.x >> 6;
  uint8_t* stage = smem + wv * kPinStage;
#pragma unroll 1
  for (int32_t c0 = 64 * wv; c0 < nkb; c0 += 64 * kSelWaves) {
    const int lane = not_hoisted(threadIdx.x & 63);
    f64x2 v[4];
    auto fetch = [&](int d) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t c = min(c0 + 16 * j + (lane >> 2), nkb - 1);
        v[j] = *reinterpret_cast<const f64x2*>(pk + (c * kHeadDim + d + 2 * (lane & 3)));
      }
    };
    double acc0 = 0.0, acc1 = 0.0;
    fetch(0);
#pragma unroll 1
    for (int d = 0; d < kHeadDim; d += kPinDims) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = 16 * j + (lane >> 2);
        *reinterpret_cast<f64x2*>(stage + r * 64 + (((lane & 3) ^ ((r >> 1) & 3)) << 4)) = v[j];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if (d + kPinDims < kHeadDim) fetch(d + kPinDims);
#pragma unroll
      for (int p = 0; p < kPinDims / 2; ++p) {
        const f64x2 k2 = *reinterpret_cast<const f64x2*>(stage + lane * 64 + ((p ^ ((lane >> 1) & 3)) << 4));
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const double prod0 = q0[d + 2 * p + e] * k2[e], prod1 = q1[d + 2 * p + e] * k2[e];
          acc0 = acc0 + prod0;
          acc1 = acc1 + prod1;
        }
        __builtin_amdgcn_sched_barrier(0);  // (so do products formed ahead)
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    if (c0 + lane < nkb) {
      key0[c0 + lane] = order_key(acc0);
      key1[c0 + lane] = order_key(acc1);
    }
  }
}

// Selection from a row's pinned keys: MSB-first radix select of the k-th
// largest (8 passes of 8 bits), ties ranked by column, the mask row written
// with the diagonal [d0, d1].
struct PinnedSelect {
  uint32_t hist[256];
  uint32_t wave_ties[kSelWaves];
  uint64_t prefix;
  int32_t remaining;
};

__device__ inline void select_pinned(const uint64_t* keys, int32_t nkb, int32_t k, int32_t d0, int32_t d1,
                                     uint8_t* out, PinnedSelect& sh) {
  const int tid = not_hoisted(threadIdx.x), lane = tid & 63, wv = tid >> 6;
  // k-th largest key: fix one byte per pass from the most significant
  uint64_t prefix = 0, pmask = 0;
  int32_t remaining = k;  // rank of the sought key among those matching prefix
#pragma unroll 1
  for (int shift = 56; shift >= 0; shift -= 8) {
    sh.hist[tid] = 0;
    __syncthreads();
#pragma unroll 1
    for (int32_t kb = tid; kb < nkb; kb += 64 * kSelWaves) {
      const uint64_t key = keys[kb];
      const bool in = (key & pmask) == prefix;
      const uint32_t digit = (uint32_t)(key >> shift) & 255u;
      // equal digits (all of them among tied scores) take one add per wave
      const uint64_t active = __ballot(in);
      if (active == 0) continue;
      const uint32_t common = (uint32_t)__builtin_amdgcn_readlane((int)digit, __builtin_ctzll(active));
      const uint64_t same = __ballot(in && digit == common);
      if (in && digit != common) atomicAdd(&sh.hist[digit], 1u);
      if (lane == __builtin_ctzll(active)) atomicAdd(&sh.hist[common], (uint32_t)__popcll(same));
    }
    __syncthreads();
    if (tid < 64) {
      // digit d of the sought key: the largest d whose keys, counted from
      // digit 255 down to d, reach `remaining` (d = 0 if none does before).
      // Lane l holds digits 255-4l .. 252-4l.
      uint32_t cnt[4], local = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        cnt[j] = sh.hist[255 - 4 * tid - j];
        local += cnt[j];
      }
      const uint32_t incl = wave_inclusive_scan(local);
      const uint64_t reach = __ballot(incl >= (uint32_t)remaining || tid == 63);
      const int first = __builtin_ctzll(reach);
      if (tid == first) {
        int32_t above = (int32_t)(incl - local);
        int d = 255 - 4 * tid;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (d == 0 || above + (int32_t)cnt[j] >= remaining) break;
          above += (int32_t)cnt[j];
          --d;
        }
        sh.remaining = remaining - above;
        sh.prefix = prefix | ((uint64_t)d << shift);
      }
    }
    __syncthreads();
    remaining = sh.remaining;
    prefix = sh.prefix;
    pmask |= 0xFFull << shift;
  }
  // prefix is the k-th largest key; `remaining` of the keys equal to it are
  // taken, the lowest columns first.  Wave w holds the w-th quarter of the row.
  const int32_t per = ((nkb + kSelWaves - 1) / kSelWaves + 63) & ~63;
  const int32_t c0 = min(nkb, wv * per), c1 = min(nkb, c0 + per);
  uint32_t ties = 0;
#pragma unroll 1
  for (int32_t b = c0; b < c1; b += 64) ties += __popcll(__ballot(b + lane < c1 && keys[b + lane] == prefix));
  if (lane == 0) sh.wave_ties[wv] = ties;
  __syncthreads();
  int32_t rank = 0;
  for (int w = 0; w < wv; ++w) rank += (int32_t)sh.wave_ties[w];
#pragma unroll 1
  for (int32_t b = c0; b < c1; b += 64) {
    const int32_t kb = b + lane;
    const uint64_t key = kb < c1 ? keys[kb] : 0ull;
    const uint64_t tie = __ballot(kb < c1 && key == prefix);
    const int32_t mine = rank + (int32_t)__popcll(tie & ((1ull << lane) - 1));
    if (kb < c1) out[kb] = (key > prefix || (key == prefix && mine < remaining) || (kb >= d0 && kb <= d1)) ? 1 : 0;
    rank += (int32_t)__popcll(tie);
  }
  __syncthreads();
}

// Selection of one score row by one wave.  Lane l holds the row's keys in
// registers, KPL of them: columns 256 g + 4 l + j in register 4 g + j (VEC:
// score and mask rows are whole 16- and 4-byte words) or 64 j + l in
// register j.
//
// The k-th largest fp32 score T and the k-th largest pinned score differ by
// at most the error bound, so columns above T by more than twice the bound
// are taken, those below T by more than that are not, and the candidates in
// between (usually T's own column alone) are settled by their pinned scores,
// ties to the lower column.  Up to 64 of them are scored by the wave's lanes
// and ranked; rows with more, with scores that are not finite, or with norms
// outside the bound's range are selected in the pinned arithmetic throughout
// once all rows of the workgroup are through: their fp32 scores are done with
// then, and the space of the workgroup's four score rows holds the keys of two.

template <int KPL, bool VEC>
__global__ __launch_bounds__(64 * kSelWaves) __attribute__((amdgpu_waves_per_eu(KPL <= 64 ? 3 : 1)))
void topk_select_kernel(SelectArgs a) {
  struct Candidates {
    int32_t column[kMaxCand];
    uint8_t take[kMaxCand];
  };
  static_assert(kPinStage * kSelWaves >= (int)sizeof(Candidates) * kSelWaves, "one array for both");
  __shared__ __attribute__((aligned(16))) uint8_t smem[kPinStage * kSelWaves];
  __shared__ PinnedSelect pinned;
  __shared__ int32_t unsettled[kSelWaves];
  constexpr int kG = VEC ? 4 : 1;  // registers of one column group
  constexpr bool kLong = KPL > 16;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * kSelWaves;
  const int32_t nkb = a.nkb;
  Candidates& cand = reinterpret_cast<Candidates*>(smem)[wv];
  auto column = [&](int j) { return VEC ? 256 * (j / 4) + 4 * lane + j % 4 : 64 * j + lane; };
  // the diagonal: columns [lo / bkv, (hi - 1) / bkv] for the row's tokens
  // [lo, hi) that also exist as keys
  auto diagonal = [&](int64_t r, int32_t* d0, int32_t* d1) {
    const int32_t qb = (int32_t)(r % a.nqb);
    const int32_t lo = qb * a.bq, hi = min(min(a.nq, a.nkv), lo + a.bq);
    const bool any = a.diagonal && lo < hi;
    *d0 = any ? lo / a.bkv : 1;
    *d1 = any ? (hi - 1) / a.bkv : 0;
  };
  auto mask_row = [&](int64_t r) { return a.mask + ((int64_t)a.bh0 * a.nqb + r) * nkb; };

  // one row; false if it has to go through the pinned arithmetic
  auto select = [&](int64_t row) -> bool {
    int32_t d0, d1;
    diagonal(row, &d0, &d1);
    uint8_t* out = mask_row(row);
    if (a.k <= 0 || a.k >= nkb) {
#pragma unroll 1
      for (int32_t c = lane; c < nkb; c += 64) out[c] = (a.k > 0 || (c >= d0 && c <= d1)) ? 1 : 0;
      return true;
    }
    const int64_t bhl = row / a.nqb;
    const double* q = a.pq + row * kHeadDim;
    const double* pk = a.pk + bhl * nkb * kHeadDim;
    const float* srow = a.scores + row * nkb;
    uint32_t key[KPL];  // 0 past the row's end, below every finite score's key
    uint32_t largest = 0;  // magnitude bits
#pragma unroll
    for (int g = 0; g < KPL; g += kG) {
      float x[kG];
      const bool in = column(g) < nkb;
      if constexpr (VEC) {
        const f32x4 v = in ? *reinterpret_cast<const f32x4*>(srow + column(g)) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < kG; ++j) x[j] = v[j];
      } else {
        x[0] = in ? srow[column(g)] : 0.f;
      }
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        largest = max(largest, __float_as_uint(x[j]) & 0x7FFFFFFFu);
        key[g + j] = in ? order_key32(x[j]) : 0u;
      }
    }
    const bool finite = largest < 0x7F800000u;
    // norms: |q| of the row, the largest |k| of the head
    const double q0 = q[lane], q1 = q[64 + lane];
    float qn = (float)(q0 * q0 + q1 * q1), kn = 0.f;
    for (int32_t i = lane; i < a.nparts; i += 64) kn = fmaxf(kn, a.knorm[bhl * a.nparts + i]);
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int j = 0; j < KPL; ++j) {
      hi = max(hi, key[j]);
      lo = min(lo, key[j] == 0u ? 0xFFFFFFFFu : key[j]);
    }
    for (int o = 32; o > 0; o >>= 1) {
      hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
      lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
      qn += __shfl_xor(qn, o, 64);
      kn = fmaxf(kn, __shfl_xor(kn, o, 64));
    }
    qn = sqrtf(qn) * 1.0001f;
    const bool zero = __ballot(q0 != 0.0 || q1 != 0.0) == 0;  // then every finite score is exactly 0
    const bool in_range = qn >= kNormMin && qn <= kNormMax && kn >= kNormMin && kn <= kNormMax;
    if (__ballot(!finite) != 0 || !(in_range || zero)) return false;

    auto count_ge = [&](uint32_t t) -> int32_t {
      int32_t c = 0;
      if constexpr (kLong) {
        int32_t own = 0;  // this lane's, then the wave's by its bits
#pragma unroll
        for (int j = 0; j < KPL; ++j) own += key[j] >= t ? 1 : 0;
#pragma unroll
        for (int bit = 0; (1 << bit) <= KPL; ++bit) c += __popcll(__ballot((own >> bit) & 1)) << bit;
      } else {
#pragma unroll
        for (int j = 0; j < KPL; ++j) c += __popcll(__ballot(key[j] >= t));
      }
      return c;
    };
    // T: the largest key with at least k keys >= it.  [lo, end) holds it, c_lo
    // >= k keys are >= lo and c_end < k are >= end.  Rows of more than 1024
    // columns take two steps of three by interpolating between the counts
    // over the scores (a handful of steps for scores without outliers, where
    // bisection takes 18); the third halves the keys, so that at most 96
    // steps are ever taken.  A count of a short row costs less than that:
    // 532 columns x 1878 rows 23.0 us with it, 19.7 without.
    lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
    uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi) + 1u;
    int32_t c_lo = nkb, c_end = 0;
    for (int step = 1; end - lo > 1u; ++step) {
      uint32_t mid = lo + ((end - lo) >> 1);
      if (kLong && step % 3 != 0) {
        const float v0 = key32_value(lo), v1 = key32_value(end - 1u);
        const float f = ((float)(c_lo - a.k) + 0.5f) / (float)(c_lo - c_end);
        mid = order_key32(v0 + f * (v1 - v0));
        mid = min(max(mid, lo + 1u), end - 1u);
        mid = (uint32_t)__builtin_amdgcn_readfirstlane((int)mid);
      }
      const int32_t c = count_ge(mid);
      if (c > a.k) {
        lo = mid;
        c_lo = c;
      } else if (c < a.k) {
        end = mid;
        c_end = c;
      } else {  // exactly k: T is the smallest of them
        uint32_t t = 0xFFFFFFFFu;
#pragma unroll
        for (int j = 0; j < KPL; ++j) t = min(t, key[j] >= mid ? key[j] : 0xFFFFFFFFu);
        for (int o = 32; o > 0; o >>= 1) t = min(t, (uint32_t)__shfl_xor((int)t, o, 64));
        lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
        end = lo + 1u;
      }
    }
    const float T = key32_value(lo);
    // twice the bound, and more than the rounding of the two sums below
    const float reach = zero ? 0.f : (2.f * kScoreEps + 0x1p-21f) * qn * kn;
    const uint32_t from = order_key32(T - reach), to = order_key32(T + reach);
    const int32_t sure = count_ge(to + 1u);
    const int32_t need = a.k - sure, m = count_ge(from) - sure;  // of m candidates, `need` are taken

    auto store = [&](int g, uint32_t word) {  // group g's mask bytes, with the diagonal
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        const int32_t c = column(g + j);
        word |= (c >= d0 && c <= d1 ? 1u : 0u) << (8 * j);
      }
      if (column(g) >= nkb) return;
      if constexpr (VEC) *reinterpret_cast<uint32_t*>(out + column(g)) = word;
      else out[column(g)] = (uint8_t)word;
    };
    if (need >= m) {  // every candidate
#pragma unroll
      for (int g = 0; g < KPL; g += kG) {
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < kG; ++j) word |= (key[g + j] >= from ? 1u : 0u) << (8 * j);
        store(g, word);
      }
      return true;
    }
    if (!zero && m > kMaxCand) return false;

    // candidate bits of one group's registers and the number of candidates
    // before this lane's first in column order; `base` counts on
    auto group = [&](int g, int32_t& base, uint64_t (&bits)[kG]) -> int32_t {
      int32_t pos = base;
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        bits[j] = __ballot(key[g + j] >= from && key[g + j] <= to);
        pos += __builtin_amdgcn_mbcnt_hi((uint32_t)(bits[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bits[j], 0u));
        base += __popcll(bits[j]);
      }
      return pos;
    };
    if (!zero) {  // (equal scores go by column alone)
      int32_t base = 0;
#pragma unroll
      for (int g = 0; g < KPL; g += kG) {
        uint64_t bits[kG];
        int32_t pos = group(g, base, bits);
#pragma unroll
        for (int j = 0; j < kG; ++j)
          if ((bits[j] >> lane) & 1ull) cand.column[pos++] = column(g + j);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      uint64_t mine = 0;  // lane i: candidate i's pinned score
      if (lane < m) mine = order_key(pinned_score(uniform_row(q), pk + (int64_t)cand.column[lane] * kHeadDim));
      int32_t rank = 0;
#pragma unroll 1
      for (int32_t i = 0; i < m; ++i) {
        const uint64_t other = (uint64_t)__shfl((unsigned long long)mine, i, 64);
        rank += (other > mine || (other == mine && i < lane)) ? 1 : 0;
      }
      if (lane < m) cand.take[lane] = rank < need ? 1 : 0;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
    int32_t base = 0;
#pragma unroll
    for (int g = 0; g < KPL; g += kG) {
      uint64_t bits[kG];
      int32_t pos = group(g, base, bits);
      uint32_t word = 0;
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        bool take = key[g + j] > to;
        if ((bits[j] >> lane) & 1ull) {
          take = zero ? pos < need : cand.take[pos] != 0;
          ++pos;
        }
        word |= (take ? 1u : 0u) << (8 * j);
      }
      store(g, word);
    }
    return true;
  };

  const bool settled = row0 + wv >= a.rows || select(row0 + wv);
  if (lane == 0) unsettled[wv] = settled ? 0 : 1;
  __syncthreads();
  // (rare, and kept small: its registers would halve the waves in flight)
  uint64_t* keys = reinterpret_cast<uint64_t*>(a.scores + row0 * nkb);
#pragma unroll 1
  for (int w = 0; w < kSelWaves; ++w) {
    if (!unsettled[w]) continue;
    const int64_t row = row0 + w, bhl = (uint32_t)row / (uint32_t)a.nqb;
    // the next such row of the same head goes with it
    int w2 = w + 1;
    while (w2 < kSelWaves && !unsettled[w2]) ++w2;
    const bool pair = w2 < kSelWaves && (uint32_t)(row0 + w2) / (uint32_t)a.nqb == bhl;
    const double* q = a.pq + row * kHeadDim;
    pinned_keys(uniform_row(q), uniform_row(pair ? a.pq + (row0 + w2) * kHeadDim : q), a.pk + bhl * nkb * kHeadDim, nkb,
                keys, keys + nkb, smem);
    __syncthreads();
#pragma unroll 1
    for (int i = 0; i < (pair ? 2 : 1); ++i) {
      const int64_t r = i ? row0 + w2 : row;
      int32_t d0, d1;
      diagonal(r, &d0, &d1);
      select_pinned(keys + i * nkb, nkb, a.k, d0, d1, mask_row(r), pinned);
    }
    if (pair) w = w2;
  }
}

template <int KPL>
hipError_t launch_select(const SelectArgs& a, hipStream_t s) {
  const bool vec = a.nkb % 4 == 0 && (reinterpret_cast<uintptr_t>(a.scores) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(a.mask) & 3) == 0;
  const dim3 grid((unsigned)((a.rows + kSelWaves - 1) / kSelWaves)), block(64 * kSelWaves);
  if (vec) hipLaunchKernelGGL((topk_select_kernel<KPL, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((topk_select_kernel<KPL, false>), grid, block, 0, s, a);
  return hipGetLastError();
}

// Score tiles of 128 x 64 leave the chip idle below two workgroups per CU.
constexpr int64_t kBigTileMin = 512;

}  // namespace

// KV blocks per score row: a wave holds its row's keys in registers, 96 a lane
int32_t sparsify_max_kv_blocks() { return 6144; }

int64_t sparsify_score_rows(int64_t rows) { return (rows + kSelWaves - 1) / kSelWaves * kSelWaves; }

hipError_t launch_block_mean(const MeanArgs& a, hipStream_t s) {
  const int64_t blocks = (int64_t)a.nbh * (a.nb[0] + (int64_t)a.nb[1]);
  if (blocks == 0) return hipSuccess;
  uint64_t mis = 0;
  for (int t = 0; t < 2; ++t)
    mis |= reinterpret_cast<uintptr_t>(a.x[t]) | (uint64_t)(2 * a.s0[t]) | (uint64_t)(2 * a.s1[t]) | (uint64_t)(2 * a.s2[t]);
  // 16 bytes a row while that leaves at least two waves per SIMD (four blocks
  // a wave), else one block a wave with 4 bytes a row
  const int cols = (mis & 15) == 0 && blocks >= 8192 ? 8 : (mis & 3) == 0 ? 2 : 1;
  const int per = 256 * cols / kHeadDim;  // blocks per workgroup
  const dim3 grid((unsigned)((blocks + per - 1) / per)), block(256);
  if (cols == 8) hipLaunchKernelGGL(block_mean_kernel<8>, grid, block, 0, s, a);
  else if (cols == 2) hipLaunchKernelGGL(block_mean_kernel<2>, grid, block, 0, s, a);
  else hipLaunchKernelGGL(block_mean_kernel<1>, grid, block, 0, s, a);
  return hipGetLastError();
}

int32_t sparsify_norm_parts(int32_t nkb) { return (nkb + 63) / 64; }

hipError_t launch_block_scores(const double* pq, const double* pk, int32_t nqb, int32_t nkb, int32_t nbh,
                               float* scores, float* knorm, int32_t* nparts, hipStream_t s) {
  const int32_t nx = (nkb + 63) / 64, ny_big = (nqb + 127) / 128;
  const bool big = (int64_t)nx * ny_big * nbh >= kBigTileMin;
  const int32_t ny = big ? ny_big : (nqb + 63) / 64;
  const int64_t ntiles = (int64_t)nx * ny * nbh;
  *nparts = nx;
  const dim3 grid((unsigned)((ntiles + 7) / 8 * 8)), block(256);
  if (big)
    hipLaunchKernelGGL((block_score_kernel<2, 1>), grid, block, 0, s, pq, pk, nqb, nkb, scores, knorm, nx, ny, ntiles);
  else
    hipLaunchKernelGGL((block_score_kernel<1, 1>), grid, block, 0, s, pq, pk, nqb, nkb, scores, knorm, nx, ny, ntiles);
  return hipGetLastError();
}

hipError_t launch_topk_select(const SelectArgs& a, hipStream_t s) {
  if (a.rows == 0) return hipSuccess;
  if (a.nkb <= 64 * 8) return launch_select<8>(a, s);
  if (a.nkb <= 64 * 16) return launch_select<16>(a, s);
  if (a.nkb <= 64 * 32) return launch_select<32>(a, s);
  if (a.nkb <= 64 * 64) return launch_select<64>(a, s);
  return launch_select<96>(a, s);
}

}  // namespace bsa
