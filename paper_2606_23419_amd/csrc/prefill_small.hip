// Prefill of short prompts over the nested layout (the contract of prefill.hip:
// every channel at b_max bits, weights rounded once to fp16, float32 sums that
// repeat bit for bit).  The tiles of prefill.hip leave the chip idle when there
// are few tokens: 128 x 128 tiles of 4096 outputs are 32 workgroups, each walking
// all of K (60 us whatever M).
//
// A wave computes 16 MT tokens x 64 outputs over its share of K, 64 channels a
// turn; the 8 waves of a workgroup split K 8 / CW ways over CW neighbouring
// columns and meet once at the end, so the loop has no barrier.  Per turn
//   - a lane reads one channel's 64 outputs, 16 bytes of each 2-bit plane
//     (8 of a 1-bit plane), assembles the codes, turns them into fp16 weights
//     (0x6400 | q reads as 1024 + q; minus 1152, exact; times the fp16 group
//     scale, uniform over the wave, one rounding) and writes them as one row
//     [k][n] of the wave's own LDS tile, in the order the unpack leaves them;
//   - ds_read_b64_tr_b16 hands them back with k along the lane's registers,
//     the operand of v_mfma_f32_16x16x32_f16; the token operand comes straight
//     from memory (16 bytes of 8 channels per lane).
// The next turn's planes and tokens are loaded while one is multiplied.  The
// waves' partial sums are added in wave order, 16 tokens at a time.
//
// Few columns also split K over two workgroups that add into a cleared y: 0 + a
// + b is the same in either order, so the result still repeats.  Adding to the
// caller's y would not: there one workgroup takes both halves of K in turn and
// adds a + b, so that y grows by exactly what overwriting it would store.
//
// Bound by the 16-byte plane pieces a lane reads, a cache line each (about 2.7
// cycles per piece and CU), and by M from about 40 tokens on by the token loads.
// us per call, before (prefill.hip) and now, at M = 1 / 16 / 77: 4096 -> 4096 59 / 60 / 61
// and 17 / 19 / 28, 4096 -> 6144 61 / 62 / 63 and 19 / 20 / 30, 14336 -> 4096 209 / 209 / 219 and
// 46 / 50 / 76, 4096 -> 28672 95 / 94 / 98 and 53 / 58 / 82.
#include "grinqh_internal.h"
#include "vmm_common.h"

namespace grinqh {

namespace {

using vmmdev::assemble_codes;
using vmmdev::spread_bits;

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));

constexpr int kPsWaves = 8;
constexpr int kPsK = 64;                   // channels per turn, one per lane
constexpr int kPsN = 64;                   // outputs per wave

// (q_a - 128, q_b - 128) s from bytes a and b of q: exact, then one rounding
__device__ __forceinline__ uint32_t weights2(uint32_t q, uint32_t a, uint32_t b, uint32_t s) {
  const uint32_t v = __builtin_amdgcn_perm(0x64646464u, q, a | 0x0400u | (b << 16) | 0x04000000u);
  const half2v c = {(_Float16)1152.0f, (_Float16)1152.0f};
  return __builtin_bit_cast(uint32_t, (__builtin_bit_cast(half2v, v) - c) * __builtin_bit_cast(half2v, s));
}

// The output (of 16) at place pos of a chunk as the unpack leaves it: dword j =
// pos / 2 holds outputs 8 (j & 1) + (j >> 1) and that + 4.
__device__ __forceinline__ int output_at(int pos) { return 8 * ((pos >> 1) & 1) + (pos >> 2) + 4 * (pos & 1); }

// HALVES: halves of K that a workgroup takes, one after the other (2 only
// without CW, and then gridDim.y is 1).
template <int U, int MT, int CW, int HALVES>
__global__ __launch_bounds__(64 * kPsWaves, 2) void k_prefill_small(
    const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales, const uint16_t* __restrict__ x,
    float* __restrict__ y, Layer L, int M, int accumulate, int row_blocks) {
  constexpr int C = kPsN / 16;
  constexpr int KW = kPsWaves / CW;        // waves that split K
  constexpr int kPsRow = 2 * kPsN + 16;    // bytes of a channel's row in LDS, padded for the banks
  constexpr int P = 8 / U;                 // planes of the widest code
  constexpr int WD = U * C / 2;            // dwords of the outputs in a plane row
  constexpr int RED = kPsN + 4;            // floats of a token's row of partial sums
  constexpr int OUTS = CW * 16 * kPsN / (64 * kPsWaves);   // outputs of 16 tokens per thread
  static_assert(HALVES == 1 || CW == 1, "two columns are never split");
  __shared__ __align__(16) uint8_t s_w[kPsWaves][kPsK * kPsRow];
  static_assert(sizeof(s_w) >= kPsWaves * 16 * RED * 4, "the partial sums reuse the tiles");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Workgroup i runs on XCD i mod 8; each XCD gets a contiguous run of columns
  // (the plane lines eight neighbours share are then fetched by one L2), the
  // row blocks of a column one after another.
  int ctile, rblk;
  {
    const int G = (int)gridDim.x, i = (int)blockIdx.x;
    const int xcd = i & 7, per = G >> 3, extra = G & 7;
    const int pos = xcd * per + min(xcd, extra) + (i >> 3);
    rblk = pos % row_blocks;
    ctile = pos / row_blocks;
  }
  const int cw = wave % CW, kw = wave / CW;
  const int n0 = (ctile * CW + cw) * kPsN, m0 = rblk * 16 * MT;
  const int K = L.K, tile = n0 / L.T, o0 = n0 - tile * L.T;
  const int np = L.P, plane_bytes = L.T * U / 8;
  // this workgroup's turns of 64 channels: all, or every other 8 (a half of K)
  const int turns = K / kPsK, stride = KW * (int)gridDim.y * HALVES;
  const int i16 = lane & 15, h = lane >> 4;

  const uint8_t* wsrc = codes + ((size_t)tile * K + lane) * L.RB + o0 * U / 8;
  const uint16_t* xsrc[MT];                // rows past M repeat the last one (never stored)
#pragma unroll
  for (int m = 0; m < MT; ++m) xsrc[m] = x + (size_t)min(m0 + 16 * m + i16, M - 1) * K + 8 * h;

  struct Turn {
    uint32_t w[P][WD];
    uint32_t s;                            // scales of outputs 2 (lane % 32) and that + 1
    half8 x[MT][2];
  };
  auto load = [&](Turn& R, int t) __attribute__((always_inline)) {
    const uint8_t* p = wsrc + (size_t)t * kPsK * L.RB;
    R.s = *(const uint32_t*)(scales + (size_t)(t * kPsK / kGroup) * L.N + n0 + 2 * (lane & 31));
#pragma unroll
    for (int j = 0; j < P; ++j)            // (a plane the code does not have reads plane 1 again, unused)
      __builtin_memcpy(R.w[j], __builtin_assume_aligned(p + (j < np ? j : 0) * plane_bytes, 2 * U * C < 16 ? 2 * U * C : 16), 4 * WD);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) R.x[m][ks] = *(const half8*)(xsrc[m] + t * kPsK + 32 * ks);
  };

  float4v acc[MT][C];
  uint8_t* tile_w = s_w[wave];
  const __attribute__((address_space(3))) uint8_t* rd =
      (const __attribute__((address_space(3))) uint8_t*)tile_w + (8 * h + (i16 >> 2)) * kPsRow + 8 * (i16 & 3);
  auto consume = [&](const Turn& R) __attribute__((always_inline)) {
    auto sp = [&](int i) __attribute__((always_inline)) { return (uint32_t)__builtin_amdgcn_readlane((int)R.s, i); };
#pragma unroll
    for (int c = 0; c < C; ++c) {          // 16 outputs
      uint32_t w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if constexpr (U == 2) {
          w[j] = j < np ? R.w[j][c] : 0u;
        } else {
          const uint32_t a = 2 * j < np ? (R.w[2 * j][c / 2] >> (16 * (c & 1))) & 0xFFFFu : 0u;
          const uint32_t b = 2 * j + 1 < np ? (R.w[2 * j + 1][c / 2] >> (16 * (c & 1))) & 0xFFFFu : 0u;
          w[j] = (spread_bits(a) << 1) | spread_bits(b);
        }
      }
      uint32_t q[4], o[8];
      assemble_codes(w[0], w[1], w[2], w[3], q);   // byte i of q[d]: output 4 i + d
#pragma unroll
      for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int p = 0; p < 2; ++p) {      // outputs 8 p + d and 8 p + 4 + d
          const uint32_t lo = sp(8 * c + 4 * p + (d >> 1)), hi = sp(8 * c + 4 * p + 2 + (d >> 1));
          const uint32_t s = d & 1 ? (lo >> 16) | (hi & 0xFFFF0000u) : (lo & 0xFFFFu) | (hi << 16);
          o[2 * d + p] = weights2(q[d], 2 * p, 2 * p + 1, s);
        }
      *(uint4*)(tile_w + lane * kPsRow + 32 * c) = make_uint4(o[0], o[1], o[2], o[3]);
      *(uint4*)(tile_w + lane * kPsRow + 32 * c + 16) = make_uint4(o[4], o[5], o[6], o[7]);
    }
    // the tile is this wave's own and its LDS accesses complete in order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int n = 0; n < C; ++n) {
        half8 b;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          const half4 v = __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (__attribute__((address_space(3))) short4v*)(rd + (32 * ks + 4 * r) * kPsRow + 32 * n)));
#pragma unroll
          for (int e = 0; e < 4; ++e) b[4 * r + e] = v[e];
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(R.x[m][ks], b, acc[m][n], 0, 0, 0);
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  float kept[HALVES > 1 ? MT : 1][OUTS];   // the first half's sums
#pragma unroll 1
  for (int half = 0; half < HALVES; ++half) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int n = 0; n < C; ++n) acc[m][n] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
    const int first = kw + KW * (int)(HALVES > 1 ? half : blockIdx.y);
    if (half) __syncthreads();             // the partial sums are read: the tiles are free
    if (first < turns) {
      // past the last turn the last one is loaded again (in bounds, never used)
      const int last = first + (turns - 1 - first) / stride * stride;
      Turn ra, rb;
      load(ra, first);
      int t = first;
      // (no condition around a consume: the compiler would move its loads there)
      for (; t + stride < turns; t += 2 * stride) {
        load(rb, t + stride);
        __builtin_amdgcn_sched_barrier(0);   // the loads go out first
        consume(ra);
        load(ra, min(t + 2 * stride, last));
        __builtin_amdgcn_sched_barrier(0);
        consume(rb);
      }
      if (t < turns) consume(ra);
    }

    // ---- the waves' sums, 16 tokens at a time: element r of lane l is token 4 h
    // + r, place i16 of the chunk
    float* red = (float*)&s_w[0][0];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      __syncthreads();
#pragma unroll
      for (int n = 0; n < C; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          red[(wave * 16 + 4 * h + r) * RED + 16 * n + output_at(i16)] = acc[m][n][r];
      __syncthreads();
#pragma unroll
      for (int i = 0; i < OUTS; ++i) {
        const int e = tid + i * 64 * kPsWaves, row = e / (CW * kPsN), cc = e / kPsN % CW, col = e % kPsN;
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < KW; ++w) v += red[((w * CW + cc) * 16 + row) * RED + col];
        v *= L.sfac;                       // 8-bit code units -> b_max units (exact)
        if constexpr (HALVES > 1) {
          if (half == 0) {
            kept[m][i] = v;
            continue;
          }
          v += 0.0f + kept[m][i];          // as in a cleared y
        }
        const int mm = m0 + 16 * m + row;
        if (mm < M) {
          float* dst = y + (size_t)mm * L.N + (ctile * CW + cc) * kPsN + col;
          if (gridDim.y == 2) atomicAdd(dst, v);   // the other half adds too: 0 + a + b in either order
          else *dst = accumulate ? *dst + v : v;
        }
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_zero_prefill(float* __restrict__ y, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = 0.0f;
}

template <int U, int CW, int HALVES>
void launch_mt(int mt, dim3 grid, hipStream_t s, const void* codes, const void* scales, const void* x, int M,
               float* y, int accumulate, const Layer& L, int row_blocks) {
#define GRINQH_PS(MM)                                                                                       \
  case MM:                                                                                                  \
    hipLaunchKernelGGL((k_prefill_small<U, MM, CW, HALVES>), grid, dim3(64 * kPsWaves), 0, s, (const uint8_t*)codes,  \
                       (const uint16_t*)scales, (const uint16_t*)x, y, L, M, accumulate, row_blocks);       \
    break;
  switch (mt) { GRINQH_PS(1) GRINQH_PS(2) GRINQH_PS(3) GRINQH_PS(4) GRINQH_PS(5) }
#undef GRINQH_PS
}

}  // namespace

namespace {

// Row blocks of up to 80 tokens (what a wave's registers hold), evenly filled.
struct Blocks {
  int rows, mt;
  explicit Blocks(int M) {
    const int tiles = (M + 15) / 16;
    rows = (tiles + 4) / 5;
    mt = (tiles + rows - 1) / rows;
  }
};

}  // namespace

// One block of tokens (M <= 80) while the workgroups of 128 outputs are a single
// round of one per CU, or prefill.hip would take its narrower tiles: 32768
// outputs on 256 CUs, M = 80, 4096 channels 68 us against 86, 33792 outputs 135
// against 160; but not with 1-bit planes, M > 64 and a few turns per wave (28672 outputs, M
// = 80: 512 / 1024 / 2048 channels 21.2 / 35.6 / 64 against 20.7 / 33.6 / 63).
// Past that prefill.hip covers 256 outputs per CU and round.  To 32 tokens this
// kernel is still ahead everywhere (65536 outputs, 512 channels, M = 32 24.9 against
// 27.4).  With more tokens it is where it has enough turns of K to pipeline, the
// more of them the more tokens, rounds and bytes a code has, as a share of
// prefill.hip's time over 69632..98304 outputs (its rounds are fewer than twice
// prefill.hip's), and over 40960 / 49152 / 57344 / 65536 outputs (twice):
//   M    bits  channels  fewer        twice
//   48   8     512       0.91..0.93   1.20 1.16 1.11 1.08
//   48   8     2048      0.84         1.07 1.04 0.99 0.96
//   48   8     4096      0.77..0.83   1.02 0.96 0.88 0.84
//   48   4     1024      0.78         0.99 0.97 0.91 0.89
//   48   8, 1-bit planes 2048  0.88   0.98 0.98 0.95 0.93   (1024: 0.95, 1.05)
//   64   8     1024      0.96..0.99   1.25 1.21 1.13 1.11   (512: 1.05)
//   64   8     4096      0.84..0.92   1.14 1.04 0.97 0.93
//   64   8, 1-bit planes 2048  0.97   1.06 1.07 1.04 1.02   (1024: 1.02; 4096: 1.00 1.00 0.97 0.94)
//   64   4     2048      0.81..0.84   1.04 1.02 0.95 0.89
//   80   6     4096      0.92..1.00   1.23 1.13 1.04 0.97   (2048: 1.04)
//   80   4     4096      0.81..0.89   1.11 1.04 0.94 0.89   (2048: 0.87..0.95, 1024: 1.01)
// and to 256 channels, where no wave has a second turn: fewer rounds 0.70..0.96, twice 0.87..0.98
// at M = 48, at M = 64 only with 1-bit planes 0.90..0.95 (1.00..1.06 with 2-bit ones).
// M = 80 at 8 bits is prefill.hip's: 65536 outputs, 1024 / 4096 channels 48 / 156 against
// 42 / 146.
// More blocks as long as one workgroup per 64 outputs and block leaves a single
// round on the chip: 4096 -> 4096 at M = 256 (256 workgroups) 39 us against 63,
// 14336 -> 4096 111 against 211, 4096 -> 6144 at M = 128 (192) 40 against 65 but at
// M = 256 (384) 72 against 65.
bool prefill_small_takes(const Layer& L, int M) {
  if (M > 80 * 256) return false;
  const Blocks b(M);
  const long cus = device_cus(), pairs = L.N / (2 * kPsN);
  if (b.rows > 1) return 2 * pairs * b.rows <= cus;
  if (2 * pairs <= cus) return true;
  const bool one_turn = L.K <= 256;
  if (L.u == 1 && b.mt == 5 && !one_turn && L.K < 2048) return false;
  const long rounds = (pairs + cus - 1) / cus;
  if (rounds == 1 || b.mt <= 2 || !prefill_wide(L, M)) return true;
  const bool light = L.u == 2 && L.bmax <= 4;
  if (rounds < 2 * ((L.N / 256 + cus - 1) / cus)) {   // (prefill.hip's rounds)
    if (one_turn || b.mt == 3) return true;
    if (b.mt == 4) return L.K >= (L.u == 2 ? 1024 : 2048);
    return L.bmax < 8 && L.K >= (light ? 2048 : 4096);
  }
  if (one_turn) return b.mt == 3 || (b.mt == 4 && L.u == 1);
  const long quarters = 4 * (pairs - (rounds - 1) * cus) / cus;   // of the last round
  if (light) return L.K >= (b.mt == 3 ? 1024 : b.mt == 4 && quarters >= 3 ? 2048 : 4096) && (b.mt < 5 || quarters >= 3);
  if (b.mt == 5 || L.K < (b.mt == 3 ? 2048 : 4096)) return false;
  return L.u == 1 || quarters >= (b.mt == 3 && L.K >= 4096 ? 2 : 3);
}

int launch_prefill_small(const Layer& L, const void* codes, const void* scales, const void* x, int M, float* y,
                         int accumulate, hipStream_t s) {
  const Blocks b(M);
  const int row_blocks = b.rows, mt = b.mt;
  const long wgs = (long)(L.N / kPsN) * row_blocks;
  // more than a round of workgroups: two columns share one (82 against 94 us at
  // 4096 -> 28672, M = 77); at most half a round: K split in two (28 against 42 us at
  // 4096 -> 4096, M = 77 and 27 against 36 at M = 128; above, 4096 -> 6144 at M = 128 has 192
  // workgroups of 256 CUs and took 51 split, 40 not), but not where the first half's
  // waves take all of K in one turn each (128 -> 8192, M = 80 8.9 split, 6.5 not)
  const int cus = device_cus();
  const int cw = wgs > cus ? 2 : 1;
  const bool halves = wgs <= cus / 2 && L.K > kPsK * kPsWaves;
  const int split = halves && !accumulate ? 2 : 1;   // else one workgroup takes both halves in turn
  const dim3 grid((unsigned)(L.N / (kPsN * cw) * row_blocks), (unsigned)split);
  if (split == 2) {
    const long n = (long)M * L.N;
    hipLaunchKernelGGL(k_zero_prefill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, y, n);
    const int st = check_launch("prefill zero-fill");
    if (st) return st;
  }
#define GRINQH_PS(UU, CC, HH) launch_mt<UU, CC, HH>(mt, grid, s, codes, scales, x, M, y, accumulate, L, row_blocks)
  if (L.u == 2) {
    if (cw == 2) GRINQH_PS(2, 2, 1);
    else if (halves && accumulate) GRINQH_PS(2, 1, 2);
    else GRINQH_PS(2, 1, 1);
  } else {
    if (cw == 2) GRINQH_PS(1, 2, 1);
    else if (halves && accumulate) GRINQH_PS(1, 1, 2);
    else GRINQH_PS(1, 1, 1);
  }
#undef GRINQH_PS
  return check_launch("prefill (short)");
}

}  // namespace grinqh
