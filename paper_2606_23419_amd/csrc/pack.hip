// Offline quantise + nest + pack (Sec. 3.3 "Storage Layout and Weight
// Loading"; App. C.1 "Sparse bit-loading", "Bit-packing").
//
// One kernel: a workgroup quantises OUT outputs of one group of 128 channels
// (the source is read once), keeps their codes in LDS and writes their fields
// into the u-bit planes of the group's rows.  Bound by memory: 4096 -> 28672 from
// fp16 moves 354 MB, 74 us at the rate of a copy, and takes 97 us (a scale kernel
// and a kernel with one thread per 32 outputs and channel, 2-byte loads and
// 8-byte stores a row apart: 508 us).
#include "grinqh_internal.h"

namespace grinqh {

// Externally quantised codes: scales arrive [n][g] and are stored [g][n].
__global__ __launch_bounds__(256) void k_transpose_scales(const uint16_t* __restrict__ src,
                                                          uint16_t* __restrict__ dst, int N, int G) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)N * G) return;
  const int g = (int)(i / N), n = (int)(i % N);
  dst[i] = src[(size_t)n * G + g];
}

// Maximum over the 16 lanes of a row, in every lane.
__device__ __forceinline__ uint32_t row_max(uint32_t v) {
#define GRINQH_ROR(n)                                                                                       \
  {                                                                                                         \
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 + n, 0xF, 0xF, false);        \
    v = v > o ? v : o;                                                                                      \
  }
  GRINQH_ROR(8) GRINQH_ROR(4) GRINQH_ROR(2) GRINQH_ROR(1)
#undef GRINQH_ROR
  return v;
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef int v2i __attribute__((ext_vector_type(2)));

// Eight fp16 weights (pairs in w) to codes: bytes of q.  The reference is
// rne(fp32 w / s).  r = w rcp(s) is off by less than 2^-15 for |r| <= 128; one
// residual step r + (w - r s) rcp(s) (the residual is exact) leaves it within
// 2^-24 relative, and exact where w / s is a multiple of 1/2.  w and s have 11-bit
// significands, so any other quotient is at least 2^-13 from the nearest
// rounding boundary: neither this error nor that of adding h (2^-17) moves it
// across, and boundaries themselves round to even in both.  s = 0: inv = 0 and
// every code is h.  Not finite, as the quotient gives it: a NaN (w, or inf / inf)
// is code 0 (lo; h where s = 0); beside an infinity (the caller passes s = inv =
// 0) the rest are h.
__device__ __forceinline__ void quantise8(const uint32_t (&w)[4], float s, float inv, float h, float lo,
                                          uint32_t (&q)[2]) {
  q[0] = q[1] = 0u;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float x = h2f((uint16_t)(i & 1 ? w[i / 2] >> 16 : w[i / 2] & 0xFFFFu));
    const float r = x * inv;
    const float e = fmaf(-r, s, x);
    float c = rintf(fmaf(e, inv, r) + h);
    c = __builtin_amdgcn_fmed3f(c, lo, 2.0f * h - 1.0f);   // a NaN: lo
    q[i / 4] |= (uint32_t)c << (8 * (i % 4));
  }
}

// 16 bytes at p; ALIGNED: p is 16-byte aligned, else it may have any alignment
// its elements allow.
template <bool ALIGNED, typename E, int NE>
__device__ __forceinline__ void load_elems(const E* p, uint32_t (&w)[NE * sizeof(E) / 4]) {
  constexpr int PER = 4 / sizeof(E);
  if constexpr (ALIGNED) {
    __builtin_memcpy(w, __builtin_assume_aligned(p, NE * sizeof(E)), NE * sizeof(E));
  } else {
#pragma unroll
    for (int i = 0; i < NE / PER; ++i) {
      w[i] = 0u;
#pragma unroll
      for (int j = 0; j < PER; ++j) w[i] |= (uint32_t)p[i * PER + j] << (8 * (int)sizeof(E) * j);
    }
  }
}

// A workgroup: OUT outputs (OUT divides the tile width) of group blockIdx.y,
// OUT threads.  Phase 1: 16 lanes read a row's 128 channels (one line of fp16),
// their maximum gives the scale, their codes go to LDS as [output][channel].
// Phase 2: ds_read_b64_tr_b8 hands a lane one channel's codes of eight
// outputs; a lane takes 64 consecutive outputs of its channel, presses plane by
// plane four codes' fields into a byte and stores each plane's 16 bytes (8 for
// U = 1); four lanes cover 256 outputs of a plane row.  b_max-bit codes are
// left-aligned in their bytes, so plane j's field is the same bit slice for
// every b_max.
template <int U, int OUT, bool FP16, bool ALIGNED>
__global__ __launch_bounds__(OUT) void k_pack(const void* __restrict__ src, uint16_t* __restrict__ scales,
                                              uint8_t* __restrict__ out, Layer L) {
  constexpr int P = 8 / U;                 // planes of the widest (8-bit) code
  constexpr int STRIDE = 144;              // bytes of an output's codes in LDS, padded for the banks
  constexpr int ROWS = OUT / 16;           // outputs per round of phase 1
  __shared__ __align__(16) uint8_t s_q[OUT * STRIDE];
  const int tid = threadIdx.x, c = tid & 15;
  const int n0 = blockIdx.x * OUT, g = blockIdx.y;
  const size_t k0 = (size_t)g * kGroup;
  const float h = (float)(1 << (L.bmax - 1));
  const int align = 8 - L.bmax;
  const uint32_t keep = 0x01010101u * (uint32_t)((0xFF << align) & 0xFF);

#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int o = ROWS * i + (tid >> 4);
    const size_t at = (size_t)(n0 + o) * L.K + k0 + 8 * c;
    uint32_t q[2];
    if constexpr (FP16) {
      uint32_t w[4];
      load_elems<ALIGNED, uint16_t, 8>((const uint16_t*)src + at, w);
      // magnitudes 0 .. 0x7C00 (infinity) raised to the top of 16 bits, where NaN
      // wraps to the bottom: the maximum leaves NaN out, unless all are
      constexpr unsigned short kUp = 0x83FF;
      const u16x2 up = {kUp, kUp};
      u16x2 m = __builtin_bit_cast(u16x2, w[0] & 0x7FFF7FFFu) + up;
#pragma unroll
      for (int j = 1; j < 4; ++j) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w[j] & 0x7FFF7FFFu) + up);
      const uint32_t mx = (row_max(m[0] > m[1] ? m[0] : m[1]) - kUp) & 0xFFFFu;
      // s = fp16_rne(fp32(max|w|) / (2^(b_max-1) - 1))
      const uint16_t sb = f2h_rn(__fdiv_rn(h2f((uint16_t)mx), h - 1.0f));
      const float s = h2f(sb);
      if (c == 0) scales[(size_t)g * L.N + n0 + o] = sb;
      const bool in_range = s != 0.0f && sb != 0x7C00u;
      quantise8(w, in_range ? s : 0.0f, in_range ? __builtin_amdgcn_rcpf(s) : 0.0f, h,
                s == 0.0f ? h : 0.0f, q);
    } else {
      load_elems<ALIGNED, uint8_t, 8>((const uint8_t*)src + at, q);
    }
    // (bits above b_max of a given code drop out)
    *(uint2*)&s_q[o * STRIDE + 8 * c] = make_uint2((q[0] << align) & keep, (q[1] << align) & keep);
  }
  __syncthreads();

  const int lane = tid & 63, wave = tid >> 6;
  const int i16 = lane & 15, hq = lane >> 4;
  const int tile = n0 / L.T, plane_bytes = L.T * U / 8;
#pragma unroll 1
  for (int unit = wave; unit < 8 * (OUT / 256); unit += OUT / 64) {
    const int kb = (unit & 7) * 16, ob = (unit >> 3) * 256 + hq * 64;   // channels, the lane's first output
    const __attribute__((address_space(3))) uint8_t* p =
        (const __attribute__((address_space(3))) uint8_t*)s_q + (ob + (i16 >> 1)) * STRIDE + kb + 8 * (i16 & 1);
    uint32_t code[16];                     // four outputs each
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const v2i v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) v2i*)(p + 8 * r * STRIDE));
      code[2 * r] = (uint32_t)v.x;
      code[2 * r + 1] = (uint32_t)v.y;
    }
    uint8_t* row = out + ((size_t)tile * L.K + k0 + kb + i16) * L.RB + (size_t)(n0 + ob - tile * L.T) * U / 8;
#pragma unroll
    for (int j = 0; j < P; ++j) {
      if (j >= L.P) break;
      uint32_t d[2 * U];
#pragma unroll
      for (int w = 0; w < 2 * U; ++w) {
        d[w] = 0u;
#pragma unroll
        for (int e = 0; e < 8 / U; ++e) {
          // the four fields of a dword, at bit 0 of its bytes, side by side
          const uint32_t f = (code[8 / U * w + e] >> (8 - (j + 1) * U)) & (0x01010101u * ((1u << U) - 1u));
          const uint32_t y = f | (f >> (8 - U));
          const uint32_t z = (y | (y >> (16 - 2 * U))) & ((1u << (4 * U)) - 1u);
          d[w] |= z << (4 * U * e);
        }
      }
      uint8_t* dst = row + (size_t)j * plane_bytes;
      if constexpr (ALIGNED) {
        __builtin_memcpy(__builtin_assume_aligned(dst, 8 * U), d, 8 * U);
      } else {
#pragma unroll
        for (int w = 0; w < 2 * U; ++w) ((uint32_t*)dst)[w] = d[w];
      }
    }
  }
}

template <int U, int OUT, bool FP16>
void launch_aligned(bool aligned, hipStream_t s, const void* src, uint16_t* scales, uint8_t* out, const Layer& L) {
  const dim3 grid((unsigned)(L.N / OUT), (unsigned)L.groups);
  if (aligned) hipLaunchKernelGGL((k_pack<U, OUT, FP16, true>), grid, dim3(OUT), 0, s, src, scales, out, L);
  else hipLaunchKernelGGL((k_pack<U, OUT, FP16, false>), grid, dim3(OUT), 0, s, src, scales, out, L);
}

int launch_pack(const Layer& L, int src_kind, const void* src, const void* src_scales,
                void* packed_codes, void* packed_scales, hipStream_t s) {
  const bool from_fp16 = src_kind == GRINQH_SRC_FP16_RTN;
  if (!from_fp16 && src_scales) {   // codes without scales: the look-up-table format
    const long n = (long)L.N * L.groups;
    hipLaunchKernelGGL(k_transpose_scales, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       (const uint16_t*)src_scales, (uint16_t*)packed_scales, L.N, L.groups);
    const int st = check_launch("pack scales");
    if (st) return st;
  }
  // Wide loads and stores where source and destination allow them (torch's
  // buffers do); rows of K elements keep the alignment (K is a multiple of 128).
  const bool aligned = (((uintptr_t)src | (uintptr_t)packed_codes) & 15u) == 0;
  uint16_t* sc = (uint16_t*)packed_scales;
  uint8_t* out = (uint8_t*)packed_codes;
  // 512 outputs per workgroup where the tile has them: whole 128-byte lines of a
  // 2-bit plane row
#define GRINQH_PACK(UU, OO)                                                    \
  if (from_fp16) launch_aligned<UU, OO, true>(aligned, s, src, sc, out, L);     \
  else launch_aligned<UU, OO, false>(aligned, s, src, sc, out, L)
  if (L.u == 2) {
    if (L.T >= 512) { GRINQH_PACK(2, 512); } else { GRINQH_PACK(2, 256); }
  } else {
    GRINQH_PACK(1, 512);   // (tiles of 1-bit planes are at least 512 wide)
  }
#undef GRINQH_PACK
  return check_launch("pack codes");
}

}  // namespace grinqh
