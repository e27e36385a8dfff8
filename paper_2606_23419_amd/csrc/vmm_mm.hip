// Nested-precision decode VMM for 1..4 tokens on the matrix cores (Sec. 3.3
// reconstruction with the midpoint bias; App. C.1 sparse bit-loading).
//
// A workgroup of 8 waves owns one group of 128 channels and a run of columns of
// W outputs (a tile or a W-wide part of it).  The plane rows that are read go
// straight from memory to LDS, all of a column's in flight at once (the other
// workgroups of the CU multiply meanwhile), and the contraction runs on
// v_mfma_i32_16x16x64_i8 with exact integers.  Grading, lists and the x operand
// are made once for the run.
//
//   - Lists.  Waves 2j and 2j+1 grade channels 32j .. 32j+31 and list the rows
//     to read (channel by channel, each to its depth; for several tokens the
//     deepest), 16 rows to a block, so only rows that are read take LDS space
//     and matrix work.  The four lists' i-th blocks form a step: 64 rows, one
//     matrix instruction's K.  The two waves share the copies of
//     their list.
//   - ds_read_b64_tr_b4 hands a lane the nibble of one byte column for the 16
//     rows of a block, so a lane holds one output's fields along K, as the
//     matrix instruction wants them: a mask (and a shift for the high nibbles)
//     turns two dwords into int8 operands of 16 rows.  A nibble holds 4/U
//     outputs; output e's field stays at its bit e*U, and its sums are scaled
//     by 2^(-e*U) at the end.
//   - x becomes a fixed-point integer X = rne(x 2^s), s from the largest |x|
//     of the group so that |X| < 2^24 (2^23 for 1-bit planes): an fp32-like 24
//     bits at the largest channel, exact down to 2^-13 of it (2^-12).  beta is
//     made of the same X.  Where the channels below that lose more than 2 units
//     of X together, add_rests puts back what they lost: so a group's x is
//     exact but for at most 2^-22 (2^-21) of its largest |x|, in all.  For a row of
//     plane j, X is shifted to the plane's weight 2^(8 - j U) and cut into four
//     balanced int8 digits; the digits of the NB tokens are the columns (4 NB
//     <= 16) of the B operand.  A token's digits are zero on planes beyond its
//     own depth, so tokens share the loads and the products.
//   - products and sums are exact in int32 (|sum| < 2^21).  The digits meet in
//     fp32 once per output.
//
// What bounds it: latencies in a chain (launch, x, grading, the first rows, the
// sums), and on large layers instruction issue beside memory.  Graphs of one
// projection at 4 bits, us per launch, against the kernels it took over from
// (per-plane or merged-nibble dequantisation in registers, v_dot2_f32_f16):
// B = 1 4096 -> 6144 7.7 -> 6.0, 4096 -> 4096 6.2 -> 5.3, 14336 -> 4096 10.2 -> 9.6,
// 1024 -> 1024 4.6 -> 3.6; B = 4 4096 -> 28672 45 -> 24, 4096 -> 4096 12.2 -> 7.2; 1-bit
// planes B = 1 4096 -> 24576 30.2 -> 15.3, 12288 -> 4096 18.4 -> 9.5.  Error against
// float64 2e-7 (2-norm), before 1e-6 to 2e-5.
// Measured and not kept: a ring of 8 KB steps over several groups with a
// barrier per step (4096 -> 28672 at B = 1 17-19 us: barriers and per-step
// overhead); two columns in LDS with the next one's copies behind (16.8: two
// workgroups per CU instead of three); four waves, one group per workgroup
// without lists (18.6); float accumulation on v_mfma_scale_f32_16x16x128 with
// fp4 fields and x cut into bf8 terms (sums rounded to about 18 bits).
//
// add_rests costs such a workgroup some microseconds.  No group needs it where
// the smallest activations are skipped (Student-t and SwiGLU x, 20% at level 0);
// with every channel active 0.01% of the groups do (0.06% with 1-bit planes).
// Having it costs the others little: 4096 -> 6144 at 2 bits 4.96 -> 5.09 us, at 4 bits 6.17 ->
// 6.21, four tokens 8.92 -> 9.06, two tokens at 8 bits 8.20 -> 8.84 (the most seen).  What
// it needs lies in masks and in the B columns' pads: as bytes of LDS it took a workgroup
// from each CU at b_max 4 and four tokens (14336 -> 4096 12.1 -> 14.8 us, now 12.0).
//
// Per group and output y_n += s_{g,n} (sum_k X_k t_k 2^-s + beta_g), t_k the
// code truncated to the channel's level (8-bit units), beta_g = sum over
// active channels of x_k (phi_b - 128).
#include "grinqh_internal.h"
#include "topk_select.h"
#include "vmm_common.h"

namespace grinqh {

namespace {

using namespace vmmdev;

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;

__device__ __forceinline__ uint32_t lds_addr(const void* p) { return (uint32_t)(uintptr_t)(const lds_u8*)p; }

// Maximum over the wave (unsigned), in a scalar.
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#define GRINQH_MAX_STEP(ctrl, rows)                                                               \
  {                                                                                               \
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xF, false);  \
    v = v > o ? v : o;                                                                            \
  }
  GRINQH_MAX_STEP(0x111, 0xF)   // row_shr:1
  GRINQH_MAX_STEP(0x112, 0xF)
  GRINQH_MAX_STEP(0x114, 0xF)
  GRINQH_MAX_STEP(0x118, 0xF)
  GRINQH_MAX_STEP(0x142, 0xA)   // row_bcast:15
  GRINQH_MAX_STEP(0x143, 0xC)   // row_bcast:31
#undef GRINQH_MAX_STEP
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Truncating conversion with the hardware's defined result for every input
// (saturated; 0 for NaN).
__device__ __forceinline__ int cvt_i32(float v) {
  int r;
  asm("v_cvt_i32_f32 %0, %1" : "=v"(r) : "v"(v));
  return r;
}

// The bytes of dg to LDS at a, a + S, a + 2 S, a + 3 S.
template <int S>
__device__ __forceinline__ void store_digits(uint32_t a, uint32_t dg) {
  const uint32_t d8 = dg >> 8;
  asm volatile(
      "ds_write_b8 %0, %1\n\tds_write_b8 %0, %2 offset:%3\n\t"
      "ds_write_b8_d16_hi %0, %1 offset:%4\n\tds_write_b8_d16_hi %0, %2 offset:%5"
      ::"v"(a), "v"(dg), "v"(d8), "n"(S), "n"(2 * S), "n"(3 * S) : "memory");
}

// 16 bytes per lane from the resource at byte offset off to LDS at lds + 16
// lane.  As asm, so that the copies in flight are counted here alone: the
// compiler would hold every LDS access it cannot tell apart until they land.
// It has no register output; whoever reads the LDS bytes waits (vmcnt) first.
__device__ __forceinline__ void copy_to_lds(uint32_t lds, uint32_t off, v4i rsrc) {
  int m0;                                  // an output: m0 is reserved and can't be a clobber
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen nt lds"
               : "={m0}"(m0) : "s"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(off), "s"(rsrc) : "memory");
}

// v added to *p in one memory instruction, which wait_copies counts (an
// atomicAdd may become another number of them).
__device__ __forceinline__ void add_to(float* p, float v) {
  asm volatile("global_atomic_add_f32 %0, %1, off" ::"v"(p), "v"(v) : "memory");
}

// The wave's own LDS accesses complete in order: it is enough to keep the
// compiler from moving them.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kMmThreads = 512;

// The scalars of a launch, in one stretch of the kernel arguments.
struct MmArgs {
  int N, log2_T, RB, n_top;
  uint64_t planes;
  int bmax, n_cut;                         // n_cut: thresholds in use
  float sfac;
  float theta[kMaxLevels - 1];
};

template <int U, int W, int PL, int NB, bool FULL>
struct MmShape {
  static constexpr int PBY = W * U / 8;              // bytes of one plane row of the W outputs
  static constexpr int CHK = PBY / 16;               // 16-byte chunks of it
  static constexpr int BLKB = 16 * PBY;              // bytes of a block
  static constexpr int MAXB = 2 * PL;                // blocks of a list, steps of a column at most
  static constexpr int COLS = 4 * NB;                // B columns: four digits per token
  static constexpr int COLB = MAXB * 64 + 16;        // bytes of one B column (padded)
  static constexpr int LEFT = MAXB * 64;             // in the pad of column j: what list j leaves of each token's x
  static constexpr int OW = W / 8;                   // outputs per wave
  static constexpr int OWP = OW + 4;
  static constexpr int NSL = 4 / U;                  // outputs per nibble
  static constexpr int NCB = PBY / 64;               // 8-byte column blocks per wave
  static constexpr int RED = 8 * COLS * OWP * 4;     // the digit sums, over the weights' place
  // Steps of a column that LDS holds at once, three workgroups per CU (at the
  // 4-bit budgets a list has 64 +- 6 rows of 2-bit planes, five steps).  The
  // first FIRST are multiplied while the others arrive; steps past SCAP then
  // take their place.  FULL: all of them, for launches of two workgroups per CU.
  static constexpr int FIXED = COLS * COLB + 4 * 16 * MAXB * 2 + 2 * W + 16 * NB + 16 * PL * NB + 64;
  static constexpr int FIT = (160 * 1024 / 3 - FIXED) / (4 * BLKB);
  static constexpr int SCAP = FULL || FIT > MAXB ? MAXB : FIT > MAXB / 2 ? FIT : MAXB / 2 + 1;
  static constexpr int FIRST = (SCAP + 1) / 2 > MAXB - SCAP ? (SCAP + 1) / 2 : MAXB - SCAP;
  static constexpr int WB = 4 * SCAP * BLKB > RED ? 4 * SCAP * BLKB : RED;
  static_assert(FIRST < SCAP && FIRST >= 2, "LDS");
};

// Wait until at most n of this wave's copies (and whatever came after them)
// are in flight, for a wave-uniform n.
__device__ __forceinline__ void wait_copies(int n) {
#define GRINQH_WAIT(i)                                     \
  case i:                                                  \
    asm volatile("s_waitcnt vmcnt(" #i ")" ::: "memory"); \
    break;
  switch (n) {
    GRINQH_WAIT(1) GRINQH_WAIT(2) GRINQH_WAIT(3) GRINQH_WAIT(4) GRINQH_WAIT(5) GRINQH_WAIT(6)
    GRINQH_WAIT(7) GRINQH_WAIT(8)
    default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
#undef GRINQH_WAIT
}

__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

constexpr float kRestMax = 2.0f;         // units of X
constexpr float kRestList = 0.25f;       // what a list may leave in any case
constexpr int kMuchLeft = 1 << 16;       // in a list's number of blocks: it leaves more than a quarter of that

// What rounding to X left of x, for one token and the W outputs from n0 on:
//   y_n += s_n sum_k rest_k (t_k + phi_b - 128) unit,  rest_k = x_k to_fix - X_k
// in units of X.  deeper[j][p]: the channels of list j read to more than p planes,
// valid in lists with left > kRestList (the others' rests stay out).  All threads call it, after a barrier; sum: W floats of LDS.
template <int U, int W, int PL>
__device__ __forceinline__ void add_rests(const uint16_t* x, const uint8_t* rows, const uint16_t* scales, float* y,
                                          const uint32_t* deeper, const float* left, int left_stride, float* sum,
                                          float to_fix,
                                          float unit, int RB, int plane_bytes, int bmax) {
  constexpr int CW = W / 16;               // 16 outputs per thread, 16 or 32 rows at once
  const int tid = threadIdx.x, o0 = 16 * (tid % CW);
  for (int o = tid; o < W; o += kMmThreads) sum[o] = 0.0f;
  lds_barrier();
  float acc[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
#pragma unroll 1
  for (int r = tid / CW; r < kGroup; r += kMmThreads / CW) {
    const float fix = h2f(x[r]) * to_fix, rest = fix - rintf(fix);
    int d = 0;
    if (left[(r >> 5) * left_stride] > kRestList && rest != 0.0f)
#pragma unroll
      for (int p = 0; p < PL; ++p) d += (int)(deeper[(r >> 5) * PL + p] >> (r & 31)) & 1;
    const uint8_t* row = rows + (size_t)r * RB + o0 * U / 8;
    uint32_t m[PL], c[4], q[4];            // planes; 2-bit fields; codes: byte i of q[j] is output 4 i + j
#pragma unroll
    for (int p = 0; p < PL; ++p)
      m[p] = p >= d ? 0u : U == 2 ? *(const uint32_t*)(row + p * plane_bytes) : *(const uint16_t*)(row + p * plane_bytes);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (U == 2) c[j] = j < PL ? m[j] : 0u;
      else c[j] = 2 * j < PL ? spread_bits(m[2 * j]) << 1 | spread_bits(m[2 * j + 1]) : 0u;
    }
    assemble_codes(c[0], c[1], c[2], c[3], q);
    const float v = d ? rest : 0.0f, off = v * phi_minus_offset(U * d, bmax);
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] += fmaf(v, (float)((q[e & 3] >> (8 * (e >> 2))) & 0xFFu), off);
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) atomicAdd(&sum[o0 + e], acc[e]);
  lds_barrier();
  for (int o = tid; o < W; o += kMmThreads) atomicAdd(&y[o], h2f(scales[o]) * unit * sum[o]);
  lds_barrier();
}

template <int U, int W, int PL, int NB, bool FULL, bool TOPK>
__global__ __launch_bounds__(kMmThreads, 4) void k_vmm_mm(
    const uint16_t* __restrict__ x, const uint8_t* __restrict__ lm, int K, int fused, int run,
    int cols, const uint8_t* __restrict__ codes, const uint16_t* __restrict__ scales, float* __restrict__ y,
    uint8_t* __restrict__ lm_out, MmArgs A, TopkCuts tk) {
  using S = MmShape<U, W, PL, NB, FULL>;
  constexpr int PBY = S::PBY, CHK = S::CHK, COLB = S::COLB, COLS = S::COLS, MAXB = S::MAXB;
  constexpr int OW = S::OW, OWP = S::OWP, NSL = S::NSL, NCB = S::NCB, BLKB = S::BLKB, SCAP = S::SCAP, FIRST = S::FIRST;

  __shared__ __align__(16) uint8_t s_w[S::WB];            // a column: list by list, SCAP blocks each
  __shared__ __align__(16) uint16_t s_scale[W];
  __shared__ __align__(16) uint8_t s_b[COLS * COLB];
  __shared__ __align__(16) uint16_t s_list[4][16][MAXB];   // row offsets / 64: row r of block b at [r][b]
  __shared__ __align__(16) float s_beta[NB][4];
  __shared__ __align__(16) int s_nblk[4];
  __shared__ __align__(16) uint32_t s_deeper[NB][4][PL];   // lists that leave something: the channels deeper than p planes
  static_assert(!(U == 2 && PL == 2) ||
                    sizeof(s_w) + sizeof(s_scale) + sizeof(s_b) + sizeof(s_list) + sizeof(s_beta) + sizeof(s_nblk) +
                            sizeof(s_deeper) <= 160 * 1024 / 4,
                "four workgroups per CU where rows have two planes");
  static_assert(!TOPK || sizeof(topksel::Scratch) <= sizeof(s_w), "the selection's scratch lies over the weights' place");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int list = wave >> 1, sub = wave & 1, half = lane >> 5;
  const int k0 = blockIdx.y * kGroup;
  const int ch = 32 * list + (lane & 31);  // both halves of both waves hold the channel
  const int k = k0 + ch;

  // loads first: this lane's channel, and two channels per lane for the
  // group's largest |x|
  uint32_t xc[NB], xm[NB], lc[NB], lm2[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    xc[t] = x[(size_t)t * K + k];
    lc[t] = (fused ? (const uint8_t*)x : lm)[(size_t)t * K + k];   // ignored when graded here
    xm[t] = *(const uint32_t*)(x + (size_t)t * K + k0 + 2 * lane);
    lm2[t] = *(const uint16_t*)((fused ? (const uint8_t*)x : lm) + (size_t)t * K + k0 + 2 * lane);
  }
  // while x is on its way: the launch's scalars, empty lists (offsets outside
  // the resource: zeros without a memory access), zero digits
  const int N = A.N, T = 1 << A.log2_T, RB = A.RB, n_top = A.n_top, bmax = A.bmax, n_cut = A.n_cut;
  const uint64_t planes = A.planes;
  asm volatile("" ::"s"(N), "s"(T), "s"(RB), "s"(n_top), "s"(planes), "s"(bmax), "s"(n_cut), "s"(A.sfac),
               "s"(A.theta[0]), "s"(A.theta[1]), "s"(A.theta[2]), "s"(A.theta[3]));
  for (int i = tid; i < COLS * COLB / 16; i += kMmThreads) *(uint4*)&s_b[16 * i] = make_uint4(0u, 0u, 0u, 0u);
  if (tid < 4 * 16 * MAXB * 2 / 16) *(uint4*)((uint8_t*)&s_list[0][0][0] + 16 * tid) = make_uint4(~0u, ~0u, ~0u, ~0u);
  lds_barrier();

  topksel::Scratch& s_tk = *reinterpret_cast<topksel::Scratch*>(s_w);
  if constexpr (TOPK) topksel::select_cuts<kMmThreads>(x, K, tk, s_tk);

  // ---- grade: depths (planes to read) per token; the deepest decides the rows
  int d[NB], du = 0;
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const float ax = fabsf(h2f((uint16_t)xc[t]));
    int graded = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) graded += ax >= A.theta[j] ? 1 : 0;
    if (n_cut > 4) {
#pragma unroll
      for (int j = 4; j < kMaxLevels - 1; ++j) graded += ax >= A.theta[j] ? 1 : 0;
    }
    const int lvl = min(fused == 1 ? graded
                        : TOPK ? topksel::level_of(xc[t], k, tk.n, s_tk) : (int)lc[t], n_top);
    if (fused && lm_out && blockIdx.x == 0 && sub == 0 && half == 0) lm_out[(size_t)t * K + k] = (uint8_t)lvl;
    d[t] = level_planes(planes, lvl);
    du = max(du, d[t]);
  }
  // ---- list: the channel's first row is the number of rows of the lower ones
  int slot0 = 0, nrow = 0;
#pragma unroll
  for (int p = 0; p < PL; ++p) {
    const uint32_t b = (uint32_t)__ballot(du > p);   // the lower half's 32 channels
    slot0 += __popc(b & ((1u << (lane & 31)) - 1u));
    nrow += __popc(b);
  }
  const int nblk = __builtin_amdgcn_readfirstlane((nrow + 15) >> 4);
  {
    const uint32_t row = (uint32_t)(ch * RB) >> 6, pstep = (uint32_t)(T * U / 8) >> 6;
#pragma unroll
    for (int j = 0; j < PL / 2; ++j) {
      const int p = 2 * j + half, sl = slot0 + p;
      if (p < du) s_list[list][sl & 15][sl >> 4] = (uint16_t)(row + p * pstep);
    }
  }
  wave_lds_order();

  // ---- copies: lane = (row, chunk); chunk c of LDS row r holds chunk c ^ (r
  // mod CHK) of the plane row, so that the transposed reads below spread over
  // the banks.  128-byte rows: the two waves of a list copy half a block each;
  // 64-byte rows: they take the blocks in turn.
  constexpr bool HALVES = CHK == 8;
  constexpr int MINE = HALVES ? MAXB : MAXB / 2;   // copies of this wave at most
  const int crow = (HALVES ? 8 * sub : 0) + lane / CHK;
  uint32_t ent[MAXB / 2];                  // the row's offsets in the list's blocks, two per dword
  __builtin_memcpy(ent, &s_list[list][crow][0], MAXB * 2);
  uint32_t voff[MINE];
#pragma unroll
  for (int i = 0; i < MINE; ++i) {
    const uint32_t e = HALVES ? (i & 1 ? ent[i / 2] >> 16 : ent[i / 2] & 0xFFFFu)
                              : (sub ? ent[i] >> 16 : ent[i] & 0xFFFFu);
    voff[i] = (e << 6) + (uint32_t)((lane % CHK) ^ (crow & (CHK - 1))) * 16u;
  }
  const int c0 = blockIdx.x * run, ncol = min(run, cols - c0);
  // this wave's blocks that wait for the second half of a column
  const int late = min(nblk, SCAP) - FIRST;
  const int nlate = late <= 0 ? 0 : HALVES ? late : (late + ((FIRST ^ sub) & 1 ? 0 : 1)) / 2;
  auto copies = [&](int col, int pass) __attribute__((always_inline)) {
    const int n0 = (c0 + col) * W, tile = n0 >> A.log2_T, ob = (n0 & (T - 1)) * U / 8;
    if (wave == 0 && pass == 0) {
      const uint64_t sb = (uint64_t)(scales + (size_t)blockIdx.y * N + n0);
      const v4i srsrc = {__builtin_amdgcn_readfirstlane((int)(uint32_t)sb),
                         __builtin_amdgcn_readfirstlane((int)(uint32_t)(sb >> 32)), 2 * W, 0x00020000};
      // (32 lanes' worth for 256 outputs; the others are outside: zeros past it)
      if (W == 512 || lane < 32) copy_to_lds(lds_addr(s_scale), 16u * lane, srsrc);
    }
    const uint64_t base = (uint64_t)(codes + ((size_t)tile * K + k0) * RB + ob);
    // the group's rows from the column on; word 3: 32-bit data format, no
    // swizzle, no stride
    const v4i rsrc = {__builtin_amdgcn_readfirstlane((int)(uint32_t)base),
                      __builtin_amdgcn_readfirstlane((int)(uint32_t)(base >> 32)), kGroup * RB - ob, 0x00020000};
    const uint32_t dst = lds_addr(s_w) + (uint32_t)(list * SCAP * BLKB + (HALVES ? sub * 1024 : 0));
#pragma unroll
    for (int i = 0; i < MINE; ++i) {
      const int b = HALVES ? i : 2 * i + sub;
      if (b >= nblk) break;
      if ((b >= SCAP) == (pass != 0)) copy_to_lds(dst + (uint32_t)((b - (pass ? SCAP : 0)) * BLKB), voff[i], rsrc);
    }
  };
  // x has landed before the copies go out: a later wait for it would wait for
  // the copies too, which the compiler does not count
#pragma unroll
  for (int t = 0; t < NB; ++t) asm volatile("" ::"v"(xm[t]), "v"(lm2[t]));
  if constexpr (TOPK) lds_barrier();       // the selection's scratch is read everywhere
  copies(0, 0);

  // ---- the B operand, while the copies are in flight
  constexpr int FIX = U == 2 ? 38 : 37;    // X = rne(x 2^(FIX - e)), |x| < 2^(e - 14)
  uint32_t e_max[NB];
  float rest[NB], most = 0.0f;             // what X leaves of the channel's x, in units of X
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const uint32_t a = xm[t] & 0x7FFF7FFFu;
    // the largest finite |x| of an active channel (graded here, a skipped
    // channel is smaller than any active one; a level map may skip any)
    uint32_t lo = a & 0xFFFFu, hi = a >> 16;
    if (lo >= 0x7C00u || (!fused && (lm2[t] & 0xFFu) == 0)) lo = 0;
    if (hi >= 0x7C00u || (!fused && (lm2[t] >> 8) == 0)) hi = 0;
    const uint32_t mx = wave_max(lo > hi ? lo : hi);
    e_max[t] = mx >> 10 ? mx >> 10 : 1u;
    const float to_fix = __builtin_bit_cast(float, (127u + FIX - e_max[t]) << 23);
    const float fx = h2f((uint16_t)xc[t]);
    const float Xf = rintf(fx * to_fix);
    const int X = cvt_i32(Xf);
    // the list's half waves take its planes in turn
#pragma unroll
    for (int j = 0; j < (PL + 3) / 4; ++j) {
      const int p = 4 * j + 2 * half + sub;
      if (p < du) {
        const uint32_t V = p < d[t] ? (uint32_t)X << (U == 2 ? 6 - 2 * p : 7 - p) : 0u;
        const uint32_t dg = (V + 0x00808080u) ^ 0x00808080u;   // balanced digits, lowest first
        // byte of row sl of a block: the masks below give a dword the even or
        // the odd rows of eight
        const int sl = slot0 + p;
        const int pos = ((sl & ~15) << 2) + (sl & 8) + ((sl & 1) << 2) + ((sl >> 1) & 3);
        store_digits<COLB>(lds_addr(s_b) + (uint32_t)(4 * t * COLB + 16 * list + pos), dg);
      }
    }
    if (sub == 0) {
      // fx * 0 carries an infinite or NaN x of an active channel into every output
      const float phi = phi_minus_offset(U * d[t], bmax);
      const float unfix = __builtin_bit_cast(float, (127u - FIX + e_max[t]) << 23);
      const float beta = half_sum_dpp(d[t] ? fmaf(Xf * unfix, phi, fx * 0.0f) : 0.0f);
      if (lane == 0) s_beta[t][list] = beta;
      rest[t] = d[t] ? fabsf(fx * to_fix - Xf) : 0.0f;
      most = fmaxf(most, rest[t]);
    }
  }

  if (sub == 0) {
    float left[NB];
    bool much = false;                     // the four lists can be past kRestMax together
#pragma unroll
    for (int t = 0; t < NB; ++t) left[t] = 0.0f;
    if (__builtin_expect(__ballot(most > kRestList / 32) != 0, 0)) {
      bool some = false;
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        left[t] = half_sum_dpp(rest[t]);
        some |= left[t] > kRestList;
        much |= left[t] > kRestMax / 4;
      }
      if (__ballot(some) != 0) {
#pragma unroll
        for (int t = 0; t < NB; ++t)
#pragma unroll
          for (int p = 0; p < PL; ++p) {
            const uint32_t deeper = (uint32_t)__ballot(d[t] > p);
            if (lane == 0) s_deeper[t][list][p] = deeper;
          }
      }
    }
    if (lane == 0) {
      __builtin_memcpy(&s_b[list * COLB + S::LEFT], left, sizeof(left));
      s_nblk[list] = nblk | (much ? kMuchLeft : 0);
    }
  }

  // ---- the columns
  const int i16 = lane & 15, h = lane >> 4;
  const uint8_t* bcol = &s_b[min(i16, COLS - 1) * COLB + h * 16];   // spare columns repeat the last
  uint32_t wcol[NCB];                      // in a buffer
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const int byte = wave * (PBY / 8) + 8 * cb;
    wcol[cb] = (uint32_t)(h * SCAP * BLKB + i16 * PBY +
                          (((byte >> 4) ^ (i16 & (CHK - 1))) << 4) + (byte & 8));
  }
  const int o = lane % OW;                 // the output this lane adds (32 per wave: two lanes each)
  const int rcb = o / (16 * NSL), ri = (o / NSL) % 16, re = o % NSL;
  const float s_e = __builtin_bit_cast(float, (uint32_t)(127 - re * U) << 23);   // 2^(-e U)

  int rests = 0;
  for (int col = 0; col < ncol; ++col) {
    // the first blocks of every list (behind the copies: the last column's adds,
    // one instruction per token; no wave skips one, half its lanes take part at least)
    wait_copies(nlate + (col ? NB : 0));
    lds_barrier();
    const int4 nb4 = *(const int4*)&s_nblk[0];
    const int steps = __builtin_amdgcn_readfirstlane(
        max(max(nb4.x & (kMuchLeft - 1), nb4.y & (kMuchLeft - 1)), max(nb4.z & (kMuchLeft - 1), nb4.w & (kMuchLeft - 1))));
    rests = __builtin_amdgcn_readfirstlane(nb4.x | nb4.y | nb4.z | nb4.w) & kMuchLeft;
    v4i acc[NCB][NSL];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int e = 0; e < NSL; ++e) acc[cb][e] = v4i{0, 0, 0, 0};
    // a step's operands are read while the one before is multiplied
    struct Ops {
      v4i b;
      v2i w[NCB];
    };
    auto read_ops = [&](Ops& q, int s) __attribute__((always_inline)) {
      q.b = *(const v4i*)(bcol + 64 * s);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
        q.w[cb] = __builtin_amdgcn_ds_read_tr4_b64_v2i32(
            (__attribute__((address_space(3))) v2i*)((const lds_u8*)s_w + wcol[cb] + (s % SCAP) * BLKB));
      __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](const Ops& q) __attribute__((always_inline)) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const int w0 = q.w[cb].x, w1 = q.w[cb].y;
        const int w0h = (int)((uint32_t)w0 >> 4), w1h = (int)((uint32_t)w1 >> 4);
#pragma unroll
        for (int e = 0; e < NSL; ++e) {
          const int m = (((1 << U) - 1) << (e * U)) * 0x01010101;
          const v4i af = {w0 & m, w0h & m, w1 & m, w1h & m};
          acc[cb][e] = __builtin_amdgcn_mfma_i32_16x16x64_i8(af, q.b, acc[cb][e], 0, 0, 0);
        }
      }
    };
    Ops q[2];
    read_ops(q[0], 0);
#pragma unroll
    for (int s = 0; s < MAXB; ++s) {       // (a column without rows: one step of zero digits)
      const bool more = s + 1 < steps;
      const bool meet = s + 1 == FIRST || s + 1 == SCAP;
      if (s + 1 < MAXB && !meet && more) read_ops(q[(s + 1) & 1], s + 1);
      multiply(q[s & 1]);
      if (!more) break;
      if (meet) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
        if (s + 1 == FIRST && steps > SCAP) copies(col, 1);
        read_ops(q[(s + 1) & 1], s + 1);
      }
    }
    lds_barrier();                         // every wave has read the column: its place is free
    // the digits: a lane holds rows 4h .. 4h+3 (nibble columns) of B column
    // i16; through LDS to one lane per output
    int* red = (int*)s_w + wave * COLS * OWP;
    if (i16 < COLS) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int e = 0; e < NSL; ++e) *(v4i*)&red[i16 * OWP + (cb * NSL + e) * 16 + 4 * h] = acc[cb][e];
    }
    wave_lds_order();
    float v[NB];
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const int* src = red + 4 * t * OWP + (rcb * NSL + re) * 16 + ri;
      // |a| < 2^21: the pairs are exact in int32
      v[t] = fmaf((float)(src[3 * OWP] * 256 + src[2 * OWP]), 65536.0f, (float)(src[OWP] * 256 + src[0]));
    }
    const float s_n = h2f(s_scale[wave * OW + o]) * A.sfac;     // 8-bit units -> b_max units
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      const float unfix = __builtin_bit_cast(float, (127u - FIX + e_max[t]) << 23);
      const float4 b4 = *(const float4*)&s_beta[t][0];
      v[t] = s_n * fmaf(v[t], unfix * s_e, (b4.x + b4.y) + (b4.z + b4.w));
    }
    if (col + 1 < ncol) {
      lds_barrier();                       // the digit sums and the scales are read
      copies(col + 1, 0);
    }
    float* yo = y + (size_t)(c0 + col) * W + wave * OW + o;
#pragma unroll
    for (int t = 0; t < NB; ++t)
      if (OW == 64 || (t & 1) == half) add_to(yo + (size_t)t * N, v[t]);   // (two lanes take the tokens in turn)
  }

  // ---- groups whose x is not exact enough
  if (__builtin_expect(rests != 0, 0)) {
    float worst = 0.0f;                    // (a token with an active infinity or NaN: NaN, left out)
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      float lost = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) lost += *(const float*)&s_b[j * COLB + S::LEFT + 4 * t];
      worst = fmaxf(worst, lost);
    }
    if (!(worst > kRestMax)) return;
    lds_barrier();                         // the digit sums are read: their place is free
#pragma unroll 1
    for (int i = 0; i < ncol * NB; ++i) {
      const int t = i % NB, n0 = (c0 + i / NB) * W, tile = n0 >> A.log2_T, ob = (n0 & (T - 1)) * U / 8;
      uint32_t e = e_max[0];
#pragma unroll
      for (int j = 1; j < NB; ++j) e = t == j ? e_max[j] : e;
      add_rests<U, W, PL>(x + (size_t)t * K + k0, codes + ((size_t)tile * K + k0) * RB + ob,
                          scales + (size_t)blockIdx.y * N + n0, y + (size_t)t * N + n0, &s_deeper[t][0][0],
                          (const float*)&s_b[S::LEFT + 4 * t], COLB / 4, (float*)s_w, __builtin_bit_cast(float, (127u + FIX - e) << 23),
                          __builtin_bit_cast(float, (127u - FIX + e) << 23) * A.sfac, RB, T * U / 8, bmax);
    }
  }
}

template <int U, int W, int PL>
void launch_nb(int B, hipStream_t s, const void* codes, const void* scales, const void* x,
               const uint8_t* lm, float* y, const Layer& L, int fused, const Thresholds& th,
               const TopkCuts& tk, uint8_t* lm_out) {
  MmArgs A{};
  A.N = L.N;
  A.log2_T = __builtin_ctz((unsigned)L.T);
  A.RB = L.RB;
  A.n_top = L.n_levels - 1;
  A.planes = L.planes_packed;
  A.bmax = L.bmax;
  A.n_cut = th.n;
  A.sfac = L.sfac;
  for (int j = 0; j < kMaxLevels - 1; ++j) A.theta[j] = th.theta[j];
  // Columns per workgroup: for one token the fewest that leave at most three
  // workgroups per CU (a further round of workgroups would start with the
  // latency of x again); for several, one (their digit sums weigh more).
  const int cols = L.N / W, cus = device_cus();
  int run = 1;
  while (B == 1 && run < cols && (long)((cols + run - 1) / run) * L.groups > 3 * cus) ++run;
  const dim3 grid((unsigned)((cols + run - 1) / run), (unsigned)L.groups);
  // Longer runs that leave only two workgroups per CU have the LDS for every
  // step of a column: no second pass at 6 and 8 bits (us at 4 / 6 / 8 bits, three workgroups' LDS
  // and two's: 14336 -> 4096 9.9 / 13.3 / 14.3 and 9.9 / 11.7 / 13.5, 4096 -> 16384 10.2 / 14.0 / 16.7 and
  // 10.0 / 12.2 / 15.3, 1-bit planes at 8 bits 20.9 and 17.3).  Not for one column, whose second
  // pass comes while other workgroups of the CU multiply: 4096 -> 6144 at 8 bits 8.2 and 8.4, with 1-bit planes 9.9
  // and 10.3; nor in place of a third workgroup: 8192 -> 10240 at 4 bits 12.5 and 14.5.
  constexpr bool kSplit = MmShape<U, W, PL, 1, false>::SCAP < MmShape<U, W, PL, 1, false>::MAXB;
  const bool full = kSplit && run > 1 && (long)grid.x * grid.y <= 2 * cus;
#define GRINQH_MM(NN, FF, TK)                                                                    \
  hipLaunchKernelGGL((k_vmm_mm<U, W, PL, NN, FF, TK>), grid, dim3(kMmThreads), 0, s, (const uint16_t*)x, lm, \
                     L.K, fused, run, cols, (const uint8_t*)codes, (const uint16_t*)scales, y, lm_out, A, tk)
  if (fused == 2) {
    if constexpr (U == 2) {
      if (full) GRINQH_MM(1, kSplit, true);
      else GRINQH_MM(1, false, true);
    }
  } else if (B == 1) {
    if (full) GRINQH_MM(1, kSplit, false);
    else GRINQH_MM(1, false, false);
  } else if (B == 2) {
    GRINQH_MM(2, false, false);
  } else if (B == 3) {
    GRINQH_MM(3, false, false);
  } else {
    GRINQH_MM(4, false, false);
  }
#undef GRINQH_MM
}

}  // namespace

int launch_vmm_mm(const Layer& L, const void* codes, const void* scales, const void* x,
                  const uint8_t* level_map, const Thresholds* th, const TopkCuts* tk,
                  uint8_t* level_map_out, int B, float* y, hipStream_t s) {
  Thresholds none{};
  TopkCuts nocuts{};
  const int fused = th ? 1 : (tk ? 2 : 0);   // levels graded here: thresholds, top-k
  const Thresholds& tt = th ? *th : none;
  const TopkCuts& cc = tk ? *tk : nocuts;
#define GRINQH_MM(UU, WW, PP) \
  launch_nb<UU, WW, PP>(B, s, codes, scales, x, level_map, y, L, fused, tt, cc, level_map_out)
  if (L.u == 2) {
    if (L.T == 256) {
      if (L.P <= 2) GRINQH_MM(2, 256, 2);
      else GRINQH_MM(2, 256, 4);
    } else {
      if (L.P <= 2) GRINQH_MM(2, 512, 2);
      else GRINQH_MM(2, 512, 4);
    }
  } else {
    if (L.P <= 4) GRINQH_MM(1, 512, 4);
    else GRINQH_MM(1, 512, 8);
  }
#undef GRINQH_MM
  return check_launch("vmm");
}

}  // namespace grinqh
