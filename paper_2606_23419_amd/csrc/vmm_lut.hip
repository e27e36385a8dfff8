// Nested-precision decode VMM over non-uniform nested weights read through
// per-output look-up tables (Sec. 3.3: the format needs only the nested
// property, which k-means-style nested weights have; their levels are
// centred, so no midpoint bias is applied).  The codes use the packed
// layout of the uniform path; a channel at width b reads its first b/u
// planes, forms the b leading bits q_b of every output's code, and adds
// x_k * table_b[n][q_b].
//
// A workgroup owns 64 outputs of one tile (a sub-tile), a run of groups and
// one token.  It lists the run's active channels sorted by level, and copies
// to LDS the tables of its 64 outputs for the levels the run uses: for each
// level they are one contiguous block of the table array.
// 4 lanes cover a channel row's 64 outputs (16 each); a wave takes 16 rows of
// the list at once.  Every weight is one LDS lookup.  Lanes holding the same
// outputs are summed in registers, waves through LDS, and the sums added into
// y with atomics.
//
// What bounds it: the lookups (one LDS read, one address and one FMA per
// weight) and, on runs of few groups, the latencies of staging, the table
// copy and the final sums.  The list leaves out level-0 channels (20..35% of
// a row's slots at the paper's budgets, which idled before) and makes the
// level the same in all lanes of a wave but at the list's level borders, so
// a table's place in LDS is an immediate and the code's byte one operand.
// The run's x and levels are loaded at once, a compile-time number per thread:
// loads under conditions were waited for one by one, up to eight latencies.
// Measured (us a call, levels {0,2,4,6,8} at 4 average bits; without the list /
// with it, the tables copied by LDS loads and the sums in registers / with the
// loads at once): 4096 -> 6144 19.3 / 14.8 / 13.7, 4096 -> 4096 15.1 / 11.6 / 10.8,
// 4096 -> 28672 60.3 / 53.4 / 49.3, 14336 -> 4096 33.6 / 31.1 / 30.5, 1024 -> 1024 11.0 / 6.9 /
// 6.3.  Where every channel is at 8 bits nothing is left out and the lookups' bank
// conflicts (random 512-byte tables) bound it: 4096 -> 6144 22.0 / 22.6 / 22.0, 14336 ->
// 4096 51.9 / 49.1 / 48.6.  Several tokens, without the list / with it, a token's workgroups
// apart / tokens side by side: two of 1536 -> 10240 at 8 bits 23.5 / 25.8 / 21.9, of 1024 -> 28672
// 39.0 / 42.3 / 36.3, four of 4096 -> 28672 306 / 305 / 197 and at 4 bits 171 / 174 / 145.
#include <algorithm>
#include <type_traits>

#include "grinqh_internal.h"
#include "vmm_common.h"

namespace grinqh {

namespace {

constexpr int kLutThreads = 256;
constexpr int kStep = kLutThreads / 4;       // channel rows the workgroup looks up at once
constexpr int kSub = 64;                     // outputs per workgroup
constexpr int kMaxRun = 16 * 128;            // channels per workgroup (16 groups)
static_assert(kMaxRun == 8 * kLutThreads, "the longest run's channels per thread");

__global__ __launch_bounds__(kLutThreads) void k_zero_lut(float* __restrict__ y, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = 0.0f;
}

// a's sum over the two halves (W = 32) or the two 16-lane rows of a half
// (W = 16) in the lower of them, b's in the upper.
template <int W>
__device__ __forceinline__ float swap_add(float a, float b) {
  uint32_t u = __builtin_bit_cast(uint32_t, a), v = __builtin_bit_cast(uint32_t, b);
  if constexpr (W == 32)
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(u), "+v"(v));
  else
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(u), "+v"(v));
  return __builtin_bit_cast(float, u) + __builtin_bit_cast(float, v);
}

// MINE: channels per thread, kLutThreads MINE the longest run.
template <int U, int MINE>
__global__ __launch_bounds__(kLutThreads) void k_vmm_lut(const uint8_t* __restrict__ codes,
                                                        const uint16_t* __restrict__ luts,
                                                        const uint16_t* __restrict__ x,
                                                        const uint8_t* __restrict__ lm,
                                                        float* __restrict__ y, Layer L, LutDesc D,
                                                        int groups_per_split, int splits, int inner, int B, int fused,
                                                        Thresholds th, uint8_t* __restrict__ lm_out) {
  extern __shared__ __align__(16) uint16_t s_lut[];          // [levels][kSub][2^b]
  __shared__ float s_red[kLutThreads / 64][kSub];
  __shared__ uint32_t s_ent[MINE * kLutThreads];              // active channels: x | row << 16 | level << 27
  __shared__ __align__(16) int s_cnt[kMaxLevels][kLutThreads / 64];         // channels of a level in a wave's share

  // Work order: consecutive work items run on one XCD (workgroup id mod 8 picks
  // the XCD), so that its L2 serves what they share.  One token: the K splits of
  // a sub-tile (its tables), then the sub-tiles of a tile (128-byte plane lines).
  // Several: up to eight tokens, the sub-tiles of a tile, its splits, as the tokens
  // share every plane line: with a token's workgroups apart from the next's
  // each token fetched the codes again, 423 MB of 59 for eight tokens of 4096 ->
  // 28672 at 4 bits of 4, 289 us; now 164.
  const int sub_bits = __builtin_ctz((unsigned)L.T) - 6, subs = 1 << sub_bits;
  static_assert(kSub == 64, "sub_bits");
  const int nwg = gridDim.x;
  const int item = (nwg % 8 == 0) ? (int)(blockIdx.x % 8) * (nwg / 8) + (int)(blockIdx.x / 8)
                                  : (int)blockIdx.x;
  int t, sub, split, tok = 0;
  if (inner == 1) {
    const int tile_sub = item / splits;
    split = item - tile_sub * splits;
    t = tile_sub >> sub_bits;
    sub = tile_sub & (subs - 1);
    tok = blockIdx.y;
  } else {
    const int of_tok = item / inner;
    t = of_tok / (splits << sub_bits);
    const int in_tile = of_tok - t * (splits << sub_bits);
    split = in_tile >> sub_bits;
    sub = in_tile & (subs - 1);
    tok = (int)blockIdx.y * inner + item - of_tok * inner;
    if (tok >= B) return;
  }
  const int n0 = t * L.T + sub * kSub;       // first output of the sub-tile
  const int g0 = split * groups_per_split;
  const int g1 = min(g0 + groups_per_split, L.groups);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rs = lane >> 2;                  // row of the wave's 16

  // LDS layout: level l's block starts at kSub * cum[l] + 4 pad (l - 1)
  // entries and holds the 64 outputs' tables as four quads of 16 outputs,
  // quad c at c (16 * 2^b + pad): the pad of 16 entries (8 banks) puts the
  // four quads a wave reads in one step on different banks (unpadded their
  // starts are 128-byte multiples apart, the same banks for every b >= 2)
  const int pad = D.quad_pad;
  // cum[l] in byte l - 1: widths are distinct and ascending, so cum[l] < 2^b_l <= 256
  uint64_t cum_packed = 0;
#pragma unroll
  for (int l = 1; l < kMaxLevels; ++l) cum_packed |= (uint64_t)(D.cum[l] & 0xFF) << (8 * (l - 1));
  const int c = tid & 3;                     // outputs 16 c .. 16 c + 15 of the sub-tile
  const int plane_bytes = L.T * U / 8;
  const int col = (sub * kSub + 16 * c) * U / 8;   // byte of the lane's outputs in a plane row
  const int n_top = L.n_levels - 1;
  const int kr0 = g0 * kGroup, nrows = (g1 - g0) * kGroup;   // the workgroup's channels

  // Levels of the run's channels (<= kMaxRun), read from the level map, or
  // graded here from |x| against the thresholds (Sec. 3.1; th.n is 0 without
  // them), the level map then written out once (by the workgroups of tile 0,
  // sub-tile 0).  Then the active channels are listed by level: a wave ranks
  // its own channels of each level by ballot, and one exchange of the waves'
  // counts gives every level and wave its place.
  uint32_t ent[MINE];
  int rank[MINE];
  int cnt[kMaxLevels];
#pragma unroll
  for (int l = 0; l < kMaxLevels; ++l) cnt[l] = 0;
  // all loads before the first use: none under a condition (past the run the
  // last channel again; without a level map x's bytes, unused)
  uint32_t xs[MINE], ls[MINE];
  const uint8_t* lmap = fused ? (const uint8_t*)x : lm;
#pragma unroll
  for (int m = 0; m < MINE; ++m) {
    const size_t k = (size_t)tok * L.K + kr0 + min(tid + m * kLutThreads, nrows - 1);
    xs[m] = x[k];
    ls[m] = lmap[k];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int m = 0; m < MINE; ++m) asm volatile("" : "+v"(xs[m]), "+v"(ls[m]));   // (the compiler sinks them otherwise)
#pragma unroll
  for (int m = 0; m < MINE; ++m) {
    const int i = tid + m * kLutThreads;
    ent[m] = 0;
    rank[m] = 0;
    int lv = 0;
    if (i < nrows) {
      const uint32_t xh = xs[m];
      if (fused) {
        const float ax = fabsf(h2f((uint16_t)xh));
#pragma unroll
        for (int j = 0; j < kMaxLevels - 1; ++j)   // unused thresholds are +inf: no
          lv += ax >= th.theta[j] ? 1 : 0;         // branch, all loaded up front
        lv = min(lv, n_top);
        if (lm_out && t == 0 && sub == 0) lm_out[(size_t)tok * L.K + kr0 + i] = (uint8_t)lv;
      } else {
        lv = min((int)ls[m], n_top);
      }
      ent[m] = xh | ((uint32_t)i << 16) | ((uint32_t)lv << 27);
    }
#pragma unroll
    for (int l = 1; l < kMaxLevels; ++l) {
      if (l > n_top) break;
      const uint64_t in = __ballot(lv == l);
      const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(in >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)in, 0u));
      rank[m] = lv == l ? cnt[l] + below : rank[m];
      cnt[l] += (int)__popcll(in);
    }
  }
#pragma unroll
  for (int l = 1; l < kMaxLevels; ++l)
    if (lane == 0) s_cnt[l][wave] = cnt[l];
  __syncthreads();
  int per_wave[kMaxLevels][kLutThreads / 64];    // read at once: one LDS latency
#pragma unroll
  for (int l = 1; l < kMaxLevels; ++l)
#pragma unroll
    for (int w = 0; w < kLutThreads / 64; ++w) per_wave[l][w] = s_cnt[l][w];
  __builtin_amdgcn_sched_barrier(0);
  int n_ent = 0;
  uint32_t used_levels = 0;   // bit l: only the tables of levels in use are copied (at
                              // the paper's 4-bit budgets the 8-bit level, three quarters
                              // of the table bytes, is empty)
#pragma unroll
  for (int l = 1; l < kMaxLevels; ++l) {
    if (l > n_top) break;
    int mine = n_ent, all = 0;
#pragma unroll
    for (int w = 0; w < kLutThreads / 64; ++w) {
      const int v = __builtin_amdgcn_readfirstlane(per_wave[l][w]);
      mine += w < wave ? v : 0;
      all += v;
    }
#pragma unroll
    for (int m = 0; m < MINE; ++m)
      if ((int)(ent[m] >> 27) == l) s_ent[mine + rank[m]] = ent[m];
    n_ent += all;
    used_levels |= all ? 1u << l : 0u;
  }
  __syncthreads();

  float acc[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.0f;

  // Entries 16 wave + rs + kStep m, m = 0, 1, ..., through a ring of four register sets:
  // three rows' plane words are in flight while one row is looked up.  The
  // loads are unconditional (planes past a row's depth, and entries past the
  // list, load from no row and read zero without a memory access), so the
  // compiler counts them and waits for the row being consumed alone.
  constexpr int kWords = 8 / U;
  constexpr int R = 4;
  // 1-bit planes: the lane's two bytes are loaded as the aligned dword that
  // holds them and its half is kept when the row is consumed (plane rows and
  // sub-tiles start at multiples of four bytes)
  const uint32_t lane_off = (uint32_t)(U == 2 ? col : (col & ~3));
  const int half_sh = U == 2 ? 0 : (col & 2) * 8;
  const __amdgpu_buffer_rsrc_t rsrc = vmmdev::tile_rsrc(codes + (size_t)t * L.K * L.RB, L);
  auto fetch = [&](int i, uint32_t (&w)[kWords], uint32_t& en) __attribute__((always_inline)) {
    const uint32_t v = s_ent[max(min(i, n_ent - 1), 0)];
    en = i < n_ent ? v : 0u;                 // past the list: level 0, no planes
    const int d = level_planes(L.planes_packed, (int)(en >> 27));
    const uint32_t row = (uint32_t)(kr0 + (int)((en >> 16) & 0x7FFu)) * (uint32_t)L.RB + lane_off;
#pragma unroll
    for (int j = 0; j < kWords; ++j)
      w[j] = vmmdev::load_plane(rsrc, j < d ? row + (uint32_t)(j * plane_bytes) : vmmdev::kNoRow);
  };
  // the 16 outputs' codes left-aligned in 8 bits (planes past the depth were
  // loaded as zero): byte i of qw[r] is output 4 i + r; q_b is its top b bits
  auto codes16 = [&](const uint32_t (&wv)[kWords], uint32_t (&qw)[4]) __attribute__((always_inline)) {
    uint32_t w[4];
    if constexpr (U == 2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = wv[j];
    } else {
      uint32_t m[kWords];
#pragma unroll
      for (int j = 0; j < kWords; ++j) m[j] = (wv[j] >> half_sh) & 0xFFFFu;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        w[j] = (vmmdev::spread_bits(m[2 * j]) << 1) | vmmdev::spread_bits(m[2 * j + 1]);
    }
    vmmdev::assemble_codes(w[0], w[1], w[2], w[3], qw);
  };
  // one level in the whole wave: its width b is a constant of the code
  auto lookup = [&](auto width, int lvl, float xv, const uint32_t (&qw)[4]) __attribute__((always_inline)) {
    constexpr int b = decltype(width)::value;
    const uint8_t* tb = (const uint8_t*)(s_lut + kSub * (int)((cum_packed >> (8 * (lvl - 1))) & 0xFF) +
                                         4 * pad * (lvl - 1) + c * ((16 << b) + pad));
    uint32_t q2[4];                          // 2 q_b (its byte offset in a table), b < 8
    if constexpr (b < 8) {
      constexpr uint32_t keep = 0x01010101u * ((2u << b) - 2u);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        q2[r] = (qw[r] >> (7 - b)) & keep;
        asm("" : "+v"(q2[r]));               // kept as bytes: one byte-select add per weight
      }
    }
    uint16_t v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      uint32_t off;
      if constexpr (b < 8) off = (q2[e & 3] >> (8 * (e >> 2))) & 0xFFu;
      else off = ((qw[e & 3] >> (8 * (e >> 2))) & 0xFFu) << 1;
      v[e] = *(const uint16_t*)(tb + off + (e << (b + 1)));
    }
    __builtin_amdgcn_sched_barrier(0);       // all sixteen reads in flight
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = fmaf(xv, h2f(v[e]), acc[e]);
  };
  auto consume = [&](const uint32_t (&wv)[kWords], uint32_t en) __attribute__((always_inline)) {
    const int lvl = (int)(en >> 27);
    const int l0 = __builtin_amdgcn_readfirstlane(lvl);
    if (l0 == 0) return;                     // the list ended before this wave's rows
    const float xv = h2f((uint16_t)en);
    uint32_t qw[4];
    codes16(wv, qw);
    if (__ballot(lvl != l0) == 0) {
      const int d = level_planes(L.planes_packed, l0);
      if constexpr (U == 2) {
        if (d == 1) lookup(std::integral_constant<int, 2>{}, l0, xv, qw);
        else if (d == 2) lookup(std::integral_constant<int, 4>{}, l0, xv, qw);
        else if (d == 3) lookup(std::integral_constant<int, 6>{}, l0, xv, qw);
        else lookup(std::integral_constant<int, 8>{}, l0, xv, qw);
        return;
      } else {
        if (d == 2) return lookup(std::integral_constant<int, 2>{}, l0, xv, qw);
        if (d == 3) return lookup(std::integral_constant<int, 3>{}, l0, xv, qw);
        if (d == 4) return lookup(std::integral_constant<int, 4>{}, l0, xv, qw);
        if (d == 8) return lookup(std::integral_constant<int, 8>{}, l0, xv, qw);
      }
    }
    // rows at a border of two levels (or of the list), and widths without a
    // form of their own
    if (lvl != 0) {
      const int b = level_planes(L.planes_packed, lvl) * U;
      const int sh = 8 - b;
      const uint16_t* tb = s_lut + kSub * (int)((cum_packed >> (8 * (lvl - 1))) & 0xFF) + 4 * pad * (lvl - 1) +
                           c * ((16 << b) + pad);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const uint32_t q8 = (qw[e & 3] >> (8 * (e >> 2))) & 0xFFu;
        acc[e] = fmaf(xv, h2f(tb[(e << b) + (q8 >> sh)]), acc[e]);
      }
    }
  };
  uint32_t wr[R][kWords], en[R];
#pragma unroll
  for (int q = 0; q < R - 1; ++q) fetch(16 * wave + rs + kStep * q, wr[q], en[q]);
  __builtin_amdgcn_sched_barrier(0);   // the first rows' loads go out before the table copy
  // Tables of the 64 outputs: level l's are kSub * 2^b entries at D.offset[l] +
  // n0 * 2^b of the table array.  Each quad's 2^(b+1) pieces of 16 bytes go to
  // LDS without passing registers, up to 64 pieces an instruction, the pieces
  // beyond a small quad masked.  (Through registers, with the last piece
  // repeated so that nothing was conditional, a workgroup wrote 2048 pieces for
  // every level, 64 times the 2-bit tables.)
  for (int l = 1; l <= n_top; ++l) {
    if (!((used_levels >> l) & 1u)) continue;
    const int b = level_planes(L.planes_packed, l) * U;
    const int per = min(64, 2 << b), units = (8 << b) / per;
    const uint4* src = (const uint4*)(luts + D.offset[l] + ((size_t)n0 << b)) + lane;
    uint16_t* dst = s_lut + kSub * (int)((cum_packed >> (8 * (l - 1))) & 0xFF) + 4 * pad * (l - 1);
    for (int u = wave; u < units; u += kLutThreads / 64) {
      const int i = per * u;                 // first piece
      if (lane < per)
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(src + i),
            (__attribute__((address_space(3))) void*)(dst + (i >> (b + 1)) * pad + 8 * i), 16, 0, 0);
    }
  }
  // the copies have no register that a reader could wait for: every wave waits
  // for its own before the barrier that lets the others read them
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  for (int i = 16 * wave; i < n_ent; i += kStep * R) {
#pragma unroll
    for (int q = 0; q < R; ++q) {
      fetch(i + rs + kStep * (q + R - 1), wr[(q + R - 1) % R], en[(q + R - 1) % R]);
      consume(wr[q], en[q]);
    }
  }

  // Lanes with equal (lane & 3) hold the same outputs.  Over lane bits 5 and
  // 4 by exchanging halves of the sums: v_permlane32_swap / 16_swap of two
  // sums leaves one of them in each half, so 16 sums become 4 per lane, of
  // outputs 8 (lane bit 5) + 4 (lane bit 4) + e; then over bits 3 and 2 by
  // rotations.  32 register operations; as shuffles through LDS they were 64
  // LDS operations, half as many as the lookups of a run of four groups.
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = swap_add<32>(acc[e], acc[e + 8]);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    acc[e] = swap_add<16>(acc[e], acc[e + 4]);
    acc[e] += vmmdev::row_ror<8>(acc[e]);
    acc[e] += vmmdev::row_ror<4>(acc[e]);
  }
  if ((lane & 12) == 0) {
    const int o = 16 * c + 8 * (lane >> 5) + 4 * ((lane >> 4) & 1);
#pragma unroll
    for (int e = 0; e < 4; ++e) s_red[wave][o + e] = acc[e];
  }
  __syncthreads();
  if (tid < kSub) {
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < kLutThreads / 64; ++w) v += s_red[w][tid];
    atomicAdd(&y[(size_t)tok * L.N + n0 + tid], v);
  }
}

}  // namespace

int lut_desc(const Layer& L, LutDesc* D) {
  long off = 0;
  int cum = 0;
  for (int l = 0; l < kMaxLevels; ++l) {
    D->offset[l] = off;
    D->cum[l] = cum;
    if (l >= 1 && l < L.n_levels) {
      off += (long)L.N << L.bits[l];
      cum += 1 << L.bits[l];
    }
  }
  D->entries = cum;
  // quad padding in LDS when it fits in 64 KB (see the kernel)
  const size_t padded = (size_t)kSub * cum * 2 + (size_t)4 * 16 * (L.n_levels - 1) * 2;
  D->quad_pad = padded <= 65536 ? 16 : 0;
  return GRINQH_OK;
}

// Groups per workgroup g of a layer of `groups` groups and `columns`
// (sub-tile, token) pairs.  A workgroup costs its groups and about four more
// (listing, table copy, sums), a CU the n workgroups that fall to it, and the
// last one's length is added once, as nothing overlaps its end: n (g + 4) + g
// is within 1.5% of the best g in the mean of 90 shapes and budgets swept (22% off
// at worst, at 6 to 9 us).  Measured (us at 4 average bits, levels {0,2,4,6,8}):
// 4096 -> 6144 13.8 with g = 4, 16.4 with 8; 4096 -> 4096 10.8 with 4, 13.0 with 8, 14.9
// with 2; 14336 -> 4096 30.7 with 14 (two workgroups per CU), 33.4 with 16, 35.5 with
// 8; 1024 -> 1024 6.3 with 1, 8.7 with 4.  More than eight groups only where K is long
// (one token of 4096 -> 28672 49.3 with 8, 51.9 with 16), for several tokens too: they
// share tables and plane lines through L2, so longer runs don't save them (four of
// 4096 -> 4096 at 8 bits 33.5 with 8, 37.0 with 16).
static int groups_per_workgroup(int groups, long columns, int cus) {
  const int most = std::min(std::max(8, (groups + 3) / 4), std::min(groups, kMaxRun / kGroup));
  int best = 1;
  long best_cost = 0;
  for (int g = 1; g <= most; ++g) {
    const long splits = (groups + g - 1) / g;
    const long cost = (columns * splits + cus - 1) / cus * (g + 4) + g;
    if (g == 1 || cost < best_cost) {
      best = g;
      best_cost = cost;
    }
  }
  return best;
}

int launch_vmm_lut(const Layer& L, const void* codes, const void* luts, const void* x,
                   const uint8_t* level_map, const Thresholds* th, uint8_t* level_map_out, int B,
                   float* y, int accumulate, hipStream_t s) {
  LutDesc D;
  lut_desc(L, &D);
  // <= 64 * 510 * 2 bytes (levels are distinct widths <= 8), plus the quad padding where it fits
  const size_t lds = (size_t)kSub * D.entries * 2 + (size_t)4 * D.quad_pad * (L.n_levels - 1) * 2;
  if (lds > 65536) return fail(GRINQH_EUNSUPPORTED, "LUT VMM: %d table entries per output", D.entries);
  if (!accumulate) {
    const long n = (long)B * L.N;
    hipLaunchKernelGGL(k_zero_lut, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, y, n);
  }
  const long subtiles = (long)L.tiles * (L.T / kSub);
  int gps = groups_per_workgroup(L.groups, subtiles * B, device_cus());
  if (const int v = option(&Options::lut_groups)) gps = v <= L.groups ? v : L.groups;
  gps = gps > kMaxRun / kGroup ? kMaxRun / kGroup : gps;
  const long splits = (L.groups + gps - 1) / gps;
  const int rows = (B + 7) / 8, inner = (B + rows - 1) / rows;   // tokens side by side: up to 8
  const dim3 grid((unsigned)(subtiles * splits * inner), (unsigned)rows);
  Thresholds none{};
  const Thresholds& tt = th ? *th : none;
  const int fused = th != nullptr;
#define GRINQH_LUT(UU, MM)                                                                                    \
  hipLaunchKernelGGL((k_vmm_lut<UU, MM>), grid, dim3(kLutThreads), lds, s, (const uint8_t*)codes,              \
                     (const uint16_t*)luts, (const uint16_t*)x, level_map, y, L, D, gps, (int)splits, inner, B, fused, \
                     tt, level_map_out)
  const int run = gps * kGroup;
  if (L.u == 2) {
    if (run <= 2 * kLutThreads) GRINQH_LUT(2, 2);
    else if (run <= 4 * kLutThreads) GRINQH_LUT(2, 4);
    else GRINQH_LUT(2, 8);
  } else {
    if (run <= 2 * kLutThreads) GRINQH_LUT(1, 2);
    else if (run <= 4 * kLutThreads) GRINQH_LUT(1, 4);
    else GRINQH_LUT(1, 8);
  }
#undef GRINQH_LUT
  return check_launch("vmm_lut");
}

}  // namespace grinqh
