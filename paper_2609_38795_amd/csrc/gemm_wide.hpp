// The GEMM of the large products: C[M,N] = A[M,K] * W[N,K]^T, bf16, one
// 256x256 tile at a time per CU, with the K loop scheduled by hand (gfx950).
//
// What bounds it: power, then the matrix pipes.  Under sustained MFMA work the
// board holds 1.3-1.7 GHz, so what counts besides keeping the pipes fed is the
// energy spent around them:
//   * four waves of 128x128 (one per SIMD) read 128 KB of operands from LDS per
//     K step of 64, eight waves of 128x64 read 192 KB;
//   * operands go from global memory straight into LDS (copy_1k), not through
//     registers;
//   * 16x16x32 MFMAs read and write half the accumulator data of 32x32x16 ones.
// A wave alone on its SIMD has nothing to cover its waits, so every LDS read is
// issued half a step (64 MFMAs, 1024 cycles) before its use and every copy a
// step and a quarter before; a compiler schedules neither with 256 accumulators
// live (its best was 1063 TFLOP/s), so the whole K loop is one asm block with
// its own registers.  Gate/up of the prefill (32768 x 28672 x 4096) alone:
// 5.82 -> 4.84 ms (1322 -> 1591 TFLOP/s) against the eight-wave ping-pong kernel it
// replaced, which staged its operands through registers; in the model 5.88 -> 4.99.
//
// Accumulators: tile (i, j) of 16x16 is a[4 (8 i + j) .. + 3].  Lane l of it holds
// rows 16 i + 4 (l / 16) + e, e = 0..3, of column 16 j + l % 16.
// Fragments: set F = k half of a step; A block i is v[128 + 64 F + 4 i ..], W block
// j v[160 + 64 F + 4 j ..]; lane l holds row l % 16, k = 8 (l / 16) .. + 7.
// v96-v103 / v104-v111: byte offsets of the lane's part of the wave's eight
// copies of an A / W tile; v112, v113 / v114, v115: LDS read addresses of the A / W
// fragments per k half.  s[40:41], s[42:43]: A and W at the K step to be copied.
#pragma once

#include "gemm_kernels.hpp"

namespace alr {

#define ALR_ACC(i, j) "a[4*(8*" #i "+" #j "):4*(8*" #i "+" #j ")+3]"
#define ALR_FA(F, i) "v[128+64*" #F "+4*" #i ":128+64*" #F "+4*" #i "+3]"
#define ALR_FB(F, j) "v[160+64*" #F "+4*" #j ":160+64*" #F "+4*" #j "+3]"
#define ALR_MF(F, i, j) \
  "v_mfma_f32_16x16x32_bf16 " ALR_ACC(i, j) ", " ALR_FA(F, i) ", " ALR_FB(F, j) ", " ALR_ACC(i, j) "\n\t"
#define ALR_MZ(F, i, j) \
  "v_mfma_f32_16x16x32_bf16 " ALR_ACC(i, j) ", " ALR_FA(F, i) ", " ALR_FB(F, j) ", 0\n\t"
// LDS reads of block i (16 rows, 2 KB apart); copies of 32-row pieces of the A and W
// tiles.  M0 holds the LDS address of the copy, and one instruction has to stand between
// its write and the copy that reads it: ALR_REFILL sets it two MFMAs before the first
// copy, and each copy is followed by the write for the next (the last A copy's for W).
#define ALR_RA(F, i) "ds_read_b128 " ALR_FA(F, i) ", v[112+" #F "] offset:2048*" #i "\n\t"
#define ALR_RB(F, j) "ds_read_b128 " ALR_FB(F, j) ", v[114+" #F "] offset:2048*" #j "\n\t"
#define ALR_CA(j) "global_load_lds_dwordx4 v[96+" #j "], s[40:41]\n\ts_add_u32 m0, %[lds], 4096+4096*" #j "\n\t"
#define ALR_CW(j) "global_load_lds_dwordx4 v[104+" #j "], s[42:43]\n\ts_add_u32 m0, %[lds], 36864+4096*" #j "\n\t"
// One k half: 64 MFMAs in rows of eight (every other row backwards, so that
// neighbours share an operand), with a slot for other work after every second.
#define ALR_ROW_F(M, F, i, a, b, c, d) M(F, i, 0) M(F, i, 1) a M(F, i, 2) M(F, i, 3) b \
  M(F, i, 4) M(F, i, 5) c M(F, i, 6) M(F, i, 7) d
#define ALR_ROW_B(M, F, i, a, b, c, d) M(F, i, 7) M(F, i, 6) a M(F, i, 5) M(F, i, 4) b \
  M(F, i, 3) M(F, i, 2) c M(F, i, 1) M(F, i, 0) d
// half 0 of a step: the reads of its half 1 in the first half of the slots; then
// every wave has read the whole stage (FREE) and its refill begins (C0 .. C7)
#define ALR_HALF0(M, FREE, C0, C1, C2, C3, C4, C5, C6, C7) \
  ALR_ROW_F(M, 0, 0, ALR_RA(1, 0), ALR_RB(1, 0), ALR_RB(1, 1), ALR_RB(1, 2)) \
  ALR_ROW_B(M, 0, 1, ALR_RB(1, 3), ALR_RB(1, 4), ALR_RB(1, 5), ALR_RB(1, 6)) \
  ALR_ROW_F(M, 0, 2, ALR_RB(1, 7), ALR_RA(1, 1), ALR_RA(1, 2), ALR_RA(1, 3)) \
  ALR_ROW_B(M, 0, 3, ALR_RA(1, 4), ALR_RA(1, 5), ALR_RA(1, 6), ALR_RA(1, 7)) \
  ALR_ROW_F(M, 0, 4, "", FREE, C0, "") \
  ALR_ROW_B(M, 0, 5, C1, "", C2, "") \
  ALR_ROW_F(M, 0, 6, C3, C4, C5, "") \
  ALR_ROW_B(M, 0, 7, C6, "", C7, "")
// half 1: the reads of the next step's half 0 (R), the rest of the refill
#define ALR_HALF1(R, C0, C1, C2, C3, C4, C5, C6, C7) \
  ALR_ROW_F(ALR_MF, 1, 0, R(A, 0), C0, R(B, 0), "") \
  ALR_ROW_B(ALR_MF, 1, 1, R(B, 1), C1, R(B, 2), "") \
  ALR_ROW_F(ALR_MF, 1, 2, R(B, 3), C2, R(B, 4), "") \
  ALR_ROW_B(ALR_MF, 1, 3, R(B, 5), C3, R(B, 6), "") \
  ALR_ROW_F(ALR_MF, 1, 4, R(B, 7), C4, R(A, 1), "") \
  ALR_ROW_B(ALR_MF, 1, 5, R(A, 2), C5, R(A, 3), "") \
  ALR_ROW_F(ALR_MF, 1, 6, R(A, 4), C6, R(A, 5), "") \
  ALR_ROW_B(ALR_MF, 1, 7, R(A, 6), C7, R(A, 7), "")
#define ALR_R0(op, i) ALR_R##op(0, i)
#define ALR_RNONE(op, i) ""
#define ALR_NO_COPIES "", "", "", "", "", "", "", ""
#define ALR_COPIES_A ALR_CA(0), ALR_CA(1), ALR_CA(2), ALR_CA(3), ALR_CA(4), ALR_CA(5), ALR_CA(6), ALR_CA(7)
#define ALR_COPIES_W ALR_CW(0), ALR_CW(1), ALR_CW(2), ALR_CW(3), ALR_CW(4), ALR_CW(5), ALR_CW(6), ALR_CW(7)
#define ALR_HALF0_(...) ALR_HALF0(__VA_ARGS__)
#define ALR_HALF1_(...) ALR_HALF1(__VA_ARGS__)
#define ALR_FREE "s_waitcnt lgkmcnt(0)\n\ts_barrier\n\t"
#define ALR_REFILL ALR_FREE "s_mov_b32 m0, %[lds]\n\t"
// the read addresses move to the other stage
#define ALR_FLIP "v_xor_b32 v112, 0x10000, v112\n\tv_xor_b32 v113, 0x10000, v113\n\t" \
  "v_xor_b32 v114, 0x10000, v114\n\tv_xor_b32 v115, 0x10000, v115\n\t"

#define ALR_WIDE_FRAGS \
  "v128", "v129", "v130", "v131", "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140", "v141", "v142", "v143", \
  "v144", "v145", "v146", "v147", "v148", "v149", "v150", "v151", "v152", "v153", "v154", "v155", "v156", "v157", "v158", "v159", \
  "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167", "v168", "v169", "v170", "v171", "v172", "v173", "v174", "v175", \
  "v176", "v177", "v178", "v179", "v180", "v181", "v182", "v183", "v184", "v185", "v186", "v187", "v188", "v189", "v190", "v191", \
  "v192", "v193", "v194", "v195", "v196", "v197", "v198", "v199", "v200", "v201", "v202", "v203", "v204", "v205", "v206", "v207", \
  "v208", "v209", "v210", "v211", "v212", "v213", "v214", "v215", "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223", \
  "v224", "v225", "v226", "v227", "v228", "v229", "v230", "v231", "v232", "v233", "v234", "v235", "v236", "v237", "v238", "v239", \
  "v240", "v241", "v242", "v243", "v244", "v245", "v246", "v247", "v248", "v249", "v250", "v251", "v252", "v253", "v254", "v255"

typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));

// Epilogue of a wave's 128x128 block whose top-left output is (row0, col0), from
// the accumulators above: acc[2 i + g] holds row block i of 64-column group g.
// `last` is called before the final quarter.
template <class Epi, class F>
__device__ __forceinline__ void wide_store_tile(const Epi& epi, const f32x16 (&acc)[16], int row0,
                                                int col0, int M, int N, F last) {
  const int lane = threadIdx.x & 63, lc = lane & 15;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (q == 3) last();
    const int ih = q & 1, g = q >> 1;
    const int col = col0 + g * 64 + lc, rb = row0 + ih * 64 + 4 * (lane >> 4);
    if (col < N && rb < M) {
      if constexpr (has_rows64<Epi>::value) {
        float v[4][16];
#pragma unroll
        for (int t = 0; t < 16; ++t)
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j][t] = acc[2 * (4 * ih + (t >> 2)) + g][4 * j + (t & 3)];
        epi.rows64(rb, M, col, v);
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          float lo[16], hi[16];
#pragma unroll
          for (int t = 0; t < 16; ++t) {
            lo[t] = acc[2 * (4 * ih + (t >> 2)) + g][4 * j + (t & 3)];
            hi[t] = acc[2 * (4 * ih + (t >> 2)) + g][4 * j + 8 + (t & 3)];
          }
          if constexpr (has_rows<Epi>::value) {
            epi.template rows<16, 16>(rb, M, col + 16 * j, lo, hi);
          } else {
#pragma unroll
            for (int t = 0; t < 16; ++t) {
              const int r = rb + 16 * (t >> 2) + (t & 3);
              if (r < M) epi(r, col + 16 * j, lo[t], hi[t]);
            }
          }
        }
      }
    }
  }
}

// Part of a product: tiles first .. first + count - 1 of its tile order, each cut into
// `splits` slices of (nearly) equal runs of K steps where the epilogue takes raw sums.
struct WideTiles {
  int first, count, splits;
};

// Raw sums of the slices of the tiles past the last full round, for
// gemm_wide_tail_kernel: part[unit][256][256].
struct EpiTail {
  float* part;
  __device__ __forceinline__ void set_unit(int unit, int tm, int tn) {
    part += ((long)unit - tm) * 65536 - tn * 256;
  }
  __device__ __forceinline__ void operator()(int row, int c, float lo, float hi) const {
    part[(long)row * 256 + c] = lo;
    part[(long)row * 256 + c + 32] = hi;
  }
};

template <class Epi, class = void>
struct has_set_unit : std::false_type {};
template <class Epi>
struct has_set_unit<Epi, decltype((void)&Epi::set_unit)> : std::true_type {};

template <class Epi>
struct is_qkv : std::false_type {};
template <typename OutT, bool PAIRS>
struct is_qkv<EpiQKV<OutT, PAIRS>> : std::true_type {};

// Workgroup b takes units b, b + gridDim.x, ...; unit u is slice u % splits of tile
// u / splits of the part.  K is a multiple of 64 and every unit has at least three K
// steps.  The first two K steps of the next unit are copied while this one's epilogue
// runs.
//
// A last round with few tiles costs most of a full one: the down projection of 10,900
// rows (N = 3584, K = 18944) is 602 tiles, 2.35 rounds of 400 us, and took 1.45 ms.  Its
// 90 tiles past the second round are cut over K, 2 slices each, by a second launch,
// and summed by a third: 0.90 + 0.21 + 0.02 ms.  Slicing them inside the first launch
// cost every epilogue registers (spills in SwiGLU's).
template <int TAG, class Epi>
__global__ __launch_bounds__(256, 1) void gemm_bf16_wide_kernel(
    const bf16* __restrict__ A, int lda, const bf16* __restrict__ W, int ldw, int M, int N, int K,
    int tiles_m, int tiles_n, Epi epi, WideTiles wt) {
  constexpr bool sliced = has_set_split<Epi>::value || has_set_unit<Epi>::value;
  constexpr int BM = 256, BN = 256, BK = 64;
  // two stages of [A tile | W tile], rows of 128 bytes swizzled as swz<64>; the
  // stages are 64 KB apart and told apart by that address bit alone
  __shared__ __attribute__((aligned(65536))) bf16 smem[2 * (BM + BN) * BK];
  const int units = sliced ? wt.count * wt.splits : wt.count;
  int unit = blockIdx.x;
  if (unit >= units) return;  // uniform over the workgroup
  const int lane = threadIdx.x & 63, r16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const uint32_t lds0 = lds_byte_addr(smem), ldsw = lds0 + wave * 1024;
  u32x4 rd;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t ch = (uint32_t)(((4 * h + (lane >> 4)) ^ ((r16 & 7) ^ (r16 >> 3))) * 16);
    rd[h] = lds0 + (uint32_t)((wm * 128 + r16) * 128) + ch;
    rd[2 + h] = lds0 + 32768u + (uint32_t)((wn * 128 + r16) * 128) + ch;
  }
  u32x16 vo;
  const bf16 *ga, *gw;
  int tm, tn, steps = K / BK;
  // K steps and tile offsets of a unit, and the copies of its first two steps
  auto begin = [&](int u) {
    int tile = wt.first + u, first = 0;
    if constexpr (sliced) {
      const int t = u / wt.splits, sl = u - t * wt.splits;
      tile = wt.first + t;
      first = K / BK * sl / wt.splits;
      steps = K / BK * (sl + 1) / wt.splits - first;
    }
    gemm_tile_coords(tile, tiles_m, tiles_n, tm, tn);
    ga = A + (long)first * BK;
    gw = W + (long)first * BK;
    // Without this the addresses of a unit's copies are formed once and kept: beside the
    // masks of QKV's rows that is more scalar registers than there are (76 spilled instead of
    // 55, 18 vector registers instead of 13; 1.38 ms instead of 1.29 at 32768 x 6144 x 4096).
    // The other epilogues leave room for them.
    if constexpr (is_qkv<Epi>::value) asm volatile("" : "+s"(ga), "+s"(gw));
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int r = 8 * (j * 4 + wave) + (lane >> 3);
      const int c = (lane & 7) ^ ((r & 7) ^ ((r >> 3) & 1));
      vo[j] = (uint32_t)(((long)min(tm * BM + r, M - 1) * lda + c * 8) * 2);
      vo[8 + j] = (uint32_t)(((long)min(tn * BN + r, N - 1) * ldw + c * 8) * 2);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int j = 0; j < 8; ++j) copy_1k(ldsw + s * 65536 + j * 4096, vo[j], ga);
#pragma unroll
      for (int j = 0; j < 8; ++j) copy_1k(ldsw + s * 65536 + 32768 + j * 4096, vo[8 + j], gw);
      ga += BK;
      gw += BK;
    }
  };
  begin(unit);
  __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));  // vmcnt(0): the first unit's copies
  while (true) {
    const int m0 = tm * BM + wm * 128, n0 = tn * BN + wn * 128;
    f32x16 acc[16];
    int n = steps - 2;  // steps that refill their stage
    uint32_t ldsc = ldsw;
    u32x4 rda = rd;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    // clang-format off
    asm volatile(
        "s_barrier\n\t"  // every wave's copies of the first two steps have landed
        ALR_RA(0, 0) ALR_RB(0, 0) ALR_RB(0, 1) ALR_RB(0, 2) ALR_RB(0, 3) ALR_RB(0, 4) ALR_RB(0, 5) ALR_RB(0, 6)
        ALR_RB(0, 7) ALR_RA(0, 1) ALR_RA(0, 2) ALR_RA(0, 3) ALR_RA(0, 4) ALR_RA(0, 5) ALR_RA(0, 6) ALR_RA(0, 7)
        "s_waitcnt lgkmcnt(0)\n\t"
        ALR_HALF0_(ALR_MZ, ALR_REFILL, ALR_COPIES_A)
        "s_branch 2f\n\t"
        "1:\n\t"
        ALR_HALF0_(ALR_MF, ALR_REFILL, ALR_COPIES_A)
        "2:\n\t"
        ALR_FLIP
        // the next step's copies have landed (the eight newest refill this one)
        "s_waitcnt vmcnt(8)\n\t"
        "s_barrier\n\t"
        ALR_HALF1_(ALR_R0, ALR_COPIES_W)
        "s_add_u32 s40, s40, 128\n\t"
        "s_addc_u32 s41, s41, 0\n\t"
        "s_add_u32 s42, s42, 128\n\t"
        "s_addc_u32 s43, s43, 0\n\t"
        "s_xor_b32 %[lds], %[lds], 0x10000\n\t"
        "s_sub_u32 %[n], %[n], 1\n\t"
        "s_waitcnt lgkmcnt(0)\n\t"
        "s_cmp_lg_u32 %[n], 0\n\t"
        "s_cbranch_scc1 1b\n\t"
        // the last two steps refill nothing
        ALR_HALF0_(ALR_MF, "s_waitcnt lgkmcnt(0)\n\t", ALR_NO_COPIES)
        ALR_FLIP
        "s_waitcnt vmcnt(0)\n\t"
        "s_barrier\n\t"
        ALR_HALF1_(ALR_R0, ALR_NO_COPIES)
        "s_waitcnt lgkmcnt(0)\n\t"
        ALR_HALF0_(ALR_MF, ALR_FREE, ALR_NO_COPIES)
        ALR_HALF1_(ALR_RNONE, ALR_NO_COPIES)
        "s_nop 15\n\t"  // the last results are written before anything reads them
        "s_nop 15\n\t"
        : "={a[0:15]}"(acc[0]), "={a[16:31]}"(acc[1]), "={a[32:47]}"(acc[2]), "={a[48:63]}"(acc[3]),
          "={a[64:79]}"(acc[4]), "={a[80:95]}"(acc[5]), "={a[96:111]}"(acc[6]), "={a[112:127]}"(acc[7]),
          "={a[128:143]}"(acc[8]), "={a[144:159]}"(acc[9]), "={a[160:175]}"(acc[10]), "={a[176:191]}"(acc[11]),
          "={a[192:207]}"(acc[12]), "={a[208:223]}"(acc[13]), "={a[224:239]}"(acc[14]), "={a[240:255]}"(acc[15]),
          "+{v[112:115]}"(rda), "+{s[40:41]}"(ga), "+{s[42:43]}"(gw), [n] "+s"(n), [lds] "+s"(ldsc)
        : "{v[96:111]}"(vo)
        : "memory", "scc", "m0", ALR_WIDE_FRAGS);
    // clang-format on
#pragma clang diagnostic pop
    unit += gridDim.x;
    const bool more = unit < units;
    Epi e = epi;
    if constexpr (has_set_split<Epi>::value) e.set_split((unit - (int)gridDim.x) % wt.splits);
    if constexpr (has_set_unit<Epi>::value) e.set_unit(unit - (int)gridDim.x, tm, tn);
    if (more) begin(unit);
    // Before the last quarter of the epilogue the next unit's copies have
    // landed, so its first reads need not wait for the stores that remain.
    wide_store_tile(e, acc, m0, n0, M, N,
                    [] { __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8)); });
    if (!more) break;
  }
}

// Sum, in slice order, and epilogue of the tiles that were cut over K: workgroup
// (t, b) takes rows 16 b .. + 15 of tile first + t, half-wave w of it the 64-column
// group w % 4 of rows 4 (w / 4) .. + 3 and those + 8.  All 16 loads of a slice are
// independent; bound by reading the partial sums (256 KB a unit).
template <class Epi>
__global__ __launch_bounds__(256) void gemm_wide_tail_kernel(int M, int N, int tiles_m, int tiles_n,
                                                             Epi epi, WideTiles wt,
                                                             const float* __restrict__ part) {
  int tm, tn;
  gemm_tile_coords(wt.first + (int)blockIdx.x, tiles_m, tiles_n, tm, tn);
  const int lc = threadIdx.x & 31, w = threadIdx.x >> 5;
  const int r0 = 16 * blockIdx.y + 4 * (w >> 2), c0 = 64 * (w & 3) + lc;
  const int rb = tm * 256 + r0, col = tn * 256 + c0;
  if (col >= N || rb >= M) return;  // the same for a whole half-wave
  const float* p = part + (long)blockIdx.x * wt.splits * 65536 + r0 * 256 + c0;
  float lo[8], hi[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) lo[t] = hi[t] = 0.f;
#pragma unroll 2
  for (int sl = 0; sl < wt.splits; ++sl)
#pragma unroll
    for (int t = 0; t < 8; ++t) {  // rows past M hold whatever was there, and are not stored
      const float* q = p + (long)sl * 65536 + (8 * (t >> 2) + (t & 3)) * 256;
      lo[t] += q[0];
      hi[t] += q[32];
    }
  if constexpr (has_rows<Epi>::value) {
    epi.template rows<8>(rb, M, col, lo, hi);
  } else {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int r = rb + 8 * (t >> 2) + (t & 3);
      if (r < M) epi(r, col, lo[t], hi[t]);
    }
  }
}

}  // namespace alr
