// Large-tile GEMM kernel whose two halves of waves alternate between loading
// and multiplying (included by gemm.hip only).
#pragma once

#include "gemm_dl.h"
#include "gemm_skinny_kn.h"

namespace occ {
namespace {

// ---------------------------------------------------------------------------
// 256 x 256 output tile, k-steps of 64, 8 waves, two LDS stages (128 KiB), one
// workgroup per CU: two waves per SIMD, one of each half of the workgroup
// (waves 0-3, waves 4-7).
//
// What bounded the 256x256 tile was the delivery of its operands (64 KiB per
// k-step and CU from the L2 through direct-to-LDS DMA): 69 % of the MFMA cycles
// with all waves loading, meeting and multiplying together.  Two groups of waves
// that take turns at it, the "ping-pong" schedule known from other GPU GEMMs, keep
// the pipes busy: a k-step never drains its DMA, and no wave reads LDS while its
// SIMD's matrix pipe is idle:
//
//  * Every k-step has two phases: rows 0-127 of the tile (A0) and rows 128-255
//    (A1), each against all 256 columns, 32 MFMAs per wave.  A phase is a load
//    slot (LDS reads of its operands, DMA issue, waits), a barrier, a multiply
//    slot and a barrier.  Waves 4-7 run one slot behind waves 0-3 (one extra
//    barrier before their first phase), so that on every SIMD one wave
//    multiplies while the other loads.
//  * A stage is four 16 KiB parts, A0 A1 B0 B1.  A0, B0 and B1 of k-step kt are
//    read in its first phase and A1 in its second, so their slots are refilled
//    for k-step kt + 2 one phase later: A0, B0, B1 in the second phase of kt,
//    A1 in the first phase of kt + 1.  Each wave issues 6 and 2 DMA per phase
//    and waits until at most 8 are outstanding: 64 to 128 KiB per CU in flight
//    at any time, every part three phases ahead of its use.
//  * Hazards.  A load slot ends with its own LDS reads done (lgkmcnt(0)) and
//    the DMA of the next phase's parts landed (vmcnt(8)), then the barrier.  A
//    part read in slot s by either half is refilled two slots after the leading
//    half's read, one after the trailing half's; a part's DMA has been waited
//    for by every wave at least one barrier before the leading half reads it.
//  * k-steps past the last are issued too (their offsets are out of range, so
//    nothing is fetched): the counts stay uniform.
//
// 16x16x32 MFMAs: they take about 13 % less energy per flop than 32x32x16 on
// random operands, and what bounds the kernel now is the board's power: 77-79 % (K x
// N) and 83-88 % (N x K) of the MFMA cycles at 1.5-1.8 GHz, 1396-1400 W of its cap of
// 1400 (8192^3, sustained; 0 LDS bank conflicts).  The
// operands go in swapped (B first), so that a lane holds 4 consecutive columns
// of one row of C; two permlane16 swaps pair two 16-column blocks into 16-byte
// stores.  At most 224 VGPRs (a CPU test reads the built kernels'), so that 64 of a
// SIMD's 512 stay free for a collective's wave.
//
// Measured (MI355X, N(0,1) operands; before = one DMA drain and one barrier per
// k-step for all waves, 32x32x16): 8192^3 B K x N 0.825 -> 0.725 ms (1.52
// PFLOP/s), B N x K 0.825 -> 0.69 ms (1.60; hipBLASLt 1.40 and 1.61);
// 16384x14336x4096 1.50 -> 1.32 and 1.26 ms; 4096^3 0.108 -> 0.097 and 0.095.
// Four phases of 16 MFMAs per k-step were 2-3 % slower, raising the wave
// priority around the MFMAs or prefetching the next tile of a persistent
// workgroup under the epilogue gained nothing.
template <bool BKN_>
struct PpTile {
  static constexpr int BM = 256, BN = 256, BK = 64, NT = 512;
  static constexpr bool BKN = BKN_;                 // B stored K x N, else N x K
  static constexpr int PART_BYTES = 128 * BK * 2;   // 128 rows (columns) of a k-step
  static constexpr int STAGE_BYTES = 4 * PART_BYTES;
  static constexpr int LDS_BYTES = 2 * STAGE_BYTES;
};

template <class T>
__global__ __launch_bounds__(T::NT) void gemm_pp_kernel(const uint16_t *__restrict__ A,
                                                        const uint16_t *__restrict__ B,
                                                        uint16_t *__restrict__ C, int M, int N, int K,
                                                        int tiles_m, int tiles_n, int prio, KHooks tr) {
  extern __shared__ __align__(16) unsigned char smem[];  // two stages, then the unused pad
  set_wave_priority(prio);
  const HookStart t0 = hooks_begin(tr);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = wave >> 2;  // which half of the waves; rows 64*half .. of A0 and of A1
  const int wn = wave & 3;     // columns 32*wn .. of B0 and of B1
  const int l16 = lane & 15, g = lane >> 4;
  const int ntiles = tiles_m * tiles_n;
  const int nk = (K + T::BK - 1) / T::BK;
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
  const uint32_t wave_lds = (uint32_t)wave * 1024u;

  // DMA slots of A and N x K B: row r_in of a 64-row pass, physical chunk
  // tid % 8 (the swizzle of gemm_dl.h, the same in every pass)
  const int r_in = threadIdx.x >> 3;
  const int c8 = 8 * swz<8>(r_in, threadIdx.x & 7);  // first k of this lane's chunk
  const uint32_t lane_off = (uint32_t)r_in * (uint32_t)K * 2u + (uint32_t)c8 * 2u;
  const uint32_t pass_step = 64u * (uint32_t)K * 2u;
  // K x N B: row kb of a 32-row pass, 256 bytes of columns per row
  const int kb = threadIdx.x >> 4;
  const int cb = swz_skn_b<256>(kb, threadIdx.x & 15);

  // LDS offsets of the operand reads: A and N x K B by 32-wide k-substep, K x N
  // B by 16-column block
  int a_rd[2], b_rd[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) a_rd[ks] = (half * 64 + l16) * 128 + swz<8>(l16, ks * 4 + g) * 16;
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    if constexpr (T::BKN) {
      const int r = 8 * g + (l16 >> 2);
      b_rd[x] = 2 * T::PART_BYTES + r * 256 + swz_skn_b<256>(r, 2 * (2 * wn + x) + ((l16 & 3) >> 1)) * 16 + 8 * (l16 & 1);
    } else {
      b_rd[x] = 2 * T::PART_BYTES + (wn * 32 + l16) * 128 + swz<8>(l16, x * 4 + g) * 16;
    }
  }

  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    int tm, tn;
    tile_coords<8>(xcd_remap(t, ntiles), tiles_m, tiles_n, tm, tn);
    const int m0 = tm * T::BM;
    const int n0 = tn * T::BN;
    const uint32_t a_bytes = (uint32_t)min(T::BM, M - m0) * (uint32_t)K * 2u;
    const uint32_t b_bytes = T::BKN ? 0u : (uint32_t)min(T::BN, N - n0) * (uint32_t)K * 2u;
    const uint16_t *Am = A + (size_t)m0 * K;
    const uint16_t *Bn = T::BKN ? B : B + (size_t)n0 * K;
    uint32_t vb[2] = {0u, 0u};
    if constexpr (T::BKN) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int n = n0 + 128 * h + 8 * cb;
        vb[h] = n < N ? (uint32_t)kb * (uint32_t)N * 2u + (uint32_t)n * 2u : 0x80000000u;
      }
    }
    // DMA of part `p` (0, 1: A0, A1; 2, 3: B0, B1) of k-step kt.  The
    // descriptor starts at the k-step's first k and ends with the operand's
    // rows; chunks past K get an offset beyond any range.
    auto issue = [&](int kt, int p) {
      const int k0 = kt * T::BK;
      const int left = __builtin_amdgcn_readfirstlane(K - k0);
      const uint32_t slot = lds0 + (uint32_t)(kt & 1) * T::STAGE_BYTES + (uint32_t)p * T::PART_BYTES + wave_lds;
      if (T::BKN && p >= 2) {
        const i32x4 rs = make_rsrc(Bn + (size_t)k0 * N, (uint32_t)min(T::BK, max(0, left)) * (uint32_t)N * 2u);
        lds_dma16(rs, slot, vb[p & 1]);
        lds_dma16(rs, slot + 8192u, vb[p & 1] + 32u * (uint32_t)N * 2u);
      } else {
        const uint32_t bytes = left > 0 ? (p >= 2 ? b_bytes : a_bytes) - (uint32_t)k0 * 2u : 0u;
        const i32x4 rs = make_rsrc((p >= 2 ? Bn : Am) + k0, bytes);
        const uint32_t v = c8 < left ? lane_off + (uint32_t)(p & 1) * 2u * pass_step : 0x80000000u;
        lds_dma16(rs, slot, v);
        lds_dma16(rs, slot + 8192u, v + pass_step);
      }
    };

    f32x4 acc[2][4][4];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[h][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    bf16x8 af[2][4], bf[2][4];  // [32-wide k-substep][16-row or 16-column block (2 of B0, 2 of B1)]
    auto read_a = [&](const unsigned char *cur, int h) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          af[ks][i] = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4 *>(cur + a_rd[ks] + h * T::PART_BYTES + i * 2048));
    };
    auto read_b = [&](const unsigned char *cur, int h) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if constexpr (T::BKN) {
            const unsigned char *p = cur + b_rd[j] + h * T::PART_BYTES + ks * 32 * 256;
            const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)p);
            const i16x4 hi =
                __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(p + 4 * 256));
            bf[ks][2 * h + j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
          } else {
            bf[ks][2 * h + j] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u32x4 *>(cur + b_rd[ks] + h * T::PART_BYTES + j * 2048));
          }
        }
    };
    auto multiply = [&](int h) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[h][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[ks][j], af[ks][i], acc[h][i][j], 0, 0, 0);
    };
    auto barrier = [&]() {  // nothing moves across it
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    };
    auto end_load_slot = [&]() {
      wait_vmcnt<8>();
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      barrier();
    };

    issue(0, 0); issue(0, 2); issue(0, 3);
    issue(0, 1);
    issue(1, 0); issue(1, 2); issue(1, 3);
    wait_vmcnt<8>();
    barrier();
    if (half == 1) barrier();
    for (int kt = 0; kt < nk; ++kt) {
      const unsigned char *cur = smem + (kt & 1) * T::STAGE_BYTES;
      read_a(cur, 0);
      read_b(cur, 0);
      read_b(cur, 1);
      issue(kt + 1, 1);
      end_load_slot();
      multiply(0);
      barrier();
      read_a(cur, 1);
      issue(kt + 2, 0); issue(kt + 2, 2); issue(kt + 2, 3);
      end_load_slot();
      multiply(1);
      barrier();
    }
    if (half == 0) barrier();
    // the DMA issued past the last k-step writes zeros into the stages: done
    // before the next tile, or the end of the workgroup, gives them other use
    wait_vmcnt<0>();
    barrier();

    // A 16x16 result block is a block of C^T: lane holds row l16, columns
    // 4g .. 4g+3.  Swapping odd rows of lanes of one 16-column block with even
    // rows of the next gives every lane 8 consecutive columns.
    int el = lane;
    asm volatile("" : "+v"(el));  // keeps the addresses below out of the k-loop's registers
    const int em = el & 15;
    const int en = wn * 32 + ((el >> 4) & 1) * 16 + (el >> 5) * 8;
    // 16-byte stores when the rows of C are 16-byte aligned (and, for the
    // 32-bit offsets of 16 rows, N within 16 M)
    const bool wide = (N & 7) == 0 && N <= (1 << 24);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int mb = m0 + h * 128 + half * 64 + i * 16;  // first row of the block
        const uint32_t c_bytes = (uint32_t)min(16, max(0, M - mb)) * (uint32_t)N * 2u;
        const CStore cs(C + (size_t)mb * N, c_bytes, tr.release);
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
          const f32x4 p = acc[h][i][2 * hb], q = acc[h][i][2 * hb + 1];
          u32x4 v;
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            const auto s = __builtin_amdgcn_permlane16_swap(pack_bf16(p[2 * d], p[2 * d + 1]),
                                                            pack_bf16(q[2 * d], q[2 * d + 1]), false, false);
            v[d] = s[0];
            v[2 + d] = s[1];
          }
          const int n = n0 + hb * 128 + en;
          if (wide) {
            cs.put(v, n < N ? ((uint32_t)em * (uint32_t)N + (uint32_t)n) * 2u : 0x80000000u);
          } else if (mb + em < M) {
            store_c_ragged(C + (size_t)(mb + em) * N + n, v, N - n, tr.release);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
  }
  hooks_end(tr, t0);
}

}  // namespace
}  // namespace occ
