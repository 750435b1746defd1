// Register-pipelined direct-to-LDS GEMM tiles (included by gemm.hip only).
#pragma once

#include "gemm_dl.h"
#include "gemm_skinny_kn.h"

namespace occ {
namespace {

// ---------------------------------------------------------------------------
// Direct-to-LDS tiles smaller than 256x256, whose MFMAs never wait for an LDS
// read: a wave holds two sets of operand fragments, and the MFMAs of one group
// of 32-wide k-substeps run while the next group's fragments are read into the
// other set and the DMA of a later k-step is issued, one instruction between
// MFMAs.
//
// What bounds such tiles is the latency from the L2 and from LDS, not the matrix
// pipes: with 256 workgroups a k-step took 1400 cycles of which 512 were MFMAs.  In
// this form the pipes are busy 55 % of the cycles with 128x128 tiles (2048x2048x4096,
// B N x K), 27 % with 64x64x128 (1024x1024x4096) and 15 % with 32x64x128
// (512x1024x4096); the waves wait at the barrier 27-38 % of theirs and to issue 14-30.
// A group is the whole k-step (GS = BK / 32) where a wave has few MFMAs, so that
// a read has a k-step to arrive, or one substep (GS = 1), which needs half the
// registers, where it has many.  k-step kt lives in stage kt % STAGES.  Before
// its last group, when the next reads go to k-step kt + 1:
//   - this wave waits for its own reads of k-step kt and its part of the DMA of
//     kt + 1, then meets the others at the k-step's one barrier: kt + 1 is
//     complete and stage kt % STAGES is no longer read;
//   - the DMA of kt + STAGES goes into that stage behind the MFMAs.
// So STAGES - 1 k-steps are in flight or landed ahead of the MFMAs.  k-steps past
// the last are issued with out-of-range offsets: nothing is fetched and the
// counts stay uniform.  LDS layouts, swizzles and the swapped MFMA operands are
// those of gemm_pp.h; the order of the k sums is that of every tile.
//
// Measured on MI355X (us per launch, B N x K / K x N; before = dl tiles, whose
// fragments were read after each barrier):
//   128x128x64, 8 waves, 3 stages: 2048x2048x4096    42 / 42 -> 32 / 32.5
//   256x128x64, 8 waves, 3 stages: 1707x2792x3488    71 / 74 -> 46 / 46
//   128x64x64,  8 waves, 4 stages: 1024x2048x4096    39 / 41 -> 22 / 23
//   64x64x128,  4 waves, 4 stages: 1024x1024x4096    31 / 31 -> 15.5 / 16.5
// The smaller ones take over where 64x64 tiles are fewer than the CUs; there a
// k-step costs a wave's ~90 instructions and one LDS round trip, about 600 cycles
// whatever the tile, so they win by the CUs they add (before = 64x64x128):
//   32x64x128,  4 waves, 3 stages: 512x1024x4096     14.5 / 16.2 -> 11.7 / 12.1
//   32x32x128,  2 waves, 4 stages: 292x448x6736      26.1 / 23.5 -> 14.9 / 17.6
//                                  25x4120x4176      15.1 / 16.9 -> 10.7 / 13.2
// 32x64 with 5 stages: one workgroup per CU instead of two, the same or slower;
// 64x32: 10-40 % slower than 32x64 with K x N B; 32x32 with 64-wide k-steps: 25 %.
// 4 waves with 128x128: 36.6 / 37.2.  More than 3 stages of 128x128 gained
// nothing; 64-wide k-steps with 6 or 8 stages of 64x64 took 17.
//
// NTB: B's DMA is non-temporal.  Chosen by the launcher when one row of tiles
// covers M (each B element is read by one workgroup) and B is too large for the
// 256 MB last-level cache anyway: 64x28672x8192 with 128x128 tiles 105 -> 90 us
// (N x K), 92 -> 86 (K x N); with a B that stays in that cache it is 30 % slower.
template <int BM_, int BN_, int BK_, int WM_, int WN_, int STAGES_, int GS_, bool BKN_, bool NTB_ = false>
struct RpTile {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, STAGES = STAGES_, GS = GS_;
  static constexpr bool BKN = BKN_;                 // B stored K x N, else N x K
  static constexpr bool NTB = NTB_;
  static constexpr int NT = 64 * WM * WN;
  static constexpr int FM = BM / WM / 16, FN = BN / WN / 16, KS = BK / 32;
  static constexpr int KCH = BK / 8;                // 16-byte chunks per operand row
  static constexpr int RPP = NT / KCH;              // rows per DMA pass
  static constexpr int BCH = BN / 8;                // 16-byte chunks per K x N B row
  static constexpr int B_RPP = BKN ? NT / BCH : RPP;
  static constexpr int A_LOADS = BM / RPP, B_LOADS = BKN ? BK / B_RPP : BN / RPP, LOADS = A_LOADS + B_LOADS;
  static constexpr int A_BYTES = BM * BK * 2, STAGE_BYTES = A_BYTES + BN * BK * 2;
  static constexpr int LDS_BYTES = STAGES * STAGE_BYTES;
  static_assert(KCH == 8 || KCH == 16, "BK must be 64 or 128");
  static constexpr int NG = KS / GS;                // fragment groups per k-step
  static_assert(KS % GS == 0 && (NG == 1 || NG % 2 == 0), "groups alternate between two register sets");
  static_assert(FN % 2 == 0, "16-column blocks are stored in pairs");
  static_assert(BM % RPP == 0 && RPP % 8 == 0 && (BKN ? BK % B_RPP == 0 && B_RPP % 16 == 0 : BN % RPP == 0),
                "uneven load passes");
  static_assert(RPP % 16 == 0 || KCH == 16, "passes of 8 rows: the swizzle of rows 8-15 is that of rows 0-7 with c ^ 8");
  static_assert(!BKN || BCH == 4 || BCH == 8 || BCH == 16, "K x N B rows of 32, 64 or 128 columns");
  static_assert((STAGES - 1) * LOADS <= 63, "vmcnt holds at most 63");
};

// Physical 16-byte chunk of logical chunk c in row r of A or N x K B: rows of 256
// bytes are one bank line each, so the 16 rows of an operand read spread by r.
template <int KCH>
__device__ __forceinline__ int swz_rp(int r, int c) {
  if constexpr (KCH == 16) return c ^ (r & 15);
  else return swz<8>(r, c);
}

template <class T>
__global__ __launch_bounds__(T::NT) void gemm_rp_kernel(const uint16_t *__restrict__ A,
                                                        const uint16_t *__restrict__ B,
                                                        uint16_t *__restrict__ C, int M, int N, int K,
                                                        int tiles_m, int tiles_n, int prio, KHooks tr) {
  extern __shared__ __align__(16) unsigned char smem[];  // tile stages, then the unused pad
  set_wave_priority(prio);
  const HookStart t0 = hooks_begin(tr);
  constexpr int S = T::STAGES;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / T::WN, wn = wave % T::WN;
  const int l16 = lane & 15, g = lane >> 4;
  const int ntiles = tiles_m * tiles_n;
  const int nk = (K + T::BK - 1) / T::BK;
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
  const uint32_t wave_lds = (uint32_t)wave * 1024u;

  // DMA slots (as in gemm_dl.h)
  const int r_in = threadIdx.x / T::KCH;
  const int c8 = 8 * swz_rp<T::KCH>(r_in, threadIdx.x % T::KCH);
  const uint32_t lane_off = (uint32_t)r_in * (uint32_t)K * 2u + (uint32_t)c8 * 2u;
  const uint32_t pass_step = (uint32_t)T::RPP * (uint32_t)K * 2u;
  const int kb = threadIdx.x / T::BCH;
  const int cb = swz_skn_b<T::BN * 2>(kb, threadIdx.x % T::BCH);

  // LDS offsets of the operand reads
  int a_rd[T::KS], b_rd[T::BKN ? T::FN : T::KS];
#pragma unroll
  for (int ks = 0; ks < T::KS; ++ks)
    a_rd[ks] = (wm * T::FM * 16 + l16) * T::BK * 2 + swz_rp<T::KCH>(l16, ks * 4 + g) * 16;
  if constexpr (T::BKN) {
    const int r = 8 * g + (l16 >> 2);
#pragma unroll
    for (int j = 0; j < T::FN; ++j)
      b_rd[j] = T::A_BYTES + r * T::BN * 2 +
                swz_skn_b<T::BN * 2>(r, 2 * (wn * T::FN + j) + ((l16 & 3) >> 1)) * 16 + 8 * (l16 & 1);
  } else {
#pragma unroll
    for (int ks = 0; ks < T::KS; ++ks)
      b_rd[ks] = T::A_BYTES + (wn * T::FN * 16 + l16) * T::BK * 2 + swz_rp<T::KCH>(l16, ks * 4 + g) * 16;
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
    const uint32_t vb = n0 + 8 * cb < N ? (uint32_t)kb * (uint32_t)N * 2u + (uint32_t)(n0 + 8 * cb) * 2u : 0x80000000u;
    (void)vb;
    (void)b_bytes;
    auto dma_b = [](i32x4 rs, uint32_t slot, uint32_t v) {
      if constexpr (T::NTB) lds_dma16_nt(rs, slot, v);
      else lds_dma16(rs, slot, v);
    };
    // DMA pass p of k-step kt (A passes, then B passes) into stage `slot`
    auto issue_pass = [&](int kt, uint32_t slot, int p) {
      const int k0 = kt * T::BK;
      const int left = __builtin_amdgcn_readfirstlane(K - k0);
      if (T::BKN && p >= T::A_LOADS) {
        const int q = p - T::A_LOADS;
        const i32x4 rs = make_rsrc(Bn + (size_t)k0 * N, (uint32_t)min(T::BK, max(0, left)) * (uint32_t)N * 2u);
        dma_b(rs, slot + (uint32_t)(T::A_BYTES + q * T::NT * 16), vb + (uint32_t)(q * T::B_RPP) * (uint32_t)N * 2u);
      } else {
        const bool b = p >= T::A_LOADS;
        const int q = b ? p - T::A_LOADS : p;
        const i32x4 rs = make_rsrc((b ? Bn : Am) + k0, left > 0 ? (b ? b_bytes : a_bytes) - (uint32_t)k0 * 2u : 0u);
        // with passes of 8 rows the odd ones are rows 8-15 of 16, whose chunks are swapped by 8 (64 elements)
        const int c = T::RPP == 8 && (q & 1) ? c8 ^ 64 : c8;
        const uint32_t v = c < left ? lane_off + (uint32_t)(c - c8) * 2u : 0x80000000u;
        if (b) dma_b(rs, slot + (uint32_t)(T::A_BYTES + q * T::NT * 16), v + (uint32_t)q * pass_step);
        else lds_dma16(rs, slot + (uint32_t)(q * T::NT * 16), v + (uint32_t)q * pass_step);
      }
    };

    f32x4 acc[T::FM][T::FN];
#pragma unroll
    for (int i = 0; i < T::FM; ++i)
#pragma unroll
      for (int j = 0; j < T::FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // fragments of a group of substeps, double-buffered
    bf16x8 af[2][T::GS][T::FM], bf[2][T::GS][T::FN];
    constexpr int NR = T::GS * (T::FM + T::FN);   // fragments of a group
    constexpr int NM = T::GS * T::FM * T::FN;     // MFMAs of a group
    // fragment x of group gi of the k-step at `cur` into register set `set`
    auto read_frag = [&](const unsigned char *cur, int gi, int set, int x) {
      const int s = x / (T::FM + T::FN), y = x % (T::FM + T::FN), ks = gi * T::GS + s;
      if (y < T::FM) {
        af[set][s][y] = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const u32x4 *>(cur + a_rd[ks] + y * 16 * T::BK * 2));
      } else if constexpr (T::BKN) {
        const int j = y - T::FM;
        const unsigned char *p = cur + b_rd[j] + ks * 32 * T::BN * 2;
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)p);
        const i16x4 hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4 *)(p + 4 * T::BN * 2));
        bf[set][s][j] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      } else {
        const int j = y - T::FM;
        bf[set][s][j] = __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const u32x4 *>(cur + b_rd[ks] + j * 16 * T::BK * 2));
      }
    };
    auto mfma = [&](int set, int x) {
      const int s = x / (T::FM * T::FN), i = x / T::FN % T::FM, j = x % T::FN;
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[set][s][j], af[set][s][i], acc[i][j], 0, 0, 0);
    };
    auto slot_of = [&](int s) { return lds0 + (uint32_t)s * T::STAGE_BYTES + wave_lds; };
    auto publish = [&]() {  // this wave's reads are done; then every wave's, and its DMA has landed
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    };

#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int p = 0; p < T::LOADS; ++p) issue_pass(s, slot_of(s), p);
    wait_vmcnt<(S - 1) * T::LOADS>();
    publish();
#pragma unroll
    for (int x = 0; x < NR; ++x) read_frag(smem, 0, 0, x);
    int stage = 0;  // stage of the k-step being multiplied
    auto step = [&](int kt, int set0) {
      const int next = stage + 1 == S ? 0 : stage + 1;
      const unsigned char *cur = smem + stage * T::STAGE_BYTES, *nxt = smem + next * T::STAGE_BYTES;
      const uint32_t slot = slot_of(stage);
#pragma unroll
      for (int gi = 0; gi < T::NG; ++gi) {
        const int set = (set0 + gi) & 1;
        const bool last = gi + 1 == T::NG;
        if (last) {
          wait_vmcnt<(S - 2) * T::LOADS>();
          publish();
        }
#pragma unroll
        for (int x = 0; x < NM; ++x) {
          mfma(set, x);
          // the reads behind the first half of the MFMAs, the DMA behind all of them
#pragma unroll
          for (int y = 0; y < NR; ++y)
            if (y * (NM / 2) / NR == x) read_frag(last ? nxt : cur, last ? 0 : gi + 1, set ^ 1, y);
#pragma unroll
          for (int p = 0; p < T::LOADS; ++p)
            if (last && p * NM / T::LOADS == x) issue_pass(kt + S, slot, p);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      stage = next;
    };
    if constexpr (T::NG == 1) {
      int kt = 0;
      for (; kt + 1 < nk; kt += 2) {
        step(kt, 0);
        step(kt + 1, 1);
      }
      if (kt < nk) step(kt, 0);
    } else {
      for (int kt = 0; kt < nk; ++kt) step(kt, 0);
    }
    // the DMA issued past the last k-step is done before the stages get other use
    wait_vmcnt<0>();
    publish();

    // as in gemm_pp.h: a lane holds 4 columns of row l16 of a block, and after
    // the swaps 8 columns of one of two neighbouring blocks
    int el = lane;
    asm volatile("" : "+v"(el));  // keeps the addresses below out of the k-loop's registers
    const int em = el & 15;
    const int en = wn * T::FN * 16 + ((el >> 4) & 1) * 16 + (el >> 5) * 8;
    const bool wide = (N & 7) == 0 && N <= (1 << 24);
#pragma unroll
    for (int i = 0; i < T::FM; ++i) {
      const int mb = m0 + (wm * T::FM + i) * 16;
      const uint32_t c_bytes = (uint32_t)min(16, max(0, M - mb)) * (uint32_t)N * 2u;
      const CStore cs(C + (size_t)mb * N, c_bytes, tr.release);
#pragma unroll
      for (int jp = 0; jp < T::FN / 2; ++jp) {
        const f32x4 p = acc[i][2 * jp], q = acc[i][2 * jp + 1];
        u32x4 v;
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          const auto s = __builtin_amdgcn_permlane16_swap(pack_bf16(p[2 * d], p[2 * d + 1]),
                                                          pack_bf16(q[2 * d], q[2 * d + 1]), false, false);
          v[d] = s[0];
          v[2 + d] = s[1];
        }
        const int n = n0 + jp * 32 + en;
        if (wide) {
          cs.put(v, n < N ? ((uint32_t)em * (uint32_t)N + (uint32_t)n) * 2u : 0x80000000u);
        } else if (mb + em < M) {
          store_c_ragged(C + (size_t)(mb + em) * N + n, v, N - n, tr.release);
        }
      }
    }
  }
  hooks_end(tr, t0);
}

}  // namespace
}  // namespace occ
