// K_g: bf16 GEMM on MFMA (gfx950), fp32 accumulation, bf16 output.
//
// Background, item 1: C = A * B, the GEMM of a linear layer, tiled and staged
// through on-chip memory.  Section 3.1: the LDS a workgroup allocates,
// S_blk ~ TILE_M*TILE_K + TILE_K*TILE_N, bounds how many GEMM workgroups
// reside on a CU; an extra dynamic-LDS pad on top of the tile's own LDS lowers
// that residency without changing the kernel's arithmetic.
//
// Layout: A is M x K and C is M x N, row-major.  B is stored K x N (occ_gemm:
// C = A * B, the B tile is staged as stored and read with LDS transpose
// reads) or N x K (occ_gemm_bt: C = A * B^T, a linear layer's weight layout,
// both MFMA operands read from LDS as 16-byte rows).
//
// The kernels live in gemm_pp.h (256x256 tiles, both layouts), gemm_rp.h
// (register-pipelined smaller tiles, both layouts), gemm_dl.h (the paper's and
// other direct-to-LDS tiles, both layouts),
// gemm_tiled.h (register-staged tiles, the paper's opt1/opt2 with B N x K),
// gemm_skinny.h and gemm_skinny_ldsb.h (M <= 16, B N x K) and
// gemm_skinny_kn.h (M <= 16, B K x N); this file holds the variant table, the
// launch plan and the launcher.
#include "gemm_dl.h"
#include "gemm_pp.h"
#include "gemm_rp.h"
#include "gemm_skinny.h"
#include "gemm_skinny_kn.h"
#include "gemm_skinny_ldsb.h"
#include "gemm_tiled.h"

#include <algorithm>
#include <cmath>

namespace occ {
namespace {

// ---------------------------------------------------------------------------
// Variant table.
typedef void (*TiledFn)(const uint16_t *, const uint16_t *, uint16_t *, int, int, int, int, int,
                        int, KHooks);

typedef void (*SkinnyFn)(const uint16_t *, const uint16_t *, uint16_t *, int, int, int, int, KHooks);

struct Variant {
  int id;
  int bm, bn, bk, threads, lds;
  TiledFn fn;        // tiled kernels
  SkinnyFn skinny;   // skinny kernels (M <= 16)
  const char *name;
  int kmax;          // largest K the kernel takes (0 = any)
  int kmult;         // K must be a multiple of this (0 = any)
  bool b_kn;         // takes B stored K x N (and only that)
  int nmax;          // largest N the kernel takes (0 = any)
  int per_cu;        // skinny kernels: persistent workgroups per CU (0 = 1)
  TiledFn fn_nt;     // the same with B's loads non-temporal, where the kernel has that form
  // the same with C's stores of device scope, where that is a kernel of its own
  // (the others choose at run time)
  TiledFn fn_through = nullptr;
  SkinnyFn skinny_through = nullptr;
};

template <class T>
constexpr Variant make_variant(int id, const char *name) {
  return Variant{id, T::BM, T::BN, T::BK, T::NT, T::LDS_BYTES, gemm_tiled_kernel<T>, nullptr, name, 0, 0, false, 0, 0,
                 nullptr};
}

// The direct-to-LDS kernel addresses an operand tile with 32-bit byte
// offsets from the tile's first row (row * K * 2 + k * 2) and marks missing
// k with an offset of 2^31: K is capped so that a tile spans at most 2^31
// bytes (no offset wraps and every marked offset is out of range).
template <class T>
constexpr int dl_kmax() {
  return (int)((0x80000000ull / (2ull * (unsigned long long)(T::BM > T::BN ? T::BM : T::BN))) & ~7ull);
}

// A K x N B k-step (BK rows of N) is addressed the same way with N in place of K.
template <class T>
constexpr int dl_nmax() {
  return T::BKN ? (int)((0x80000000ull / (2ull * (unsigned long long)T::BK)) & ~7ull) : 0;
}

template <class T>
constexpr Variant make_dl_variant(int id, const char *name) {
  return Variant{id, T::BM, T::BN, T::BK, T::NT, T::LDS_BYTES, gemm_dl_kernel<T, false>, nullptr, name,
                 dl_kmax<T>(), 0, T::BKN, dl_nmax<T>(), 0, nullptr, gemm_dl_kernel<T, true>};
}

// The two-group kernel addresses its operands in the same way.
template <class T>
constexpr Variant make_pp_variant(int id, const char *name) {
  return Variant{id, T::BM, T::BN, T::BK, T::NT, T::LDS_BYTES, gemm_pp_kernel<T>, nullptr, name,
                 dl_kmax<T>(), 0, T::BKN, dl_nmax<T>(), 0, nullptr};
}

// So do the register-pipelined tiles; NT also has the form with non-temporal B.
template <class T, class NT>
constexpr Variant make_rp_variant(int id, const char *name) {
  return Variant{id, T::BM, T::BN, T::BK, T::NT, T::LDS_BYTES, gemm_rp_kernel<T>, nullptr, name,
                 dl_kmax<T>(), 0, T::BKN, dl_nmax<T>(), 0, gemm_rp_kernel<NT>};
}
template <class T>
constexpr Variant make_rp_variant(int id, const char *name) {
  Variant v = make_rp_variant<T, T>(id, name);
  v.fn_nt = nullptr;
  return v;
}

template <int WAVES, int UNROLL>
constexpr Variant make_skinny_variant(int id, const char *name) {
  return Variant{id, 16, 16, kSkinnyKB * UNROLL, 64 * WAVES, (WAVES - 1) * 64 * 16, nullptr,
                 gemm_skinny_kernel<WAVES, UNROLL>, name, 0, 0, false, 0, 0, nullptr};
}

// A K x N B block (32 rows of N) is addressed with 32-bit offsets from its
// first row (columns past N marked with 2^31), an A row (M <= 16 rows of K)
// likewise from A.
template <int WAVES, int STAGES, int COLS>
constexpr Variant make_skinny_kn_variant(int id, const char *name) {
  return Variant{id, 16, COLS, kSknKB, 64 * WAVES, SkinnyKn<WAVES, STAGES, COLS>::LDS_BYTES, nullptr,
                 gemm_skinny_kn_kernel<WAVES, STAGES, COLS, false>, name, (int)((0x80000000ull / 32u) & ~7ull), 0,
                 true, (int)((0x80000000ull / (2u * kSknKB)) & ~7ull), 2, nullptr, nullptr,
                 gemm_skinny_kn_kernel<WAVES, STAGES, COLS, true>};
}

// B staged through LDS in 128-k blocks, A in registers: K a multiple of
// 128 * WAVES, at most 32 * WAVES * KBW.
template <int WAVES, int STAGES, int KBW>
constexpr Variant make_skinny_ldsb_variant(int id, const char *name) {
  return Variant{id, 16, 16, kSlbKB, 64 * WAVES, SkinnyLdsB<WAVES, STAGES, KBW>::LDS_BYTES, nullptr,
                 gemm_skinny_ldsb_kernel<WAVES, STAGES, KBW, false>, name, 32 * WAVES * KBW, kSlbKB * WAVES, false, 0, 1,
                 nullptr, nullptr, gemm_skinny_ldsb_kernel<WAVES, STAGES, KBW, true>};
}

// B stored N x K (occ_gemm_bt)
using T64x64_opt1 = Tile<64, 64, 32, 2, 2, 1>;   // Table 1 opt1: 64x64x32
using T64x64_opt2 = Tile<64, 64, 64, 2, 2, 1>;   // Table 1 opt2: 64x64x64
// the opt2 tile with two direct-to-LDS stages: the automatic choice for small
// shapes (one k-step's DMA in flight while the previous one is used)
using D64x64_4w_2s = Tile<64, 64, 64, 2, 2, 2>;
// two workgroups per CU: each has its own barriers, so one computes while the
// other waits (48 KiB of LDS, 4 waves of 128x64 each)
using P128x256k32_4w_2s = Tile<128, 256, 32, 1, 4, 2, true, 2>;

// B stored K x N (occ_gemm): the same tiles with the B tile staged as stored
// and its MFMA operands read with LDS transpose reads
using KN64x64_opt1 = Tile<64, 64, 32, 2, 2, 1, false, 1, true>;   // Table 1 opt1, one stage
using KN64x64_opt2 = Tile<64, 64, 64, 2, 2, 1, false, 1, true>;   // Table 1 opt2, one stage
using KN64x64_4w_2s = Tile<64, 64, 64, 2, 2, 2, false, 1, true>;
using PKN128x256k32_4w_2s = Tile<128, 256, 32, 1, 4, 2, true, 2, true>;

// the register-pipelined tiles, both layouts
template <bool BKN>
using R256x128 = RpTile<256, 128, 64, 4, 2, 3, 1, BKN>;
template <bool BKN, bool NTB = false>
using R128x128 = RpTile<128, 128, 64, 2, 4, 3, 1, BKN, NTB>;
template <bool BKN>
using R128x64 = RpTile<128, 64, 64, 4, 2, 4, 2, BKN>;
template <bool NTB>
using R64x128k128 = RpTile<64, 128, 128, 2, 4, 3, 2, false, NTB>;
template <bool BKN>
using R64x64k128 = RpTile<64, 64, 128, 2, 2, 4, 4, BKN>;
template <bool BKN>
using R32x64k128 = RpTile<32, 64, 128, 2, 2, 3, 4, BKN>;
template <bool BKN>
using R32x32k128 = RpTile<32, 32, 128, 2, 1, 4, 4, BKN>;

const Variant kVariants[] = {
    // B stored N x K
    make_variant<T64x64_opt1>(6, "64x64x32 opt1, B N x K"),
    make_variant<T64x64_opt2>(7, "64x64x64 opt2, B N x K"),
    make_dl_variant<D64x64_4w_2s>(9, "dl 64x64x64 4w 2st, B N x K"),
    make_rp_variant<R256x128<false>>(10, "rp 256x128x64 8w 3st, B N x K"),
    make_rp_variant<R128x64<false>>(11, "rp 128x64x64 8w 4st, B N x K"),
    make_rp_variant<R32x64k128<false>>(17, "rp 32x64x128 4w 3st, B N x K"),
    make_rp_variant<R32x32k128<false>>(18, "rp 32x32x128 2w 4st, B N x K"),
    make_rp_variant<R64x64k128<false>>(12, "rp 64x64x128 4w 4st, B N x K"),
    make_rp_variant<R64x128k128<false>, R64x128k128<true>>(13, "rp 64x128x128 8w 3st, B N x K"),
    make_rp_variant<R128x128<false>, R128x128<false, true>>(14, "rp 128x128x64 8w 3st, B N x K"),
    make_pp_variant<PpTile<false>>(16, "pp 256x256x64 8w 2st, B N x K"),
    make_skinny_variant<8, 8>(21, "skinny M<=16, 8 waves, unroll 8, B N x K"),
    make_dl_variant<P128x256k32_4w_2s>(25, "dl+pipe 128x256x32 4w 2st 2wg/cu, B N x K"),
    make_skinny_ldsb_variant<8, 2, 32>(34, "skinny M<=16, B via LDS in 256-byte row pieces, A in registers, 8 waves, K<=8192, K%1024==0, B N x K"),
    // B stored K x N
    make_pp_variant<PpTile<true>>(32, "pp 256x256x64 8w 2st, B K x N"),
    make_skinny_kn_variant<4, 2, 128>(33, "skinny M<=16, units of up to 128 columns, 4 waves, 2 LDS stages, B K x N"),
    make_rp_variant<R128x128<true>, R128x128<true, true>>(35, "rp 128x128x64 8w 3st, B K x N"),
    make_dl_variant<KN64x64_opt1>(36, "dl 64x64x32 opt1 1st, B K x N"),
    make_dl_variant<KN64x64_opt2>(37, "dl 64x64x64 opt2 1st, B K x N"),
    make_dl_variant<PKN128x256k32_4w_2s>(38, "dl+pipe 128x256x32 4w 2st 2wg/cu, B K x N"),
    make_dl_variant<KN64x64_4w_2s>(39, "dl 64x64x64 4w 2st, B K x N"),
    make_rp_variant<R256x128<true>>(40, "rp 256x128x64 8w 3st, B K x N"),
    make_rp_variant<R128x64<true>>(41, "rp 128x64x64 8w 4st, B K x N"),
    make_rp_variant<R64x64k128<true>>(42, "rp 64x64x128 4w 4st, B K x N"),
    make_rp_variant<R32x64k128<true>>(43, "rp 32x64x128 4w 3st, B K x N"),
    make_rp_variant<R32x32k128<true>>(44, "rp 32x32x128 2w 4st, B K x N"),
};

// Variant 33's narrower units (gemm_skinny_kn.h); same sums, bit for bit.
const Variant kSkinnyKn64 = make_skinny_kn_variant<4, 3, 64>(33, "skinny M<=16, 64-column units, 4 waves, 3 LDS stages, B K x N");
const Variant kSkinnyKn32 = make_skinny_kn_variant<4, 4, 32>(33, "skinny M<=16, 32-column units, 4 waves, 4 LDS stages, B K x N");

constexpr int kMaxVariantId = 63;  // launch-attribute caches are indexed by id
constexpr int kMaxDevices = 64;    // and by device

bool is_skinny(const Variant *v) { return v->skinny != nullptr; }

const Variant *find_variant(int id) {
  for (const Variant &v : kVariants)
    if (v.id == id) return &v;
  return nullptr;
}

int ceil_div(long long a, long long b) { return (int)((a + b - 1) / b); }

// The form of variant `id` for a call: variant 33 takes the widest units that
// leave no CU without one, down to a quarter of the CUs with 32 columns.
const Variant *variant_form(const GemmCall &c, int id, int num_cus) {
  if (id == 33) {
    if (ceil_div(c.N, 32) <= num_cus / 4) return &kSkinnyKn32;
    if (ceil_div(c.N, 64) <= num_cus) return &kSkinnyKn64;
  }
  return find_variant(id);
}

// B too large for the 256 MB last-level cache.
bool b_exceeds_llc(int N, int K) { return (long long)N * K * 2 > (256ll << 20); }

// Estimated time (us) of a tile on a shape: the launch, then the rounds in which
// `slots` workgroups at a time work off the tiles, each `fixed` (prologue,
// epilogue) plus `step` per 64 of K.  The constants are the measured times of
// single rounds on MI355X: 2048x2048x4096 takes one round of 128x128 tiles, 33.5
// us = 3 + 2 + 64 * 0.44; 64x64 tiles of two small stages share a CU, so their
// rounds need not be whole.  On 47 shapes of 64..8192 (M), 128..28672 (N) and
// 128..8192 (K) in both layouts the choice is within 0.7 % of the fastest tile
// on average (11 % at most), and 22 % faster than 256x256, 128x128 and 64x64
// chosen by tile count alone.  The 32-row tiles win where 64x64 ones leave half
// of the CUs or more idle: on 39 more shapes of 17..1200 (M), 128..28672 (N) and
// 520..8192 (K) the choice with them is within 0.5 (N x K) and 0.1 % (K x N) of the
// fastest on average (19 and 3 % at most).  On 35 shapes of K 64..512 it is within
// 3 and 1.5 % (16 and 9 % at most: up to K = 256 the 64x64 tile's estimate is too
// low against 32x32, 134x352x256 N x K 3.8 us and 3.3), and up to 26 % faster than
// with the 64x64 tile wherever it takes a 32-row one (512x512x512 4.6 -> 3.8 N x K,
// 4.6 -> 4.0 K x N; the schedule of that GEMM and a 4 x 2^18 chunk sum with the
// device counter 114 -> 102 us for 10 iterations, sequential 71 -> 66).
struct TileCost {
  int id_nk, id_kn;
  double launch, fixed, step;
  bool shared;  // several workgroups per CU
};
const TileCost kTileCosts[] = {
    {16, 32, 3.0, 4.0, 1.1, false},   // 256x256
    {10, 40, 3.0, 2.5, 0.68, false},  // 256x128
    {14, 35, 3.0, 2.0, 0.44, false},  // 128x128
    {11, 41, 3.0, 1.6, 0.29, false},  // 128x64
    {12, 42, 3.0, 1.6, 0.19, false},  // 64x64x128
    {17, 43, 2.5, 1.3, 0.155, false},  // 32x64x128
    {18, 44, 2.4, 1.2, 0.148, false},  // 32x32x128
    {9, 39, 1.6, 0.4, 0.45, true},    // 64x64
};

// The tile for M > 16 among those whose LDS fits in `room` bytes, 0 if none: the
// one with the least estimated time, except that a B which is read once and
// comes from memory goes to a tile that covers M and whose loads can be
// non-temporal: the tile then matters little, the loads much.  That is 128x128,
// or for N x K B and M <= 64 64x128 with k-steps of 128, which read 256-byte
// pieces of B's rows (64x28672x8192 98 -> 92 us, 64x65536x4096 114 -> 104; K x N
// B has 256-byte pieces in both and no difference).
int fastest_tile(const GemmCall &c, int num_cus, int room) {
  const int M = c.M, N = c.N, K = c.K;
  const int mid = c.b_kn ? 35 : 14;
  if (M <= 128 && b_exceeds_llc(N, K)) {
    if (!c.b_kn && M <= 64 && find_variant(13)->lds <= room) return 13;
    if (find_variant(mid)->lds <= room) return mid;
  }
  const int slots = c.grid_cap > 0 && c.grid_cap < num_cus ? c.grid_cap : num_cus;
  double best = 0;
  int v = 0;
  for (const TileCost &tc : kTileCosts) {
    const Variant *pv = find_variant(c.b_kn ? tc.id_kn : tc.id_nk);
    if (pv->lds > room) continue;
    const double tiles = (double)ceil_div(M, pv->bm) * ceil_div(N, pv->bn);
    const double rounds = tc.shared ? std::max(1.0, tiles / slots) : std::ceil(tiles / slots);
    const double t = tc.launch + rounds * (tc.fixed + tc.step * ceil_div(K, 64));
    if (best == 0 || t < best) {
      best = t;
      v = pv->id;
    }
  }
  return v;
}

// The kernel for a shape.  M <= 16: skinny.  Otherwise the fastest tile, with or
// without a pad, so that a pad changes its residency and nothing else.  Where the
// tile does not fit beside the pad, the fastest one that does takes its place, but
// only up to the pads that the largest of 256x256, 128x128 and 64x64 that gives a
// 256x256 tile per CU or a 128x128 one per two CUs leaves room for: larger pads
// are refused (a pad asks for a residency; it is never clamped, nor met by an ever
// smaller tile).  A K or N beyond what the chosen tile addresses with 32-bit
// offsets takes the 64x64 tile.  A K beyond that one's takes the register-staged
// opt2 tile (B N x K) or is refused (K x N), also where a 32x32 tile would reach it.
int auto_variant(const GemmCall &c, const DeviceInfo &di) {
  const int M = c.M, N = c.N, K = c.K;
  const bool b_kn = c.b_kn;
  if (M <= 16) {
    if (b_kn) return 33;
    // A kept in registers and B staged through LDS when K is whole
    // 1024-wide slices that fit, else 8 k-blocks of A and B in flight per lane
    if (K >= 1024 && K % 1024 == 0 && K <= 8192) return 34;
    return 21;
  }
  const int large = b_kn ? 32 : 16, mid = b_kn ? 35 : 14, small = b_kn ? 39 : 9;
  auto addressable = [&](int v) {
    if (K > find_variant(small)->kmax) return b_kn ? small : 7;
    const Variant *pv = find_variant(v);
    return (pv->kmax > 0 && K > pv->kmax) || (pv->nmax > 0 && N > pv->nmax) ? small : v;
  };
  int v = addressable(fastest_tile(c, di.num_cus, di.max_lds_per_wg));
  if (c.lds_bytes > 0 && c.lds_bytes <= (size_t)di.max_lds_per_wg) {
    const int room = di.max_lds_per_wg - (int)c.lds_bytes;
    auto fits = [&](int id) { return find_variant(id)->lds <= room; };
    const long long big = (long long)ceil_div(M, 256) * ceil_div(N, 256);
    const long long mids = (long long)ceil_div(M, 128) * ceil_div(N, 128);
    const int by_count = addressable(big >= di.num_cus ? large : (mids >= di.num_cus / 2 ? mid : small));
    if (!fits(v) && fits(by_count)) {
      v = fastest_tile(c, di.num_cus, room);
      v = v != 0 && fits(addressable(v)) ? addressable(v) : by_count;
    }
  }
  return v;
}

}  // namespace

bool gemm_variant_is_kn(int id) {
  const Variant *v = find_variant(id);
  return v != nullptr && v->b_kn;
}

static int fill_plan(const GemmCall &c, int variant, const DeviceInfo &di, occ_gemm_plan *p) {
  const Variant *v = variant_form(c, variant, di.num_cus);
  if (v == nullptr) return OCC_EINVAL;
  const bool skinny = is_skinny(v);
  if (skinny && c.M > 16) return OCC_EINVAL;
  if (v->kmax > 0 && c.K > v->kmax) return OCC_EINVAL;
  if (v->kmult > 0 && (c.K == 0 || c.K % v->kmult != 0)) return OCC_EINVAL;
  if (v->b_kn != c.b_kn) return OCC_EINVAL;  // the variant reads B in the other layout
  if (v->nmax > 0 && c.N > v->nmax) return OCC_EINVAL;
  if (v->id < 0 || v->id > kMaxVariantId) return OCC_EINVAL;
  p->tile_m = v->bm;
  p->tile_n = v->bn;
  p->tile_k = v->bk;
  p->threads = v->threads;
  p->tile_lds_bytes = v->lds;
  p->tiles = skinny ? ceil_div(c.N, v->bn) : ceil_div(c.M, v->bm) * ceil_div(c.N, v->bn);
  p->grid = p->tiles;
  const int skinny_grid = di.num_cus * (v->per_cu > 0 ? v->per_cu : 1);
  if (skinny && p->grid > skinny_grid) p->grid = skinny_grid;  // persistent
  if (c.grid_cap > 0 && c.grid_cap < p->grid) p->grid = c.grid_cap;
  p->max_lds_per_wg = di.max_lds_per_wg;
  p->lds_per_cu = di.lds_per_cu;
  p->num_cus = di.num_cus;
  p->kernel_id = variant;
  p->wg_per_cu = 0;
  if (c.lds_bytes > (size_t)di.max_lds_per_wg ||
      (size_t)v->lds + c.lds_bytes > (size_t)di.max_lds_per_wg)
    return OCC_ELDS;
  return OCC_OK;
}

// The launch plan without the occupancy figure: all a launch needs (the
// occupancy query costs host time on every call, which launch-bound
// schedules cannot spare).
int gemm_launch_plan(const GemmCall &c, occ_gemm_plan *plan) {
  const DeviceInfo *di = nullptr;
  int st = current_device_info(&di);
  if (st != OCC_OK) return st;
  int variant = c.variant;
  if (variant == 0) variant = auto_variant(c, *di);
  return fill_plan(c, variant, *di, plan);
}

int gemm_plan(const GemmCall &c, occ_gemm_plan *plan) {
  int st = gemm_launch_plan(c, plan);
  if (st != OCC_OK) return st;
  const Variant *v = variant_form(c, plan->kernel_id, plan->num_cus);
  int dyn = (int)(v->fn ? v->lds + c.lds_bytes : c.lds_bytes);
  int nb = 0;
  hipError_t e = v->fn ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, v->fn, v->threads, dyn)
                       : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, v->skinny, v->threads, dyn);
  if (e != hipSuccess) return OCC_EHIP;
  plan->wg_per_cu = nb;
  return OCC_OK;
}

int gemm_launch(const GemmCall &c, hipStream_t s) {
  occ_gemm_plan p;
  int st = gemm_launch_plan(c, &p);
  if (st != OCC_OK) return st;
  if (c.M == 0 || c.N == 0) return OCC_OK;
  const Variant *v = variant_form(c, p.kernel_id, p.num_cus);
  const uint16_t *A = static_cast<const uint16_t *>(c.A);
  const uint16_t *B = static_cast<const uint16_t *>(c.B);
  uint16_t *C = static_cast<uint16_t *>(c.C);
  // the dynamic-LDS limit is a per-device attribute of each kernel: set it
  // once per device and variant
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return OCC_ENODEV;
  if (v->fn) {
    int dyn = v->lds + (int)c.lds_bytes;
    int tiles_m = ceil_div(c.M, v->bm), tiles_n = ceil_div(c.N, v->bn);
    // B read by one workgroup only and too large to stay cached: non-temporal
    const bool nt = v->fn_nt != nullptr && tiles_m == 1 && b_exceeds_llc(c.N, c.K);
    const bool through = c.trace.release && v->fn_through != nullptr;
    const TiledFn fn = nt ? v->fn_nt : through ? v->fn_through : v->fn;
    static bool attr_set[kMaxDevices][kMaxVariantId + 1][2] = {};
    const int form = nt || through;  // a variant has at most one of the two
    if (!attr_set[dev][v->id][form]) {
      if (hipFuncSetAttribute(reinterpret_cast<const void *>(fn),
                              hipFuncAttributeMaxDynamicSharedMemorySize,
                              p.max_lds_per_wg) != hipSuccess)
        return OCC_EHIP;
      attr_set[dev][v->id][form] = true;
    }
    hipLaunchKernelGGL(fn, dim3(p.grid), dim3(v->threads), dyn, s, A, B, C, c.M, c.N, c.K,
                       tiles_m, tiles_n, c.priority, c.trace);
  } else {
    // the attribute matters to pads only
    const bool through = c.trace.release && v->skinny_through != nullptr;
    const SkinnyFn fn = through ? v->skinny_through : v->skinny;
    const int width = v->bn >= 128 ? 0 : v->bn >= 64 ? 1 : 2;  // variant 33's forms
    static bool attr_set_skinny[kMaxDevices][kMaxVariantId + 1][2][3] = {};
    if (c.lds_bytes > 0 && !attr_set_skinny[dev][v->id][through][width]) {
      if (hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                              p.max_lds_per_wg - v->lds) != hipSuccess)
        return OCC_EHIP;
      attr_set_skinny[dev][v->id][through][width] = true;
    }
    hipLaunchKernelGGL(fn, dim3(p.grid), dim3(v->threads), (int)c.lds_bytes, s, A, B, C, c.M, c.N, c.K,
                       c.priority, c.trace);
  }
  return hipGetLastError() == hipSuccess ? OCC_OK : OCC_EHIP;
}

}  // namespace occ
