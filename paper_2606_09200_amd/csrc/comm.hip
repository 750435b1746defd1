// K_c: one GPU's local share of a collective (Background, item 2).
//
//   share_reduce  -- allreduce share: fixed-order binary32 sum of the chunks.
//   share_permute -- alltoall share: gather of whole chunks by a permutation.
//
// Both are HBM-bound streams: 16-byte non-temporal loads and stores (so the
// stream does not evict the concurrently running GEMM's operands from L2),
// several independent loads in flight per lane, and a grid that is a knob
// (communication kernels are meant to be light, Section 3.1).  The comm
// kernel's wave priority is raised with s_setprio when asked: that is how the
// collective is given precedence over co-resident GEMM waves (Section 3.3).
#include "device_util.h"
#include "occ_internal.h"

#include <string.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace occ {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// the same at the alignment of their elements (one load or store all the same)
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4_a1 __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x2_a2 __attribute__((ext_vector_type(2), aligned(2)));

// bf16 bit pattern -> binary32 (exact: the bf16 bits are the high half)
__device__ __forceinline__ float widen_bf16(uint32_t bits16) { return __builtin_bit_cast(float, bits16 << 16); }

// One own term, read at device scope (see reduce_vec_kernel).
__device__ __forceinline__ float widen_own(const uint16_t *p) {
  return widen_bf16(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Workgroup sizes.  The chunk sum runs two waves per workgroup: at the
// default grid of one workgroup per CU, two of a CU's four SIMDs carry a comm
// wave.  Measured on MI355X against four waves per workgroup: the isolated
// 8-term sum is 8 % faster, and the overlapped schedules are 1.5-8 % shorter
// (8192^3 with 8 x 128 MiB, the same with the own term, and 16 x 28672 x 8192
// with 8 x 64 MiB, at both comm priorities); one wave per workgroup slows the
// isolated sum by 40 % and lengthens the decode-like schedule.  The
// permutation also runs two waves, with twice the loads in flight per lane
// of a four-wave workgroup (kPermuteUnroll): against four waves it is 0.5-1 %
// faster alone and never slower overlapped (8192^3 with 4 x 224 MiB: 0.3-0.9 %
// shorter).
constexpr int kReduceThreads = 128;
constexpr int kPermuteThreads = 128;

struct ChunkPtrs {
  const float *p[kMaxReduceChunks];
};

// Chunk sum.  Element j's sum is acc = c0[j]; acc = acc + c1[j]; ... exactly
// in chunk order; the loads of all chunks for UNROLL positions are issued
// before any addition.  A position is 4 elements, loaded with one 16-byte load
// per chunk at the element's own 4-byte alignment: chunks are often rows of
// one buffer, and with an odd row length each starts at another offset from a
// 16-byte boundary (a misaligned wave reads 9 lines instead of 8).  The
// launcher starts positions where `out` is 16-byte aligned; the elements before
// and after (`head` and the remainder, at most 6) go to the last workgroup's
// first lanes.
//
// What bounds it is bytes in flight: the default grid is one workgroup of two
// waves per CU, so a lane needs 8-16 loads outstanding.  NC >= 0 (the number
// of fp32 chunks) therefore has its own instantiation for every term count up
// to 16, with UNROLL from reduce_unroll; NC < 0 folds `nchunks` chunks in
// batches of 8 loads.  Measured on MI355X at 0.5 GB of chunks, 256 workgroups:
// batches of 8 reach 2.7 / 3.5 / 3.8 / 3.6 TB/s with 3 / 5 / 6 / 12 terms, the
// exact counts 5.5-6.2; 6 x 11 000 003 as rows of one buffer took 700 us an
// element at a time and takes 54.  At most 64 VGPRs: what the 256x256 GEMM's
// two waves leave of a SIMD's 512, so that both fit on one CU.
//
// OWN: the first term is a bf16 buffer (this GPU's own contribution, e.g. its
// GEMM output), widened exactly to binary32; the chunks follow it in order.
// Its 8 bytes per position are one load, of device scope (kOwnDevice: the GEMM
// that wrote them may have ended on another XCD while this kernel waited for
// it, KHooks; the buffer is then 8-byte aligned) or an ordinary one at 2-byte
// alignment (kOwnPlain).  The scope costs a sum that waits for nothing nothing, so
// it has no form of its own: 7 peers x 2^24 97.8 us at device scope, 98.2 with
// ordinary loads, 2^16 2.25 and 2.28; 1 peer x 2^24 30.4 and 30.2.
enum { kOwnNone = 0, kOwnDevice = 1, kOwnPlain = 2 };

template <int NC, int UNROLL, bool OFF32, int OWN>
__global__ __launch_bounds__(kReduceThreads) void reduce_vec_kernel(ChunkPtrs cp, int nchunks, size_t nvec,
                                                                    float *__restrict__ out,
                                                                    const uint16_t *__restrict__ own, int head,
                                                                    int tail, int prio, uint32_t pace, KHooks tr) {
  // OFF32: every byte offset the loop forms fits in 32 bits (checked by the
  // host), so each access is a scalar base plus one shared 32-bit lane
  // offset instead of a 64-bit address per chunk: fewer vector instructions
  // per byte, which is issue time a co-running GEMM on the same SIMD gets back.
  using I = typename std::conditional<OFF32, uint32_t, size_t>::type;
  set_wave_priority(prio);
  const HookStart t0 = hooks_begin(tr);
  Pacer pc = pace_start(pace);
  const I n = (I)nvec;
  const I stride = (I)gridDim.x * kReduceThreads;
  I i = (I)blockIdx.x * kReduceThreads + threadIdx.x;
  auto ld = [&](int c, I k) {
    return __builtin_nontemporal_load(
        reinterpret_cast<const f32x4_a4 *>(reinterpret_cast<const char *>(cp.p[c]) + k * (I)sizeof(f32x4)));
  };
  auto st = [&](f32x4 v, I k) {
    __builtin_nontemporal_store(v, reinterpret_cast<f32x4_a4 *>(reinterpret_cast<char *>(out) + k * (I)sizeof(f32x4)));
  };
  auto ld_own = [&](I k) {
    const char *p = reinterpret_cast<const char *>(own) + k * (I)sizeof(uint64_t);
    u32x2 w;
    if constexpr (OWN == kOwnDevice) {
      const uint64_t d = __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
      w = u32x2{(uint32_t)d, (uint32_t)(d >> 32)};
    } else {
      w = __builtin_nontemporal_load(reinterpret_cast<const u32x2_a2 *>(p));
    }
    f32x4 r;
    r[0] = widen_bf16(w[0] & 0xFFFFu);
    r[1] = widen_bf16(w[0] >> 16);
    r[2] = widen_bf16(w[1] & 0xFFFFu);
    r[3] = widen_bf16(w[1] >> 16);
    return r;
  };
  auto add = [](f32x4 a, f32x4 b) {
    a[0] = a[0] + b[0];
    a[1] = a[1] + b[1];
    a[2] = a[2] + b[2];
    a[3] = a[3] + b[3];
    return a;
  };
  constexpr int C0 = OWN ? 0 : 1;  // first fp32 chunk added to the first term

  if constexpr (NC >= 0) {
    auto trip = [&](auto positions) {
      constexpr int U = decltype(positions)::value;
      f32x4 v[NC > 0 ? NC : 1][U], o[U];
      if constexpr (OWN) {
#pragma unroll
        for (int u = 0; u < U; ++u) o[u] = ld_own(i + u * stride);
      }
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int u = 0; u < U; ++u) v[c][u] = ld(c, i + u * stride);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        f32x4 acc = OWN ? o[u] : v[0][u];
#pragma unroll
        for (int c = C0; c < NC; ++c) acc = add(acc, v[c][u]);
        st(acc, i + u * stride);
      }
    };
    for (bool first = true; i + (UNROLL - 1) * stride < n; i += UNROLL * stride, first = false) {
      if (!first) pace_wait(pc);
      trip(std::integral_constant<int, UNROLL>{});
    }
    if constexpr (UNROLL > 1)
      for (; i < n; i += stride) trip(std::integral_constant<int, 1>{});
  } else {
    // chunk count known at run time: batches of 8 loads, folded in order
    for (bool first = true; i < n; i += stride, first = false) {
      if (!first) pace_wait(pc);
      f32x4 acc = OWN ? ld_own(i) : ld(0, i);
      for (int c0 = C0; c0 < nchunks; c0 += 8) {
        f32x4 v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c)
          if (c0 + c < nchunks) v[c] = ld(c0 + c, i);
#pragma unroll
        for (int c = 0; c < 8; ++c)
          if (c0 + c < nchunks) acc = add(acc, v[c]);
      }
      st(acc, i);
    }
  }
  if (blockIdx.x == gridDim.x - 1 && (int)threadIdx.x < head + tail) {
    const ptrdiff_t j = (int)threadIdx.x < head ? (ptrdiff_t)threadIdx.x - head
                                                : (ptrdiff_t)(nvec * 4) + (ptrdiff_t)threadIdx.x - head;
    float acc = OWN ? widen_own(own + j) : cp.p[0][j];
    for (int c = C0; c < nchunks; ++c) acc = acc + cp.p[c][j];
    out[j] = acc;
  }
  if (pace != 0) {
    // the positions of this workgroup's first lane, and one for the elements above
    const size_t first = (size_t)blockIdx.x * kReduceThreads, step = (size_t)gridDim.x * kReduceThreads;
    const size_t positions = (first < nvec ? (nvec - first + step - 1) / step : 0) +
                             (blockIdx.x == gridDim.x - 1 && head + tail > 0 ? 1 : 0);
    pace_until(pc.start + pace_share(pace, positions, UNROLL));
  }
  hooks_end(tr, t0);
}

struct PermTable {
  int32_t p[kMaxPermuteChunks];
};

// Permutation copy.  Work item w covers part (w % parts) of destination chunk
// (w / parts); workgroups stride over work items, threads over the part's
// 16-byte units with UNROLL loads in flight before the stores (also in a part's
// last, partial round).  Units start where the destination chunk reaches a
// 16-byte boundary, so stores are aligned whatever the chunk size; ALIGNED
// (src, dst and chunk_bytes multiples of 16) lets the loads be aligned too.
// Otherwise loads have the source's own byte alignment, and the fewer than 32
// bytes before and after the units are copied by the last part's first lanes.
// Measured on MI355X: 24 x 5 000 002 bytes took 897 us a byte per lane and takes
// 51, against 46 at the rate of a 16-byte multiple.
template <int UNROLL, bool OFF32, bool ALIGNED>
__global__ __launch_bounds__(kPermuteThreads) void permute_vec_kernel(const char *__restrict__ src,
                                                                      char *__restrict__ dst, PermTable pt,
                                                                      int nchunks, size_t chunk_bytes, int parts,
                                                                      int prio, uint32_t pace, KHooks tr) {
  // OFF32: offsets inside a chunk fit in 32 bits (checked by the host): the
  // work item's chunk bases are scalar and the lanes share one 32-bit offset.
  using I = typename std::conditional<OFF32, uint32_t, size_t>::type;
  typedef typename std::conditional<ALIGNED, u32x4, u32x4_a1>::type Unit;
  set_wave_priority(prio);
  const HookStart t0 = hooks_begin(tr);
  // Pacing: a full round of a part waits for the one before it, and the next part (or
  // the kernel's end) for the time of all bytes of this one, partial round included.
  uint64_t part_end = 0;
  const int nwork = nchunks * parts;
  for (int w = blockIdx.x; w < nwork; w += gridDim.x) {
    const int chunk = w / parts;
    const int part = w - chunk * parts;
    const char *s = src + (size_t)pt.p[chunk] * chunk_bytes;
    char *d = dst + (size_t)chunk * chunk_bytes;
    size_t cvec = chunk_bytes / 16;
    uint32_t edge_units = 0;  // the bytes outside the units, for the pacing
    if constexpr (!ALIGNED) {
      size_t head = (16 - (reinterpret_cast<uintptr_t>(d) & 15)) & 15;
      if (head > chunk_bytes) head = chunk_bytes;
      cvec = (chunk_bytes - head) / 16;
      const size_t edge = chunk_bytes - cvec * 16;  // bytes outside the units
      if (part == parts - 1 && threadIdx.x < edge) {
        const size_t b = threadIdx.x < head ? threadIdx.x : cvec * 16 + threadIdx.x;
        d[b] = s[b];
      }
      if (part == parts - 1) edge_units = (uint32_t)(edge + 15) / 16;
      s += head;
      d += head;
    }
    const I lo = (I)(cvec * part / parts);
    const I hi = (I)(cvec * (part + 1) / parts);
    Pacer pc = pace_start(pace, part_end);
    if (pace != 0) part_end = pc.start + pace_share(pace, (uint64_t)(hi - lo) + edge_units, UNROLL * kPermuteThreads);
    bool first = true;
    auto ld = [&](I k) { return __builtin_nontemporal_load(reinterpret_cast<const Unit *>(s + k * (I)16)); };
    auto st = [&](u32x4 v, I k) { __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(d + k * (I)16)); };
    I i = lo + threadIdx.x;
    u32x4 v[UNROLL];
    for (; i + (UNROLL - 1) * kPermuteThreads < hi; i += UNROLL * kPermuteThreads) {
      if (!first) pace_wait(pc);
      first = false;
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) v[u] = ld(i + u * kPermuteThreads);
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) st(v[u], i + u * kPermuteThreads);
    }
    if (i < hi) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
        if (i + u * kPermuteThreads < hi) v[u] = ld(i + u * kPermuteThreads);
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
        if (i + u * kPermuteThreads < hi) st(v[u], i + u * kPermuteThreads);
    }
  }
  if (pace != 0) pace_until(part_end);
  hooks_end(tr, t0);
}

__global__ void stamps_reset_kernel(uint64_t *stamps, int npairs, uint32_t *wg) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (stamps != nullptr && i < npairs) {
    stamps[2 * i] = ~0ull;
    stamps[2 * i + 1] = 0ull;
  }
  if (wg != nullptr && i == 0) wg[0] = 0u;
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// At most one workgroup per `threads` work units, at least one.
int clamp_wgs(size_t work_units, int wanted, int threads) {
  size_t cap = (work_units + threads - 1) / threads;
  if (cap < 1) cap = 1;
  return (int)(wanted < (long long)cap ? wanted : cap);
}

// Positions per lane per trip of the vector chunk sum for a number of terms
// (fp32 chunks plus the own term); the launch table and the pacing period
// both take it from here.  8-16 loads in flight per lane (a single term 4), as far
// as 64 VGPRs hold them; 64-bit offsets need registers of their own.
constexpr int kExactTerms = 16;  // term counts with an instantiation of their own
constexpr bool exact_terms(int terms, bool off32) {
  return off32 ? terms <= kExactTerms : (terms == 2 || terms == 4 || terms == 8 || terms == 16);
}
constexpr int reduce_unroll(int terms, bool off32) {
  if (!exact_terms(terms, off32)) return 1;
  return terms <= 3 ? 4 : terms == 4 ? 2 : (terms <= 8 && off32) ? 2 : 1;
}

// Loads in flight per lane of the vector permutation (launch, pacing and the
// 32-bit offset check).  With four-wave workgroups 2 and 8 gave no shorter
// overlapped schedule than 4 (16384x14336x4096 with 64 x 4 MiB, 8192^3 with
// 4 x 224 MiB); the two-wave workgroups take 8, the same bytes per CU.
constexpr int kPermuteUnroll = 8;

// Period (10 ns ticks, rounded up) a wave's trip takes at least, so that the whole
// grid moves trip_bytes per period, i.e. streams at rate_gbs; 0 = unpaced.
uint32_t pace_ticks(double trip_bytes, double rate_gbs) {
  if (!(rate_gbs > 0.0)) return 0;
  double t = std::ceil(trip_bytes / (rate_gbs * 1e9) * 1e8);
  if (t < 1.0) t = 1.0;
  if (t > 4.0e9) t = 4.0e9;
  return (uint32_t)t;
}

}  // namespace

// Launch with the instantiation of c.nchunks (+ own) terms, T counting up.
template <bool OFF32, int OWN, int T = 1>
void launch_reduce(int nchunks, int g, hipStream_t s, const ChunkPtrs &cp, size_t nvec, float *out,
                   const uint16_t *own, int head, int tail, int prio, uint32_t pace, const KHooks &tr) {
  if constexpr (T > kExactTerms) {
    hipLaunchKernelGGL((reduce_vec_kernel<-1, 1, OFF32, OWN>), dim3(g), dim3(kReduceThreads), 0, s, cp, nchunks, nvec,
                       out, own, head, tail, prio, pace, tr);
  } else {
    if constexpr (exact_terms(T, OFF32)) {
      if (nchunks + (OWN ? 1 : 0) == T) {
        hipLaunchKernelGGL((reduce_vec_kernel<T - (OWN ? 1 : 0), reduce_unroll(T, OFF32), OFF32, OWN>), dim3(g),
                           dim3(kReduceThreads), 0, s, cp, nchunks, nvec, out, own, head, tail, prio, pace, tr);
        return;
      }
    }
    launch_reduce<OFF32, OWN, T + 1>(nchunks, g, s, cp, nvec, out, own, head, tail, prio, pace, tr);
  }
}

int reduce_default_wgs(const ReduceCall &c) {
  const DeviceInfo *di = nullptr;
  int cus = current_device_info(&di) == OCC_OK ? di->num_cus : 256;
  return clamp_wgs(c.len / 4 + 1, cus, kReduceThreads);
}

int reduce_launch(const ReduceCall &c, hipStream_t s) {
  if (c.len == 0) return OCC_OK;
  ChunkPtrs cp;
  memset(&cp, 0, sizeof cp);
  const bool own = c.own != nullptr;
  const int wgs = c.wgs > 0 ? c.wgs : reduce_default_wgs(c);
  const int prio = c.priority;
  // a dependency wait is acknowledged by every workgroup of the kernel
  KHooks tr = c.trace;
  // positions start at out's first 16-byte boundary; with an own term at
  // element 0, which keeps its 8-byte loads aligned
  size_t head = own ? 0 : ((16 - (reinterpret_cast<uintptr_t>(c.out) & 15)) & 15) / 4;
  if (head > c.len) head = c.len;
  for (int i = 0; i < c.nchunks; ++i) cp.p[i] = c.bufs[i] + head;
  const size_t nvec = (c.len - head) / 4;
  const int tail = (int)(c.len - head - nvec * 4);
  const int g = clamp_wgs(nvec, wgs, kReduceThreads);
  if (tr.wait != nullptr) tr.ack_target = (uint32_t)g;
  const int terms = c.nchunks + (own ? 1 : 0);
  // 32-bit offsets when the largest byte offset the loop can form, (nvec
  // plus one unrolled grid stride) * 16, stays below 2^32
  const bool off32 = ((double)nvec + 4.0 * g * kReduceThreads) * 16.0 < 4294967296.0;
  // the bytes one position moves
  const double pos_bytes = 16.0 * (c.nchunks + 1) + (own ? 8.0 : 0.0);
  const uint32_t pace = pace_ticks((double)g * kReduceThreads * reduce_unroll(terms, off32) * pos_bytes, c.rate_gbs);
  float *out = c.out + head;
  auto launch = [&](auto mode) {
    constexpr int OWN = decltype(mode)::value;
    if (off32) launch_reduce<true, OWN>(c.nchunks, g, s, cp, nvec, out, c.own, (int)head, tail, prio, pace, tr);
    else launch_reduce<false, OWN>(c.nchunks, g, s, cp, nvec, out, c.own, (int)head, tail, prio, pace, tr);
  };
  if (!own) launch(std::integral_constant<int, kOwnNone>{});
  else if ((reinterpret_cast<uintptr_t>(c.own) & 7u) == 0) launch(std::integral_constant<int, kOwnDevice>{});
  else launch(std::integral_constant<int, kOwnPlain>{});
  return hipGetLastError() == hipSuccess ? OCC_OK : OCC_EHIP;
}

// Parts per chunk for `wgs` workgroups: parts of at most 256 KiB and, unless
// the chunk is smaller, at least 16 KiB (one round of a workgroup's loads),
// their number the one that leaves the workgroups the least to do one after
// another (rounds of items x part size; a 257th item on 256 workgroups would
// double it).  4 x 17 MiB: 272 items of 256 KiB on 256 workgroups take 37.3 us,
// 512 of 136 KiB 28.9.
static int permute_parts(const PermuteCall &c, int wgs) {
  const size_t kMin = 16u << 10, kMax = 256u << 10;
  size_t lo = (c.chunk_bytes + kMax - 1) / kMax, hi = c.chunk_bytes / kMin;
  lo = std::min<size_t>(std::max<size_t>(lo, 1), 4096);
  // enough items for every workgroup, and as many candidates again for a better fit
  const size_t fill = ((size_t)wgs + c.nchunks - 1) / c.nchunks;
  hi = std::min(std::max(hi, lo), std::max(2 * lo, 2 * fill));
  // from 16 rounds on a partial last one costs too little to look further
  if (lo * c.nchunks >= (size_t)wgs * 16) return (int)lo;
  size_t best = lo, best_rounds = 0;
  for (size_t p = lo; p <= hi; ++p) {
    const size_t rounds = (c.nchunks * p + wgs - 1) / wgs;
    if (best_rounds == 0 || rounds * best < best_rounds * p) {
      best = p;
      best_rounds = rounds;
    }
  }
  return (int)best;
}

// One workgroup per CU, fewer for short inputs.
int permute_default_wgs(const PermuteCall &c) {
  const DeviceInfo *di = nullptr;
  const int cus = current_device_info(&di) == OCC_OK ? di->num_cus : 256;
  return (int)std::min<long long>((long long)c.nchunks * permute_parts(c, cus), cus);
}

int permute_launch(const PermuteCall &c, hipStream_t s) {
  if (c.chunk_bytes == 0) return OCC_OK;
  PermTable pt;
  memset(&pt, 0, sizeof pt);
  for (int i = 0; i < c.nchunks; ++i) pt.p[i] = c.perm[i];
  const int wgs = c.wgs > 0 ? c.wgs : permute_default_wgs(c);
  const int parts = permute_parts(c, wgs);
  const int g = (int)std::min<long long>(wgs, (long long)c.nchunks * parts);
  KHooks tr = c.trace;
  if (tr.wait != nullptr) tr.ack_target = (uint32_t)g;
  const uint32_t pace = pace_ticks((double)g * kPermuteThreads * kPermuteUnroll * 16.0 * 2.0, c.rate_gbs);
  const bool aligned = aligned16(c.src) && aligned16(c.dst) && c.chunk_bytes % 16 == 0;
  // 32-bit offsets when a chunk plus one unrolled block stays below 2^32 bytes
  const bool off32 = (double)c.chunk_bytes + (double)kPermuteUnroll * kPermuteThreads * 16.0 < 4294967296.0;
  auto fn = off32 ? (aligned ? permute_vec_kernel<kPermuteUnroll, true, true> : permute_vec_kernel<kPermuteUnroll, true, false>)
                  : (aligned ? permute_vec_kernel<kPermuteUnroll, false, true> : permute_vec_kernel<kPermuteUnroll, false, false>);
  hipLaunchKernelGGL(fn, dim3(g), dim3(kPermuteThreads), 0, s, static_cast<const char *>(c.src),
                     static_cast<char *>(c.dst), pt, c.nchunks, c.chunk_bytes, parts, c.priority, pace, tr);
  return hipGetLastError() == hipSuccess ? OCC_OK : OCC_EHIP;
}

int trace_reset(uint64_t *stamps, int npairs, uint32_t *wg, hipStream_t s) {
  if (stamps == nullptr && wg == nullptr) return OCC_OK;
  int n = npairs > 1 ? npairs : 1;
  hipLaunchKernelGGL(stamps_reset_kernel, dim3((n + 255) / 256), dim3(256), 0, s, stamps, npairs, wg);
  return hipGetLastError() == hipSuccess ? OCC_OK : OCC_EHIP;
}

}  // namespace occ
