// tpcca_kernels.hip -- the tracking path on gfx950.
//
// Paper, Sec. "Track reconstruction in the TPC": cellular-automaton seeding
// with one thread per cluster, Kalman-filter following with one thread per
// track, every sector independent.  Here every (event, sector) pair is an
// independent unit, so one launch of each phase covers all events of a
// batch.  Phases:
//   a1 binning    count per (event, sector, row) -> scan -> bucket -> per
//                 row: sort by id in LDS, canonical SoA, 2-D (z, y) grid
//   a2 links      one lane per cluster, windows on the adjacent rows' grids
//   a3/a4         reciprocal-link cleaning, start and seed flags, wave ballot
//                 compaction in canonical (event, sector, row, id) order
//   a5 tracklets  one lane per seed: chain fit, upward and downward
//                 following with grid searches
//   a6 selection  64-bit atomicMax ownership per cluster
//   a7 final fit  outermost-to-innermost Kalman refit of the owned hits,
//                 ordered compaction into the caller's flat buffers
#include <algorithm>
#include <type_traits>

#include "internal.hpp"
#include "kf_c2.hpp"

namespace tpcca {
namespace {

constexpr int TB = 256;
constexpr int kXcd = 8;   // accelerator complex dies (each with its own L2) of the chip
constexpr int kBackRows = 32;   // longest transport (rows) back to a seed's first row
constexpr int kRefillMin = 16;  // waiting lanes that make a wave take new seeds

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, kCtrl, 0xF, 0xF, true);
}
template <int kCtrl>
__device__ __forceinline__ float dpp_f32(float v) { return __uint_as_float(dpp_u32<kCtrl>(__float_as_uint(v))); }
// Lane exchanges inside groups of two, four and eight lanes (the last one
// mirrors the eight: enough once each four hold one value).
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppMirror8 = 0x141;
constexpr int kDppRor4 = 0x124, kDppRor8 = 0x128;   // rotations inside rows of 16 lanes

// Row shifts inside 16 lanes, then the last lane of a row (of the first two
// rows) to the rows behind it: six adds, no LDS crossbar.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += dpp_u32<0x111>(v);
  v += dpp_u32<0x112>(v);
  v += dpp_u32<0x114>(v);
  v += dpp_u32<0x118>(v);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
  return v;
}

// Exclusive scan over a 256-thread block; *tot receives the block total.
__device__ uint32_t block_excl_scan(uint32_t v, uint32_t* tot) {
  __shared__ uint32_t s_w[TB / 64];
  const uint32_t inc = wave_incl_scan(v);
  const int wid = threadIdx.x >> 6;
  if (lane_id() == 63) s_w[wid] = inc;
  __syncthreads();
  uint32_t base = 0, total = 0;
#pragma unroll
  for (int i = 0; i < TB / 64; ++i) {
    const uint32_t t = s_w[i];
    if (i < wid) base += t;
    total += t;
  }
  __syncthreads();
  *tot = total;
  return base + inc - v;
}

__device__ __forceinline__ uint64_t lanemask_lt() { return (1ull << lane_id()) - 1ull; }

// ---------------------------------------------------------------- utilities
__global__ void k_fill(uint32_t* __restrict__ p, uint32_t v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x; i < n; i += (int64_t)gridDim.x * TB) p[i] = v;
}

// Two ranges cleared by one launch.
__global__ void k_zero2(uint32_t* __restrict__ p, int64_t n, uint32_t* __restrict__ q, int64_t m) {
  for (int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x; i < n + m; i += (int64_t)gridDim.x * TB) {
    if (i < n) p[i] = 0u;
    else q[i - n] = 0u;
  }
}

// Exclusive scans, out[n] = total (out may equal in).  Up to two arrays of
// the same length are scanned by the same launches (blockIdx.y selects the
// array): one workgroup each when n <= kScanSmall, else reduce / partials /
// down-sweep over tiles of 1024.
struct ScanArgs {
  const uint32_t* in[2];
  uint32_t* out[2];
  int ind[2];   // 1: scan the indicator (value > 0) of the input instead of the value
};
__device__ __forceinline__ uint32_t scan_in(const ScanArgs& a, int y, uint32_t v) {
  return a.ind[y] ? (v > 0u ? 1u : 0u) : v;
}
constexpr int kScanNT = 1024;                        // threads of a one-workgroup scan
constexpr int64_t kScanSmall = 4 * 4 * kScanNT;      // at most four tiles of 4 x kScanNT

// Size classes of row units.  The row and link kernels come in variants by
// row size; with few row units (RU <= kScanSmall, e.g. one event) each
// variant's launch covers every row unit and skips the others, with many
// (batches of events) the binning builds one list per variant and the
// variants other than the wave-per-unit ones run over their list only, so
// that the hundreds of thousands of mostly tiny units of a batch do not
// each cost a workgroup launch in every variant.
constexpr uint32_t kTiny = 64;         // clusters of a row unit handled by one wave, one per lane
constexpr uint32_t kWaveRow = 256;     // clusters of a row unit handled by one wave, four per lane
constexpr uint32_t kSlab = 896;        // clusters of one row staged in LDS (3 workgroups per CU fit)
__host__ __device__ inline bool ru_lists(int64_t RU) { return RU > kScanSmall; }
// 0: k_rows_tiny (empty units too), 1: k_rows_wave, 2: k_rows<false>, 3: k_rows<true>
__device__ __forceinline__ int rows_class(uint32_t n) {
  return n <= kTiny ? 0 : n <= kWaveRow ? 1 : n <= 4u * TB ? 2 : 3;
}
// Workgroups of a list-driven launch (each loops over list entries).
constexpr unsigned kListGrid = 2048, kListGridBig = 1024;

// Exclusive scan over a kScanNT-thread block; *tot receives the block total.
__device__ uint32_t block_excl_scan_big(uint32_t v, uint32_t* tot) {
  __shared__ uint32_t s_w[kScanNT / 64];
  const uint32_t inc = wave_incl_scan(v);
  const int wid = threadIdx.x >> 6;
  if (lane_id() == 63) s_w[wid] = inc;
  __syncthreads();
  uint32_t base = 0, total = 0;
#pragma unroll
  for (int i = 0; i < kScanNT / 64; ++i) {
    const uint32_t t = s_w[i];
    if (i < wid) base += t;
    total += t;
  }
  __syncthreads();
  *tot = total;
  return base + inc - v;
}

__global__ __launch_bounds__(kScanNT) void k_scan_small(ScanArgs a, int64_t n) {
  const uint32_t* in = a.in[blockIdx.x];
  uint32_t* out = a.out[blockIdx.x];
  const uint32_t n32 = (uint32_t)n;   // n <= kScanSmall
  // tiles of four coalesced values per thread with a running carry; past
  // the end a thread reads element 0 and drops it (no branch around loads)
  uint32_t carry = 0;
  for (uint32_t t0 = 0; t0 < n32; t0 += 4u * kScanNT) {
    const uint32_t base = t0 + 4u * threadIdx.x;
    uint32_t v[4], sum = 0;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t x = scan_in(a, blockIdx.x, in[base + j < n32 ? base + j : 0u]);
      v[j] = base + j < n32 ? x : 0u;
      sum += v[j];
    }
    uint32_t tot;
    uint32_t ex = carry + block_excl_scan_big(sum, &tot);
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      if (base + j < n32) out[base + j] = ex;
      ex += v[j];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) out[n32] = carry;
}

// Row-unit offsets in one workgroup (RU <= kScanSmall): scans the counts
// into ru_off and the cell capacities (grid_cells(count) + 1, computed here)
// into cell_base, then clears the counts for their second use as the
// scatter's fill cursors.
__global__ __launch_bounds__(kScanNT) void k_scan_rows(Ws w) {
  const uint32_t n32 = (uint32_t)w.RU;
  uint32_t carry0 = 0, carry1 = 0;
  for (uint32_t t0 = 0; t0 < n32; t0 += 4u * kScanNT) {
    const uint32_t base = t0 + 4u * threadIdx.x;
    uint32_t v0[4], v1[4], s0 = 0, s1 = 0;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint32_t x = w.ru_count[base + j < n32 ? base + j : 0u];
      v0[j] = base + j < n32 ? x : 0u;
      v1[j] = base + j < n32 ? grid_cells(x) + 1u : 0u;
      s0 += v0[j];
      s1 += v1[j];
    }
    uint32_t tot0, tot1;
    uint32_t e0 = carry0 + block_excl_scan_big(s0, &tot0);
    uint32_t e1 = carry1 + block_excl_scan_big(s1, &tot1);
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      if (base + j < n32) {
        w.ru_off[base + j] = e0;
        w.cell_base[base + j] = e1;
        w.ru_count[base + j] = 0u;
      }
      e0 += v0[j];
      e1 += v1[j];
    }
    carry0 += tot0;
    carry1 += tot1;
  }
  if (threadIdx.x == 0) { w.ru_off[n32] = carry0; w.cell_base[n32] = carry1; }
}

__global__ __launch_bounds__(TB) void k_scan_reduce(ScanArgs a, int64_t n, uint32_t* __restrict__ part,
                                                    int64_t pstride) {
  const uint32_t* in = a.in[blockIdx.y];
  part += blockIdx.y * pstride;
  const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) if (base + j < n) s += scan_in(a, blockIdx.y, in[base + j]);
  uint32_t tot;
  block_excl_scan(s, &tot);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(TB) void k_scan_parts(uint32_t* __restrict__ part, int64_t np, int64_t pstride) {
  part += blockIdx.x * pstride;
  uint32_t carry = 0;
  for (int64_t b = 0; b < np; b += TB) {
    const int64_t i = b + threadIdx.x;
    const uint32_t v = i < np ? part[i] : 0u;
    uint32_t tot;
    const uint32_t ex = block_excl_scan(v, &tot);
    if (i < np) part[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) part[np] = carry;
}

__global__ __launch_bounds__(TB) void k_scan_down(ScanArgs a, int64_t n, const uint32_t* __restrict__ part,
                                                  int64_t np, int64_t pstride) {
  const uint32_t* in = a.in[blockIdx.y];
  uint32_t* out = a.out[blockIdx.y];
  part += blockIdx.y * pstride;
  const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  uint32_t v[4], s = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) { v[j] = base + j < n ? scan_in(a, blockIdx.y, in[base + j]) : 0u; s += v[j]; }
  uint32_t tot;
  uint32_t ex = block_excl_scan(s, &tot) + (blockIdx.x < np ? part[blockIdx.x] : 0u);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (base + j < n) out[base + j] = ex;
    ex += v[j];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = part[np];
}

// Exclusive scans of narr (1 or 2) arrays of n values; part holds
// 2 (n / 1024 + 2) values.
hipError_t scan_arrays(ScanArgs a, int narr, int64_t n, uint32_t* part, hipStream_t st) {
  if (n <= kScanSmall) {
    k_scan_small<<<dim3((unsigned)narr), dim3(kScanNT), 0, st>>>(a, n);
    return hipGetLastError();
  }
  const int64_t np = (n + 1023) / 1024;
  const int64_t ps = np + 2;
  k_scan_reduce<<<dim3((unsigned)np, (unsigned)narr), dim3(TB), 0, st>>>(a, n, part, ps);
  k_scan_parts<<<dim3((unsigned)narr), TB, 0, st>>>(part, np, ps);
  k_scan_down<<<dim3((unsigned)np, (unsigned)narr), dim3(TB), 0, st>>>(a, n, part, np, ps);
  return hipGetLastError();
}

hipError_t scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* part, hipStream_t st) {
  ScanArgs a{{in, in}, {out, out}, {0, 0}};
  return scan_arrays(a, 1, n, part, st);
}

// ind0: the first array is scanned as the indicator of its values.
hipError_t scan_u32x2(const uint32_t* in0, uint32_t* out0, const uint32_t* in1, uint32_t* out1, int64_t n,
                      uint32_t* part, hipStream_t st, int ind0 = 0) {
  ScanArgs a{{in0, in1}, {out0, out1}, {ind0, 0}};
  return scan_arrays(a, 2, n, part, st);
}

inline unsigned blocks_for(int64_t n, int64_t cap = 1 << 16) {
  int64_t b = (n + TB - 1) / TB;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (unsigned)b;
}

// A multiple of kXcd workgroups (at most 2^14) for kernels that split their
// work by XCD.
inline unsigned xcd_blocks(int64_t n) {
  const int64_t b = blocks_for(n, 1 << 14);
  return (unsigned)((b + kXcd - 1) / kXcd * kXcd);
}

// ------------------------------------------------------------- a1: binning
// Raw fields of one input cluster, then its validation and row unit.  The
// binning kernels take kGroup clusters per thread at a time and issue all
// their loads before the first is used.
struct RawCl { float x, y, z; int r, s; };

__device__ __forceinline__ RawCl load_cluster(const EventIn& E, int64_t l) {
  return RawCl{E.x[l], E.y[l], E.z[l], (int)E.row[l], (int)E.sector[l]};
}

__device__ __forceinline__ bool check_cluster(const Ws& w, const RawCl& c, int e, int64_t l, uint32_t& ru,
                                              float4& v) {
  if (!(isfinite(c.x) && isfinite(c.y) && isfinite(c.z)) || c.r < 0 || c.r >= w.R || c.s >= w.S) return false;
  ru = ((uint32_t)e * (uint32_t)w.S + (uint32_t)c.s) * (uint32_t)w.R + (uint32_t)c.r;
  v = make_float4(c.x, c.y, c.z, __uint_as_float((uint32_t)l));
  return true;
}

constexpr int kGroup = 4;
// threads of the binning workgroups: a chunk's clusters and bins are spread
// over sixteen waves, so the few hundred chunks of a large event still keep
// several waves on every SIMD
constexpr int TBB = 1024;

// f(ok, ru, v) for every cluster of the chunk [c0, c1) of event e taken by
// this thread (stride TBB), kGroup at a time.
template <class F>
__device__ __forceinline__ void for_chunk(const Ws& w, int64_t c0, int64_t c1, int e, F&& f) {
  const EventIn& E = w.ev[e];
  for (int64_t g0 = c0 + threadIdx.x; g0 < c1; g0 += (int64_t)kGroup * TBB) {
    RawCl c[kGroup];
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
      const int64_t g = g0 + (int64_t)k * TBB;
      if (g < c1) c[k] = load_cluster(E, g - E.base);
    }
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
      const int64_t g = g0 + (int64_t)k * TBB;
      if (g >= c1) continue;
      uint32_t ru = 0;
      float4 v;
      const bool ok = check_cluster(w, c[k], e, g - E.base, ru, v);
      f(ok, ru, v);
    }
  }
}

// Binning histograms are privatised in LDS per chunk (up to kChunkCl
// clusters of one event, from the host's chunk table): the bins are the
// event's row units.  Count: one global atomic per non-empty bin.  Scatter:
// one global range reservation per non-empty bin, then LDS ranks.
constexpr int kLdsBins = 8192;

__global__ __launch_bounds__(TBB) void k_count(Ws w) {
  __shared__ uint32_t s_h[kLdsBins];
  const ChunkIn ch = w.chunk[blockIdx.x];
  if (ch.c0 >= ch.c1) return;
  const int64_t c0 = ch.c0, c1 = ch.c1;
  const int e = ch.e;
  const uint32_t per = (uint32_t)w.S * (uint32_t)w.R;
  const bool lds = per <= (uint32_t)kLdsBins;
  const uint32_t rb = (uint32_t)e * per;
  if (lds) for (uint32_t b = threadIdx.x; b < per; b += TBB) s_h[b] = 0u;
  __syncthreads();
  for_chunk(w, c0, c1, e, [&](bool ok, uint32_t ru, const float4&) {
    if (!ok) { atomicOr(&w.flags[F_ERR], ERR_INVALID); return; }
    if (lds && ru - rb < per) atomicAdd(&s_h[ru - rb], 1u);
    else atomicAdd(&w.ru_count[ru], 1u);
  });
  __syncthreads();
  if (lds)
    for (uint32_t b = threadIdx.x; b < per; b += TBB)
      if (s_h[b]) atomicAdd(&w.ru_count[rb + b], s_h[b]);
}

// Appends v to a list (forward from 0, or backward from cap - 1) for every
// lane with p: one atomic per wave.  The order of the entries is not
// defined; every consumer's results are independent of it.
__device__ __forceinline__ void list_push(bool p, uint32_t v, uint32_t* ctr, uint32_t* list, bool backward,
                                          int64_t cap) {
  const uint64_t m = __ballot(p);
  if (m == 0ull) return;
  const int leader = __ffsll((unsigned long long)m) - 1;
  uint32_t base = 0;
  if (lane_id() == leader) base = atomicAdd(ctr, (uint32_t)__popcll(m));
  base = (uint32_t)__shfl((int)base, leader, 64);
  if (p) {
    const uint32_t k = base + (uint32_t)__popcll(m & lanemask_lt());
    list[backward ? cap - 1 - (int64_t)k : (int64_t)k] = v;
  }
}

// cells + 1 offsets per row unit; with many row units also the lists of the
// row variants (from the counts, before they are reused as cursors)
__global__ void k_cell_caps(Ws w) {
  const bool lists = ru_lists(w.RU);
  for (int64_t b0 = (int64_t)blockIdx.x * TB; b0 < w.RU; b0 += (int64_t)gridDim.x * TB) {
    const int64_t ru = b0 + threadIdx.x;
    const bool ok = ru < w.RU;
    const uint32_t n = ok ? w.ru_count[ru] : 0u;
    if (ok) w.cell_cap[ru] = grid_cells(n) + 1u;
    if (!lists) continue;
    const int rc = rows_class(n);
    list_push(ok && rc == 1, (uint32_t)ru, &w.flags[F_LROWS1], w.ru_rows, false, w.RU);
    list_push(ok && rc == 2, (uint32_t)ru, &w.flags[F_LROWS2], w.ru_rows, true, w.RU);
    list_push(ok && rc == 3, (uint32_t)ru, &w.flags[F_LROWS3], w.ru_big, false, w.RU);
  }
}

// ru_count is reused as the global fill cursor (zeroed after the scans).
// Each cluster travels with its coordinates and event-local id, so the row
// kernel reads its row unit contiguously instead of gathering from the
// (arbitrarily ordered) input.
__global__ __launch_bounds__(TBB) void k_scatter(Ws w) {
  __shared__ uint32_t s_h[kLdsBins];
  const ChunkIn ch = w.chunk[blockIdx.x];
  if (ch.c0 >= ch.c1) return;
  const int64_t c0 = ch.c0, c1 = ch.c1;
  const int e = ch.e;
  const uint32_t per = (uint32_t)w.S * (uint32_t)w.R;
  const bool lds = per <= (uint32_t)kLdsBins;
  const uint32_t rb = (uint32_t)e * per;
  if (lds) {
    for (uint32_t b = threadIdx.x; b < per; b += TBB) s_h[b] = 0u;
    __syncthreads();
    for_chunk(w, c0, c1, e, [&](bool ok, uint32_t ru, const float4&) {
      if (ok && ru - rb < per) atomicAdd(&s_h[ru - rb], 1u);
    });
    __syncthreads();
    // range reservations: the returning atomics of a thread's bins are all
    // issued before their results are stored
    constexpr int kPer = kLdsBins / TBB;
    uint32_t got[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t b = threadIdx.x + (uint32_t)i * TBB;
      const uint32_t n = b < per ? s_h[b] : 0u;
      got[i] = n ? atomicAdd(&w.ru_count[rb + b], n) : 0u;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const uint32_t b = threadIdx.x + (uint32_t)i * TBB;
      if (b < per) s_h[b] = got[i];
    }
    __syncthreads();
  }
  for_chunk(w, c0, c1, e, [&](bool ok, uint32_t ru, const float4& v) {
    if (!ok) return;
    const uint32_t k = (lds && ru - rb < per) ? atomicAdd(&s_h[ru - rb], 1u) : atomicAdd(&w.ru_count[ru], 1u);
    float4 o = v;
    if (w.cal) {
      // the installed calibration, applied on the way into the row buckets:
      // every later step sees only corrected clusters (the row is kept)
      const int s = (int)((ru / (uint32_t)w.R) % (uint32_t)w.S);
      const int S = w.S;
      const Corrected c = correct_cluster(w.cal_geo, w.cal[s], w.cal[S + s], w.cal + 2 * S + s * 64, s, v.x,
                                          v.y, v.z);
      o.x = c.x;
      o.z = c.z;
    }
    w.tmp4[w.ru_off[ru] + k] = o;
  });
}

__device__ __forceinline__ uint32_t cell_coord(float v, float v0, float inv, uint32_t nc) {
  float t = (v - v0) * inv;
  t = fminf(fmaxf(t, 0.0f), (float)(nc - 1u));
  return (uint32_t)t;
}

__device__ __forceinline__ uint32_t cell_of(const GridParams& G, float y, float z) {
  return cell_coord(z, G.z0, G.inv_bz, G.nz()) * G.ny() + cell_coord(y, G.y0, G.inv_by, G.ny());
}

// Search grid of a row unit of n clusters with the given bounding box: about
// grid_cells(n) cells of equal shape over the box (one cell if the box is
// degenerate or n < 4).  The grid only bounds what a search visits, so
// hardware reciprocals and roots (1 ulp) do; nz ny <= cap holds as a
// quotient of integers up to kMaxCells that is not an integer lies further
// than a few ulp below the next one.  The reciprocal cell sizes stay finite
// where the box is subnormal (its entries then share a cell): the search
// adds and subtracts products with them, which must not be infinite.
constexpr float kMaxInv = 0x1p60f;
__device__ __forceinline__ GridParams make_grid(uint32_t n, uint32_t cbase, uint32_t off, float ymin, float ymax,
                                                float zmin, float zmax) {
  const uint32_t cap = grid_cells(n);
  const float fcap = (float)cap;
  float nz = 1.0f, ny = 1.0f;
  float dz = zmax - zmin, dy = ymax - ymin;
  if (!(n > 0)) { zmin = 0.f; ymin = 0.f; dz = 0.f; dy = 0.f; }
  if (n >= 4 && dz > 0.0f && dy > 0.0f) {
    const float ia = __builtin_amdgcn_rsqf((dz * dy) * __builtin_amdgcn_rcpf(fcap));   // 1 / cell edge
    nz = floorf(fminf(fmaxf(dz * ia, 1.0f), fcap));
    ny = floorf(fmaxf(fminf(dy * ia, fcap * __builtin_amdgcn_rcpf(nz)), 1.0f));
  }
  GridParams G;
  G.cell_base = cbase; G.base = off; G.dims = GridParams::pack((uint32_t)nz, (uint32_t)ny); G.pad = 0u;
  G.z0 = zmin; G.y0 = ymin;
  G.inv_bz = dz > 0.0f ? fminf(nz * __builtin_amdgcn_rcpf(dz), kMaxInv) : 0.0f;
  G.inv_by = dy > 0.0f ? fminf(ny * __builtin_amdgcn_rcpf(dy), kMaxInv) : 0.0f;
  return G;
}

// Ordering of LDS accesses between the lanes of one wave (the wave's LDS
// operations complete in order; this waits for them and keeps the compiler
// from moving accesses across).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Minima over the wave of four values a lane (returned to every lane as x,
// y, z, w): two exchanges leave one value per lane, by its two low bits,
// four more finish it.
__device__ __forceinline__ float4 wave_min4(float a, float b, float c, float d) {
  const bool o1 = threadIdx.x & 1, o2 = threadIdx.x & 2;
  const float ab = fminf(o1 ? b : a, dpp_f32<kDppXor1>(o1 ? a : b));
  const float cd = fminf(o1 ? d : c, dpp_f32<kDppXor1>(o1 ? c : d));
  float v = fminf(o2 ? cd : ab, dpp_f32<kDppXor2>(o2 ? ab : cd));
  v = fminf(v, dpp_f32<kDppRor4>(v));
  v = fminf(v, dpp_f32<kDppRor8>(v));
  v = fminf(v, __shfl_xor(v, 16, 64));
  v = fminf(v, __shfl_xor(v, 32, 64));
  auto at = [&](int l) { return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), l)); };
  return make_float4(at(0), at(1), at(2), at(3));
}

__device__ __forceinline__ uint2 wave_min2(uint32_t a, uint32_t b) {
  const bool o1 = threadIdx.x & 1;
  uint32_t v = min(o1 ? b : a, dpp_u32<kDppXor1>(o1 ? a : b));
  v = min(v, dpp_u32<kDppXor2>(v));
  v = min(v, dpp_u32<kDppRor4>(v));
  v = min(v, dpp_u32<kDppRor8>(v));
  v = min(v, (uint32_t)__shfl_xor((int)v, 16, 64));
  v = min(v, (uint32_t)__shfl_xor((int)v, 32, 64));
  return make_uint2((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 1));
}

// Sorting the ids of a row unit.  They are distinct, so an entry's place is
// the number of smaller ids.  Up to 64 entries count over all of them; in
// larger units NT threads of four entries put the ids into 4 NT buckets over
// equal ranges between the least and the largest id and count over their own
// bucket: the ids of a row are spread evenly over the event's (or follow
// each other if the input is sorted), so it holds one or two.  Where one
// holds more than kBucketMax (clumped ids), every bucket of c ids is divided
// again, into c buckets between its own least and largest id, up to three
// times; a bucket that is still full takes longer and gives the same places.
// Against a bitonic network over lanes and LDS: k_rows on a 3.8 M cluster
// event 161 -> 45 us, ids in two clumps 162 -> 80, k_rows_wave and
// k_rows_tiny on 64 small events 179 -> 81 and 303 -> 193.
constexpr uint32_t kBucketMax = 24;

// hist: 4 NT + 1 words, the first 4 NT cleared; list: 4 NT words; bnd: 8 NT
// words.  place[k]: the place of K[k] where in[k].
template <int NT>
__device__ __forceinline__ void id_places(const uint32_t K[4], const bool in[4], uint32_t n, uint32_t kmin,
                                          uint32_t kmax, uint32_t* hist, uint32_t* list, uint32_t* bnd,
                                          uint32_t place[4]) {
  const uint32_t t = threadIdx.x % NT;
  auto sync = [] { if (NT == 64) wave_sync(); else __syncthreads(); };
  uint32_t bk[4], arr[4], st[4], en[4], m;
  const float scale = (float)(4 * NT) * __builtin_amdgcn_rcpf((float)(kmax - kmin) + 1.0f);
#pragma unroll
  for (int k = 0; k < 4; ++k) bk[k] = min((uint32_t)((float)(K[k] - kmin) * scale), 4u * NT - 1u);
  for (int level = 0;; ++level) {
#pragma unroll
    for (int k = 0; k < 4; ++k) arr[k] = in[k] ? atomicAdd(&hist[bk[k]], 1u) : 0u;
    sync();
    const uint4 h = ((const uint4*)hist)[t];
    const uint32_t sum = h.x + h.y + h.z + h.w;
    uint32_t e, tot;
    if constexpr (NT == 64) e = wave_incl_scan(sum) - sum;
    else e = block_excl_scan(sum, &tot);
    ((uint4*)hist)[t] = make_uint4(e, e + h.x, e + h.x + h.y, e + h.x + h.y + h.z);
    if (t == 0) hist[4 * NT] = n;
    sync();
    m = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      st[k] = hist[bk[k]];
      en[k] = in[k] ? hist[bk[k] + 1u] : st[k];
      m = max(m, en[k] - st[k]);
    }
    const bool full = m > kBucketMax;
    const bool again = (NT == 64 ? __ballot(full) != 0ull : __syncthreads_or(full) != 0) && level < 3;
    if (!again) break;
    sync();
    ((uint4*)hist)[t] = make_uint4(0u, 0u, 0u, 0u);
    ((uint4*)bnd)[t] = make_uint4(~0u, ~0u, ~0u, ~0u);
    ((uint4*)bnd)[t + NT] = make_uint4(0u, 0u, 0u, 0u);
    sync();
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (in[k]) { atomicMin(&bnd[bk[k]], K[k]); atomicMax(&bnd[bk[k] + 4u * NT], K[k]); }
    sync();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (!in[k]) continue;
      const uint32_t lo = bnd[bk[k]], hi = bnd[bk[k] + 4u * NT], c = en[k] - st[k];
      const float sc = (float)c * __builtin_amdgcn_rcpf((float)(hi - lo) + 1.0f);
      bk[k] = st[k] + min((uint32_t)((float)(K[k] - lo) * sc), c - 1u);
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (in[k]) list[st[k] + arr[k]] = K[k];
    place[k] = st[k];
  }
  sync();
  for (uint32_t q = 0; q < m; ++q) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool on = st[k] + q < en[k];
      const uint32_t o = list[on ? st[k] + q : 0u];
      place[k] += on && o < K[k] ? 1u : 0u;
    }
  }
  sync();
}

// Cells' start offsets of a row unit (one wave): the cell histogram hist[0
// .. nc) becomes its exclusive scan, also stored.
__device__ __forceinline__ void wave_cell_offsets(const Ws& w, uint32_t* hist, uint32_t nc, uint32_t cbase,
                                                  uint32_t n) {
  const int lane = lane_id();
  uint32_t carry = 0;
  for (uint32_t c0 = 0; c0 < nc; c0 += 64) {
    const uint32_t c = c0 + lane;
    const uint32_t v = c < nc ? hist[c] : 0u;
    const uint32_t inc = wave_incl_scan(v);
    if (c < nc) { hist[c] = carry + inc - v; w.cell_off[cbase + c] = (uint16_t)(carry + inc - v); }
    carry += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
  }
  if (lane == 0) w.cell_off[cbase + nc] = (uint16_t)n;
}

// Row units of at most 64 clusters (most units of small events): one wave
// each, four per workgroup, no workgroup barrier.  Lane k holds the k-th
// entry: its place is counted over the ids (eight per two LDS reads that
// every lane shares), the entries change lanes through LDS; the grid is
// built as in k_rows with a per-wave LDS histogram.  Same results as k_rows.
// Bound by its instructions.
__global__ __launch_bounds__(TB) void k_rows_tiny(Ws w) {
  constexpr uint32_t kH = (kCellsPerCluster * kTiny + 2 + 3) & ~3u;
  __shared__ alignas(16) uint32_t s_h[TB / 64][kH];
  __shared__ float4 s_rec[TB / 64][kTiny];
  const int wv = threadIdx.x >> 6, lane = lane_id();
  const int64_t ru = (int64_t)blockIdx.x * (TB / 64) + wv;
  if (ru >= w.RU) return;
  const uint32_t off = w.ru_off[ru];
  const uint32_t n = w.ru_off[ru + 1] - off;
  if (n > kTiny) return;
  const uint32_t cbase = w.cell_base[ru];
  uint32_t* hist = s_h[wv];
  float4* rec = s_rec[wv];
  const bool mine = (uint32_t)lane < n;
  float4 v = make_float4(0.f, 0.f, 0.f, __uint_as_float(0xFFFFFFFFu));
  if (mine) v = w.tmp4[off + lane];
  const uint32_t key = __float_as_uint(v.w);
  hist[lane] = key;
  const float4 box = wave_min4(mine ? v.y : INFINITY, mine ? -v.y : INFINITY, mine ? v.z : INFINITY,
                               mine ? -v.z : INFINITY);
  wave_sync();
  uint32_t place = 0;
  const uint4* k4 = (const uint4*)hist;
  for (uint32_t i = 0; i < n; i += 8) {
    const uint4 a = k4[i >> 2], b = k4[(i >> 2) + 1];
    place += a.x < key; place += a.y < key; place += a.z < key; place += a.w < key;
    place += b.x < key; place += b.y < key; place += b.z < key; place += b.w < key;
  }
  if (mine) rec[place] = v;
  wave_sync();
  // grid parameters: every lane computes the same values, lane 0 stores them
  const GridParams G = make_grid(n, cbase, off, box.x, -box.y, box.z, -box.w);
  if (lane == 0) w.grid[ru] = G;
  const uint32_t nc = G.nz() * G.ny();
  for (uint32_t c = lane; c < nc; c += 64) hist[c] = 0u;
  if (mine) {
    v = rec[lane];
    w.cpk[off + lane] = v;
    w.cid[off + lane] = __float_as_uint(v.w); w.cru[off + lane] = (uint32_t)ru;
  }
  wave_sync();
  const uint32_t cell = mine ? cell_of(G, v.y, v.z) : 0u;
  if (mine) atomicAdd(&hist[cell], 1u);
  wave_sync();
  wave_cell_offsets(w, hist, nc, cbase, n);
  wave_sync();
  if (mine) {
    const uint32_t pos = atomicAdd(&hist[cell], 1u);
    w.gbuf[off + pos] = make_float4(v.y, v.z, v.x, __uint_as_float(off + lane));
  }
}

// Row units of kTiny < n <= kWaveRow clusters: one wave each, four per
// workgroup, no workgroup barrier.  Lane l holds entries l, 64 + l, ..; their
// places come from id buckets, the entries change lanes through LDS; the
// grid is built with a per-wave LDS histogram.  Same results as k_rows.
__global__ __launch_bounds__(TB) void k_rows_wave(Ws w) {
  constexpr uint32_t kList = kWaveRow + 4;   // the bucketed ids behind the buckets' bounds
  constexpr uint32_t kH = kList + kWaveRow;
  static_assert(kH >= kCellsPerCluster * kWaveRow + 1, "cells");
  __shared__ alignas(16) uint32_t s_h[TB / 64][kH];
  __shared__ float4 s_rec[TB / 64][kWaveRow];
  const int wv = threadIdx.x >> 6, lane = lane_id();
  uint32_t* hist = s_h[wv];
  uint32_t* list = hist + kList;
  float4* rec = s_rec[wv];
  auto unit = [&](const int64_t ru) {
    const uint32_t off = w.ru_off[ru];
    const uint32_t n = w.ru_off[ru + 1] - off;
    if (rows_class(n) != 1) return;
    const uint32_t cbase = w.cell_base[ru];
    float4 v[4];
    uint32_t K[4];
    bool in[4];
    float b0 = INFINITY, b1 = INFINITY, b2 = INFINITY, b3 = INFINITY;
    uint32_t k0 = 0xFFFFFFFFu, k1 = 0xFFFFFFFFu;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t i = (uint32_t)lane + 64u * k;
      in[k] = i < n;
      v[k] = w.tmp4[off + (in[k] ? i : 0u)];
    }
    ((uint4*)hist)[lane] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int k = 0; k < 4; ++k) {   // (entries past the end repeat the first)
      K[k] = __float_as_uint(v[k].w);
      b0 = fminf(b0, v[k].y); b1 = fminf(b1, -v[k].y); b2 = fminf(b2, v[k].z); b3 = fminf(b3, -v[k].z);
      k0 = min(k0, K[k]); k1 = min(k1, ~K[k]);
    }
    const float4 box = wave_min4(b0, b1, b2, b3);
    const uint2 kr = wave_min2(k0, k1);
    wave_sync();
    uint32_t place[4];
    id_places<64>(K, in, n, kr.x, ~kr.y, hist, list, (uint32_t*)rec, place);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (in[k]) rec[place[k]] = v[k];
    wave_sync();
    // every lane computes the same grid, lane 0 stores it
    const GridParams G = make_grid(n, cbase, off, box.x, -box.y, box.z, -box.w);
    if (lane == 0) w.grid[ru] = G;
    const uint32_t nc = G.nz() * G.ny();
    for (uint32_t c = lane; c < nc; c += 64) hist[c] = 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t i = (uint32_t)lane + 64u * k;
      if (in[k]) {
        v[k] = rec[i];
        w.cpk[off + i] = v[k];
        w.cid[off + i] = __float_as_uint(v[k].w); w.cru[off + i] = (uint32_t)ru;
      }
    }
    wave_sync();
    uint32_t cell[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      cell[k] = in[k] ? cell_of(G, v[k].y, v[k].z) : 0u;
      if (in[k]) atomicAdd(&hist[cell[k]], 1u);
    }
    wave_sync();
    wave_cell_offsets(w, hist, nc, cbase, n);
    wave_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (in[k]) {
        const uint32_t pos = atomicAdd(&hist[cell[k]], 1u);
        w.gbuf[off + pos] = make_float4(v[k].y, v[k].z, v[k].x, __uint_as_float(off + (uint32_t)lane + 64u * k));
      }
    }
  };
  if (!ru_lists(w.RU)) {
    const int64_t ru = (int64_t)blockIdx.x * (TB / 64) + wv;
    if (ru < w.RU) unit(ru);
    return;
  }
  const uint32_t cnt = w.flags[F_LROWS1];
  for (uint32_t i = blockIdx.x * (TB / 64) + wv; i < cnt; i += gridDim.x * (TB / 64)) {
    unit(w.ru_rows[i]);
    wave_sync();   // the histogram is reused by the next unit
  }
}

// One workgroup per row unit: the row unit's (x, y, z, id) entries sorted by
// id, canonical SoA written in that order, then a uniform 2-D grid over the
// row's bounding box with about kCellsPerCluster cells per cluster, filled by
// an LDS counting sort.
//
// Two instantiations: row units of kWaveRow < n <= 4 TB clusters (small LDS,
// so many workgroups share a CU) and larger ones (LDS for kMaxRow ids).  With few row
// units a launch covers every unit and skips those of the other sizes; with
// many its workgroups loop over the class's list.
template <bool kLarge>
__global__ __launch_bounds__(TB) void k_rows(Ws w) {
  constexpr uint32_t kIds = kLarge ? (uint32_t)kMaxRow : 4u * TB;
  constexpr uint32_t kCells = kLarge ? (uint32_t)kMaxCells : kCellsPerCluster * 4u * TB + 1u;   // grid_cells(n) bound
  // large units: the ids being sorted; others: the bucketed ids, then the
  // entries on their way to the threads of their places
  __shared__ float4 s_mem[kLarge ? kIds / 4 : kIds];
  // large units: slots (16 bit) during the sort; others: the bounds of the
  // id buckets; then the cell histogram
  __shared__ alignas(16) uint32_t s_aux[(kCells + 1) > kIds / 2 ? (kCells + 1) : kIds / 2];
  __shared__ float4 s_box[TB / 64];
  __shared__ uint2 s_key[TB / 64];
  uint32_t* s_ids = (uint32_t*)s_mem;
  uint16_t* s_slot = (uint16_t*)s_aux;
  uint32_t* s_hist = s_aux;
  // one row unit (workgroup-uniform); called once per unit of the launch
  auto unit = [&](const int64_t ru) {
    const uint32_t off = w.ru_off[ru];
    const uint32_t n = w.ru_off[ru + 1] - off;
    const uint32_t cbase = w.cell_base[ru];
    const int tid = threadIdx.x;
    if (rows_class(n) != (kLarge ? 3 : 2)) return;   // (smaller units: k_rows_tiny, k_rows_wave)
    if (n > (uint32_t)kMaxRow) {
      if (tid == 0) {
        atomicOr(&w.flags[F_ERR], ERR_LIMIT);
        GridParams G{cbase, off, GridParams::pack(1u, 1u), 0u, 0.f, 0.f, 0.f, 0.f};
        w.grid[ru] = G;
        w.cell_off[cbase] = 0;
        w.cell_off[cbase + 1] = 0;
      }
      // every per-position array still gets a defined entry (its own position
      // in the grid copy), so later kernels stay in bounds until the error is
      // reported
      const float nan = __int_as_float(0x7fc00000);
      for (uint32_t k = tid; k < n; k += TB) {
        w.cpk[off + k] = make_float4(nan, nan, nan, 0.0f);
        w.cid[off + k] = 0u; w.cru[off + k] = (uint32_t)ru;
        w.gbuf[off + k] = make_float4(nan, nan, nan, __uint_as_float(off + k));
      }
      return;
    }
    // Units of up to 4 TB clusters (all but extreme ones): thread t holds
    // entries t, TB + t, ..; their places come from id buckets, the entries
    // change threads through LDS and stay in registers for the grid passes.
    const bool fast = !kLarge;
    float4 v[4];
    bool in[4];
    float b0 = INFINITY, b1 = INFINITY, b2 = INFINITY, b3 = INFINITY;
    uint32_t k0 = 0xFFFFFFFFu, k1 = 0xFFFFFFFFu;
    // the workgroup's minima of the box (all threads); the ids' in k0, k1
    auto reduce = [&]() {
      const float4 b = wave_min4(b0, b1, b2, b3);
      const uint2 kk = wave_min2(k0, k1);
      if (lane_id() == 0) { s_box[tid >> 6] = b; s_key[tid >> 6] = kk; }
      __syncthreads();
  #pragma unroll
      for (int i = 0; i < TB / 64; ++i) {
        const float4 o = s_box[i];
        const uint2 q = s_key[i];
        b0 = fminf(b0, o.x); b1 = fminf(b1, o.y); b2 = fminf(b2, o.z); b3 = fminf(b3, o.w);
        k0 = min(k0, q.x); k1 = min(k1, q.y);
      }
    };
    if (fast) {
      uint32_t K[4];
  #pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t i = (uint32_t)tid + TB * k;
        in[k] = i < n;
        v[k] = w.tmp4[off + (in[k] ? i : 0u)];
      }
      ((uint4*)s_aux)[tid] = make_uint4(0u, 0u, 0u, 0u);
  #pragma unroll
      for (int k = 0; k < 4; ++k) {   // (entries past the end repeat the first)
        K[k] = __float_as_uint(v[k].w);
        b0 = fminf(b0, v[k].y); b1 = fminf(b1, -v[k].y); b2 = fminf(b2, v[k].z); b3 = fminf(b3, -v[k].z);
        k0 = min(k0, K[k]); k1 = min(k1, ~K[k]);
      }
      reduce();
      uint32_t place[4];
      id_places<TB>(K, in, n, k0, ~k1, s_aux, s_ids, s_ids + 4 * TB, place);
  #pragma unroll
      for (int k = 0; k < 4; ++k)
        if (in[k]) s_mem[place[k]] = v[k];
      __syncthreads();
  #pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t i = (uint32_t)tid + TB * k;
        if (in[k]) {
          v[k] = s_mem[i];
          w.cpk[off + i] = v[k];
          w.cid[off + i] = __float_as_uint(v[k].w); w.cru[off + i] = (uint32_t)ru;
        }
      }
    } else {
      uint32_t npad = 2;
      while (npad < n) npad <<= 1;
      for (uint32_t k = tid; k < npad; k += TB) {
        s_ids[k] = k < n ? __float_as_uint(w.tmp4[off + k].w) : 0xFFFFFFFFu;
        s_slot[k] = (uint16_t)k;
      }
      __syncthreads();
      for (uint32_t kk = 2; kk <= npad; kk <<= 1) {
        for (uint32_t j = kk >> 1; j > 0; j >>= 1) {
          for (uint32_t i = tid; i < npad; i += TB) {
            const uint32_t ixj = i ^ j;
            if (ixj > i) {
              const uint32_t a = s_ids[i], b = s_ids[ixj];
              const bool asc = (i & kk) == 0;
              if ((a > b) == asc) {
                s_ids[i] = b; s_ids[ixj] = a;
                const uint16_t t = s_slot[i]; s_slot[i] = s_slot[ixj]; s_slot[ixj] = t;
              }
            }
          }
          __syncthreads();
        }
      }
      for (uint32_t k = tid; k < n; k += TB) {
        const float4 v = w.tmp4[off + s_slot[k]];
        const float y = v.y, z = v.z;
        w.cpk[off + k] = v;
        w.cid[off + k] = s_ids[k]; w.cru[off + k] = (uint32_t)ru;
        b0 = fminf(b0, y); b1 = fminf(b1, -y); b2 = fminf(b2, z); b3 = fminf(b3, -z);
      }
      reduce();
    }
    const GridParams G = make_grid(n, cbase, off, b0, -b1, b2, -b3);
    if (tid == 0) w.grid[ru] = G;
    const uint32_t nc = G.nz() * G.ny();
    for (uint32_t c = tid; c <= nc; c += TB) s_hist[c] = 0u;
    __syncthreads();
    if (fast) {
  #pragma unroll
      for (int k = 0; k < 4; ++k)
        if (in[k]) atomicAdd(&s_hist[cell_of(G, v[k].y, v[k].z)], 1u);
    } else {
      // the canonical entries were written by this same thread (same k
      // stride): re-read them, coalesced
      for (uint32_t k = tid; k < n; k += TB) {
        const float4 c = w.cpk[off + k];
        atomicAdd(&s_hist[cell_of(G, c.y, c.z)], 1u);
      }
    }
    __syncthreads();
    uint32_t carry = 0;
    for (uint32_t c0 = 0; c0 < nc; c0 += TB) {
      const uint32_t c = c0 + tid;
      const uint32_t v = c < nc ? s_hist[c] : 0u;
      uint32_t tot;
      const uint32_t ex = block_excl_scan(v, &tot) + carry;
      if (c < nc) { s_hist[c] = ex; w.cell_off[cbase + c] = (uint16_t)ex; }
      carry += tot;
    }
    if (tid == 0) w.cell_off[cbase + nc] = (uint16_t)n;
    __syncthreads();
    if (fast) {
  #pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (in[k]) {
          const uint32_t slot = atomicAdd(&s_hist[cell_of(G, v[k].y, v[k].z)], 1u);
          w.gbuf[off + slot] = make_float4(v[k].y, v[k].z, v[k].x, __uint_as_float(off + (uint32_t)tid + TB * k));
        }
      }
    } else {
      for (uint32_t k = tid; k < n; k += TB) {
        const float4 c = w.cpk[off + k];
        const uint32_t slot = atomicAdd(&s_hist[cell_of(G, c.y, c.z)], 1u);
        w.gbuf[off + slot] = make_float4(c.y, c.z, c.x, __uint_as_float(off + k));
      }
    }
  };
  if (!ru_lists(w.RU)) {
    unit(blockIdx.x);
    return;
  }
  const uint32_t cnt = w.flags[kLarge ? F_LROWS3 : F_LROWS2];
  for (uint32_t i = blockIdx.x; i < cnt; i += gridDim.x) {
    unit(kLarge ? w.ru_big[i] : w.ru_rows[w.RU - 1 - (int64_t)i]);
    __syncthreads();   // LDS is reused by the next unit
  }
}

// Cell rectangle [iz0, iz1] x [iy0, iy1] covering |y - yq| <= wy, |z - zq| <= wz
// (the margin absorbs the rounding of the bounds; the exact test is done per
// candidate).  The bounds are cell coordinates of positions, by the same
// monotone function as the entries': wherever the query lies and however
// small the cells are beside the window, an entry between two positions has
// its cell between theirs.
struct CellBox { uint32_t iz0, iz1, iy0, iy1; };
__device__ __forceinline__ CellBox cell_box(const GridParams& G, float yq, float zq, float wy, float wz) {
  const float m = 1e-3f;
  CellBox b;
  b.iz0 = cell_coord(zq - wz - m, G.z0, G.inv_bz, G.nz());
  b.iz1 = cell_coord(zq + wz + m, G.z0, G.inv_bz, G.nz());
  b.iy0 = cell_coord(yq - wy - m, G.y0, G.inv_by, G.ny());
  b.iy1 = cell_coord(yq + wy + m, G.y0, G.inv_by, G.ny());
  return b;
}

// ---------------------------------------------------------- a2: neighbours
// For the middle cluster i: the (down, up) pair on rows r-1 / r+1 inside the
// windows minimising the deviation of i from the chord d-u, accepted iff the
// score <= link_cut, ties by smaller up id then smaller down id (canonical
// positions are ordered like ids within a row).  D/U: the grid-ordered
// entries of the two rows; Dc/Uc: their cell start offsets (index into D/U).
template <class F4, class U32>
__device__ __forceinline__ void find_pair(const Ws& w, float xi, float yi, float zi,
                                          const GridParams& Gd, F4 D4, U32 Dc,
                                          const GridParams& Gu, F4 U4, U32 Uc,
                                          int32_t& bu, int32_t& bd) {
  const float WY = w.P.win_y, WZ = w.P.win_z, IWY = w.P.inv_var_y, IWZ = w.P.inv_var_z;
  const float CUT = w.P.link_cut;
  const CellBox bdn = cell_box(Gd, yi, zi, WY, WZ);
  const CellBox bup = cell_box(Gu, yi, zi, WY, WZ);
  bool have = false;
  float bs = 0.0f;
  bu = -1; bd = -1;
  for (uint32_t izd = bdn.iz0; izd <= bdn.iz1; ++izd) {
    const uint32_t cd0 = izd * Gd.ny();
    const uint32_t kd1 = Dc[cd0 + bdn.iy1 + 1];
    for (uint32_t kd = Dc[cd0 + bdn.iy0]; kd < kd1; ++kd) {
      const float4 D = D4[kd];
      if (!(fabsf(D.x - yi) <= WY && fabsf(D.y - zi) <= WZ)) continue;
      const int32_t pd = (int32_t)__float_as_uint(D.w);
      for (uint32_t izu = bup.iz0; izu <= bup.iz1; ++izu) {
        const uint32_t cu0 = izu * Gu.ny();
        const uint32_t ku1 = Uc[cu0 + bup.iy1 + 1];
        for (uint32_t ku = Uc[cu0 + bup.iy0]; ku < ku1; ++ku) {
          const float4 U = U4[ku];
          if (!(fabsf(U.x - yi) <= WY && fabsf(U.y - zi) <= WZ)) continue;
          const float wgt = (xi - D.z) / (U.z - D.z);
          const float ey = yi - fmaf(U.x - D.x, wgt, D.x);
          const float ez = zi - fmaf(U.y - D.y, wgt, D.y);
          const float score = fmaf(ez * ez, IWZ, (ey * ey) * IWY);
          if (!(score <= CUT)) continue;
          const int32_t pu = (int32_t)__float_as_uint(U.w);
          const bool better = !have || score < bs || (score == bs && (pu < bu || (pu == bu && pd < bd)));
          if (better) { have = true; bs = score; bu = pu; bd = pd; }
        }
      }
    }
  }
}

constexpr int kCand = 15;          // passing candidates per side kept per lane

// Candidates of a lane in the band kernel: up to kBandCand entry indexes of 8
// bits, written to LDS one by one and read back at once.
constexpr int kBandCand = 16;
constexpr uint32_t kBandRow = 256;   // entries of a row with such candidates, at most
struct CandList {
  uint64_t lo, hi;
  __device__ __forceinline__ explicit CandList(const uint4& v)
      : lo(((uint64_t)v.y << 32) | v.x), hi(((uint64_t)v.w << 32) | v.z) {}
  __device__ __forceinline__ uint32_t pop() {
    const uint32_t k = (uint32_t)lo & 0xFFu;
    lo = (lo >> 8) | (hi << 56);
    hi >>= 8;
    return k;
  }
};

// Window scan of one row's box: indices (into D4) of the entries within the
// windows, the first kMax of them to out; returns their count.  Two z rows
// of the box at a time are taken as one list, so that a lane waits for LDS
// once for their bounds and once per four entries.
template <int kMax, class Idx>
__device__ __forceinline__ int collect(const GridParams& G, const float4* D4, const uint16_t* Dc, float yi, float zi,
                                       float WY, float WZ, Idx* out) {
  const CellBox b = cell_box(G, yi, zi, WY, WZ);
  const uint32_t ny = G.ny(), iz0 = b.iz0, iz1 = b.iz1, iy0 = b.iy0, iy1 = b.iy1 + 1u;
  int n = 0;
  for (uint32_t iz = iz0; iz <= iz1; iz += 2) {
    const uint16_t* c0 = Dc + iz * ny;
    const uint16_t* c1 = iz < iz1 ? c0 + ny : c0;
    const uint32_t a0 = c0[iy0], a1 = c0[iy1], e0 = c1[iy0], e1 = c1[iy1];
    const uint32_t la = a1 - a0, tot = la + (iz < iz1 ? e1 - e0 : 0u), eo = e0 - la;
    for (uint32_t t = 0; t < tot; t += 4) {
      float4 D[4];
      uint32_t k[4];
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        const uint32_t u = min(t + j, tot - 1u);
        k[j] = u + (u < la ? a0 : eo);
        D[j] = D4[k[j]];
      }
#pragma unroll
      for (uint32_t j = 0; j < 4; ++j) {
        if (t + j < tot && fabsf(D[j].x - yi) <= WY && fabsf(D[j].y - zi) <= WZ) {
          out[min(n, kMax - 1)] = (Idx)k[j];
          ++n;
        }
      }
    }
  }
  return n;
}

// Pairs of one lane's candidates (at most kBandCand a side), same arithmetic
// and tie-break as find_pair.  The least key (score bits, up offset, down
// offset) is find_pair's choice: a score that passes the cut is >= 0, so its
// bits order like its value, and the offsets of the rows' canonical
// positions (fewer than 2^16 entries) order like the positions.  The first
// four up candidates are read together and kept, the next down candidate is
// read ahead.  The interpolation weight depends only on the x coordinates:
// where those of the up candidates agree (clusters on their row planes) its
// quotient is taken once per x of the down candidates.
__device__ __forceinline__ void best_pair(const Ws& w, float xi, float yi, float zi, const float4* D4, CandList ld,
                                          int nd, uint32_t offd, const float4* U4, CandList lu, int nu, uint32_t offu,
                                          int32_t& bu, int32_t& bd) {
  const float IWY = w.P.inv_var_y, IWZ = w.P.inv_var_z;
  bu = -1; bd = -1;
  if (nu == 0) return;
  // (just above every key that passes the cut)
  const uint64_t none = ((uint64_t)__float_as_uint(w.P.link_cut) << 32) | 0xFFFFFFFFull;
  uint64_t best = none;
  constexpr int kKeep = 4;
  float4 U[kKeep];
  uint32_t ku[kKeep];
  bool plane = nu <= kKeep;
#pragma unroll
  for (int t = 0; t < kKeep; ++t) {
    const uint32_t k = lu.pop();
    U[t] = U4[t < nu ? k : 0u];
    ku[t] = (__float_as_uint(U[t].w) - offu) << 16;
    plane = plane && (t >= nu || U[t].z == U[0].z);
  }
  auto pair = [&](const float4& D, const float4& Ut, uint32_t low, float wq) {
    const float ey = yi - fmaf(Ut.x - D.x, wq, D.x);
    const float ez = zi - fmaf(Ut.y - D.y, wq, D.y);
    const float score = fmaf(ez * ez, IWZ, (ey * ey) * IWY);
    const uint64_t key = ((uint64_t)__float_as_uint(score) << 32) | low;
    best = key < best ? key : best;
  };
  float4 Dn = D4[ld.pop()];
  float wx = 0.0f, wq = 0.0f;
  for (int i = 0; i < nd; ++i) {
    const float4 D = Dn;
    const uint32_t k = ld.pop();
    Dn = D4[i + 1 < nd ? k : 0u];   // (past the last one: not used)
    const uint32_t kd = __float_as_uint(D.w) - offd;
    if (plane) {
      if (i == 0 || D.z != wx) { wq = (xi - D.z) / (U[0].z - D.z); wx = D.z; }
#pragma unroll
      for (int t = 0; t < kKeep; ++t)
        if (t < nu) pair(D, U[t], ku[t] | kd, wq);
    } else {
#pragma unroll
      for (int t = 0; t < kKeep; ++t)
        if (t < nu) pair(D, U[t], ku[t] | kd, (xi - D.z) / (U[t].z - D.z));
      CandList rest = lu;
      for (int j = kKeep; j < nu; ++j) {
        const float4 Uj = U4[rest.pop()];
        pair(D, Uj, ((__float_as_uint(Uj.w) - offu) << 16) | kd, (xi - D.z) / (Uj.z - D.z));
      }
    }
  }
  if (best != none) {
    bu = (int32_t)(offu + ((uint32_t)best >> 16));
    bd = (int32_t)(offd + ((uint32_t)best & 0xFFFFu));
  }
}

// The pairs of a wave's lanes scored by all 64 lanes, same arithmetic and
// tie-break as find_pair.  Lane l (has: a cluster whose lists fit) owns
// cd_l cu_l pairs, listed in lane order and, within a lane, down-major; the
// list is cut into 64 contiguous ranges, one per lane, so a wave runs about
// its mean pair count instead of its lanes' largest candidate counts.  A lane
// keeps the least key of the pairs it scored for the current owner and folds
// it into the owner's LDS word (atomic minimum) when it moves on.  The key
// is (score bits, up offset, down offset) in 32 + 10 + 10 bits: a score that
// passes the cut is >= 0, so its bits order like its value, and the offsets
// of the neighbour rows' canonical positions (rows of at most kSlab entries)
// order like the positions, so the least key is find_pair's choice.  Called
// by all lanes of the wave; ld_w/lu_w/key_w: the wave's slices of the
// candidate lists and of the key words.
constexpr unsigned long long kNoKey = ~0ull;
static_assert(kSlab <= 1024u, "row offsets in the pair key take 10 bits");

__device__ __forceinline__ void wave_pairs(const Ws& w, bool has, float xi, float yi, float zi, uint32_t cd,
                                           uint32_t cu, const float4* D4, const float4* U4, const uint16_t* ld_w,
                                           const uint16_t* lu_w, unsigned long long* key_w, uint32_t offd,
                                           uint32_t offu, int32_t& bu, int32_t& bd) {
  const float IWY = w.P.inv_var_y, IWZ = w.P.inv_var_z, CUT = w.P.link_cut;
  const int lane = lane_id();
  const uint32_t cnt = has ? cd * cu : 0u;
  const uint32_t incl = wave_incl_scan(cnt);
  const uint32_t P = (uint32_t)__shfl((int)incl, 63, 64);
  bu = -1; bd = -1;
  if (P == 0u) return;   // (uniform)
  key_w[lane] = kNoKey;
  wave_sync();
  const uint64_t owners = __ballot(cnt > 0u);
  uint32_t t = (uint32_t)(((uint64_t)lane * P) >> 6);
  const uint32_t t1 = (uint32_t)(((uint64_t)(lane + 1) * P) >> 6);
  // owner of pair t (< P): the lowest lane whose inclusive count exceeds t
  int o = 0;
#pragma unroll
  for (int st = 32; st > 0; st >>= 1) {
    const uint32_t v = (uint32_t)__shfl((int)incl, o + st - 1, 64);
    if (v <= t) o += st;
  }
  // the owner's cluster, up count and pair range (shuffles by every lane)
  float oxi, oyi, ozi;
  uint32_t ocu, oend;
  auto fetch = [&](int src) {
    oxi = __shfl(xi, src, 64);
    oyi = __shfl(yi, src, 64);
    ozi = __shfl(zi, src, 64);
    ocu = (uint32_t)__shfl((int)cu, src, 64);
    oend = (uint32_t)__shfl((int)incl, src, 64);
  };
  fetch(o);
  const uint32_t ocnt = (uint32_t)__shfl((int)cnt, o, 64);
  uint32_t i = 0, j = 0;
  if (t < t1) {
    const uint32_t rel = t - (oend - ocnt);
    i = rel / ocu;
    j = rel - i * ocu;
  }
  unsigned long long best = kNoKey;
  // the interpolation quotient of the last pair, reused while the three x
  // coordinates repeat (clusters on their row planes)
  float wx_i = 0.0f, wx_d = 0.0f, wx_u = 0.0f, wq = 0.0f;
  bool wk = false;
  const uint32_t steps = (P + 63u) >> 6;   // the longest range
  for (uint32_t k = 0; k < steps; ++k) {
    const bool act = t < t1;
    if (act) {
      const float4 D = D4[ld_w[kCand * o + (int)i]];
      const float4 U = U4[lu_w[kCand * o + (int)j]];
      if (!(wk && oxi == wx_i && D.z == wx_d && U.z == wx_u)) {
        wq = (oxi - D.z) / (U.z - D.z);
        wx_i = oxi; wx_d = D.z; wx_u = U.z; wk = true;
      }
      const float ey = oyi - fmaf(U.x - D.x, wq, D.x);
      const float ez = ozi - fmaf(U.y - D.y, wq, D.y);
      const float score = fmaf(ez * ez, IWZ, (ey * ey) * IWY);
      if (score <= CUT) {
        const unsigned long long key = ((unsigned long long)__float_as_uint(score) << 20) |
                                       ((unsigned long long)(__float_as_uint(U.w) - offu) << 10) |
                                       (unsigned long long)(__float_as_uint(D.w) - offd);
        best = key < best ? key : best;
      }
      ++t;
      if (++j == ocu) { j = 0; ++i; }
    }
    const bool fold = act && (t == oend || t == t1);
    if (fold && best != kNoKey) atomicMin(&key_w[o], best);
    if (fold) best = kNoKey;
    // the range goes on into the next owner (a later lane with pairs)
    const bool next = act && t == oend && t < t1;
    if (__ballot(next) != 0ull) {
      const int on = next ? __ffsll((unsigned long long)(owners & ~((2ull << o) - 1ull))) - 1 : o;
      fetch(on);
      if (next) { o = on; i = 0; j = 0; }
    }
  }
  wave_sync();
  const unsigned long long b = key_w[lane];
  if (has && b != kNoKey) {
    bu = (int32_t)(offu + (uint32_t)((b >> 10) & 1023ull));
    bd = (int32_t)(offd + (uint32_t)(b & 1023ull));
  }
}

// Links of a band of rows of one (event, sector): the grids of the rows and
// of the two beside them (entries and cell offsets, each one contiguous
// range) are staged in LDS and the rows' clusters taken in grid order, one
// per lane, without regard to where a row ends.  A lane first collects the
// down and up candidates inside the windows (two flat scans), then scores
// the pairs; nested scanning would make a wave run the product of its lanes'
// largest candidate counts.  Where the band does not fit, the workgroup
// takes as many of its rows at a time as fit; a row that does not fit with
// its neighbours alone is left to k_links.  Results do not depend on the
// order.  Bound by its instructions: a wave or workgroup per row left half
// the lanes idle on rows of 33 clusters and staged every row twice (64 small
// events 583 us, this way 315; 0.77 M clusters 44 and 38).
constexpr int kLinkRows = 8;             // rows of a band, at most
// Entries staged, at most and at least (five and six workgroups share a
// compute unit's LDS).
constexpr uint32_t kLinkE = 1152, kLinkEMin = 768;
// 32-bit words of the cell offsets of up to e entries (pairs of 16-bit
// offsets, aligned as in memory)
__host__ __device__ inline uint32_t link_words(uint32_t e) { return (kCellsPerCluster * e + 2u * (kLinkRows + 2)) / 2 + 1; }

__global__ __launch_bounds__(TB) void k_links_band(Ws w, int rows, uint32_t cap) {
  extern __shared__ float4 s_e[];   // cap entries, then the words of their cell offsets
  uint32_t* s_c = (uint32_t*)(s_e + cap);
  __shared__ float4 s_g[2 * (kLinkRows + 2)];
  __shared__ uint32_t s_off[kLinkRows + 3], s_cb[kLinkRows + 3];
  __shared__ uint4 s_ld[TB], s_lu[TB];
  const int nband = (w.R + rows - 1) / rows;
  const int64_t ru0 = (int64_t)(blockIdx.x / nband) * w.R;
  const int r_lo = (int)(blockIdx.x % nband) * rows, r_hi = min(r_lo + rows, w.R) - 1;
  const int first = max(r_lo - 1, 0), last = min(r_hi + 1, w.R - 1);   // rows read
  const int tid = threadIdx.x;
  if (tid <= last + 1 - first) {
    s_off[tid] = w.ru_off[ru0 + first + tid];
    s_cb[tid] = w.cell_base[ru0 + first + tid];
  }
  __syncthreads();
  auto off = [&](int r) { return s_off[r - first]; };
  // entries of rows r .. r + m - 1 and the two beside them
  auto need = [&](int r, int m) { return off(min(r + m, w.R - 1) + 1) - off(max(r - 1, 0)); };
  // a row for k_links
  auto is_over = [&](int r) {
    return need(r, 1) > cap || off(r) - off(max(r - 1, 0)) > kBandRow ||
           off(min(r + 1, w.R - 1) + 1) - off(r + 1) > kBandRow;
  };
  if (tid < 64) {
    const int r = min(r_lo + tid, r_hi);
    const bool over = r_lo + tid <= r_hi && off(r + 1) > off(r) && is_over(r);
    if (ru_lists(w.RU)) list_push(over, (uint32_t)(ru0 + r), &w.flags[F_LLINKS], w.ru_links, false, w.RU);
    else if (over) w.flags[F_LLINKS] = 1u;   // (thousands of additions to one counter would take 35 us)
  }
  const float WY = w.P.win_y, WZ = w.P.win_z;
  for (int r = r_lo; r <= r_hi;) {   // (uniform)
    const int a = max(r - 1, 0);
    // the most rows that fit (the lanes try all)
    const int l = lane_id();
    const int q = min(r + l, r_hi);
    const uint64_t ov = __ballot(l > r_hi - r || is_over(q)), fit = __ballot(need(r, q - r + 1) <= cap);
    const int m = min(__popcll(fit), __ffsll((unsigned long long)ov) - 1);
    if (m == 0) { ++r; continue; }   // (k_links)
    const int z = min(r + m, w.R - 1) + 1;   // rows a .. z - 1 are staged
    const uint32_t o0 = off(a), o1 = off(z), f0 = off(r), f1 = off(r + m);
    const uint32_t c0 = s_cb[a - first] & ~1u, c1 = s_cb[z - first];
    if (f1 > f0) {
      // kLinkEMin entries and their cell offsets per pass, the loads of a
      // pass issued before its first LDS store (indexes past the end load
      // the first entry)
      constexpr int kE = (int)(kLinkEMin / TB), kC = (int)((kCellsPerCluster * kLinkEMin / 2 + kLinkRows + 3 + TB - 1) / TB);
      const uint32_t* cells = (const uint32_t*)(w.cell_off + c0);
      const float4* ent = w.gbuf + o0;
      const uint32_t nc2 = (c1 - c0 + 1u) >> 1, ne = o1 - o0;
      if (tid < 2 * (z - a)) s_g[tid] = ((const float4*)(w.grid + ru0 + a))[tid];
      for (uint32_t b0 = 0, d0 = 0; b0 < ne || d0 < nc2; b0 += kE * TB, d0 += kC * TB) {
        float4 ve[kE];
        uint32_t vc[kC];
  #pragma unroll
        for (int j = 0; j < kE; ++j) {
          const uint32_t i = b0 + (uint32_t)tid + TB * j;
          ve[j] = ent[i < ne ? i : 0u];
        }
  #pragma unroll
        for (int j = 0; j < kC; ++j) {
          const uint32_t i = d0 + (uint32_t)tid + TB * j;
          vc[j] = cells[i < nc2 ? i : 0u];
        }
  #pragma unroll
        for (int j = 0; j < kE; ++j) {
          const uint32_t i = b0 + (uint32_t)tid + TB * j;
          if (i < ne) s_e[i] = ve[j];
        }
  #pragma unroll
        for (int j = 0; j < kC; ++j) {
          const uint32_t i = d0 + (uint32_t)tid + TB * j;
          if (i < nc2) s_c[i] = vc[j];
        }
      }
      __syncthreads();
      const GridParams* g = (const GridParams*)s_g;
      const uint16_t* cell = (const uint16_t*)s_c;
      // lane k: where the k-th of the staged rows begins
      const uint32_t start = l < z - a ? off(a + min(l, z - a)) - o0 : ~0u;
      for (uint32_t i = f0 - o0 + (uint32_t)tid; i < f1 - o0; i += TB) {
        const float4 me = s_e[i];
        // the cluster's row: the last one that begins at or before it (rows
        // without clusters begin with the one behind them)
        int q = -1;
  #pragma unroll
        for (int k = 0; k < kLinkRows + 2; ++k) q += (uint32_t)__builtin_amdgcn_readlane((int)start, k) <= i ? 1 : 0;
        const uint32_t p = __float_as_uint(me.w);
        int32_t bu = -1, bd = -1;
        if (a + q >= 1 && a + q <= w.R - 2) {   // (edge rows have no links)
          const float xi = me.z, yi = me.x, zi = me.y;
          const GridParams Gd = g[q - 1], Gu = g[q + 1];
          const float4* de = s_e + (Gd.base - o0);
          const float4* ue = s_e + (Gu.base - o0);
          const uint16_t* dc = cell + (Gd.cell_base - c0);
          const uint16_t* uc = cell + (Gu.cell_base - c0);
          const int cd = collect<kBandCand>(Gd, de, dc, yi, zi, WY, WZ, (uint8_t*)&s_ld[tid]);
          const int cu = cd > 0 ? collect<kBandCand>(Gu, ue, uc, yi, zi, WY, WZ, (uint8_t*)&s_lu[tid]) : 0;
          if (cd <= kBandCand && cu <= kBandCand)
            best_pair(w, xi, yi, zi, de, CandList(s_ld[tid]), cd, Gd.base, ue, CandList(s_lu[tid]), cu, Gu.base, bu, bd);
          else find_pair(w, xi, yi, zi, Gd, de, dc, Gu, ue, uc, bu, bd);
        }
        w.up[p] = bu;
        w.dn[p] = bd;
      }
      __syncthreads();   // LDS is reused by the next rows
    }
    r += m;
  }
}

// Rows too large for k_links_band, one workgroup each (with many row units
// from its list): the
// grids of rows r-1 and r+1 are staged in LDS when each holds at most kSlab
// clusters.  Lanes take the row's clusters in grid order, so the lanes of a
// wave are spatial neighbours with similar candidate counts; a wave's pairs
// are scored by all its lanes (wave_pairs).
__global__ __launch_bounds__(TB) void k_links(Ws w, uint32_t cap) {
  // one spare slot at the end of each array takes the staging stores of
  // slots past a row's end (never read)
  constexpr uint32_t kSpareE = kSlab, kSpareC = kCellsPerCluster * kSlab + 2;
  __shared__ float4 sd[kSlab + 1], su[kSlab + 1];
  // cell offsets relative to the slab (< kSlab): 16 bit; a row of <= kSlab
  // clusters has at most kCellsPerCluster kSlab + 1 cells
  __shared__ uint16_t scd[kSpareC + 1], scu[kSpareC + 1];
  __shared__ uint16_t s_ld[kCand * TB], s_lu[kCand * TB];
  // per-lane best pair keys of the wave-level pair scoring
  __shared__ unsigned long long s_key[TB];
  const uint32_t tid = threadIdx.x;
  // one row unit (workgroup-uniform); called once per unit of the launch
  auto unit = [&](const int64_t ru) {
    const int r = (int)(ru % w.R);
    const bool inner = r >= 1 && r <= w.R - 2;
    // every row offset and both neighbour grids in one round of loads
    const int64_t rdn = inner ? ru - 1 : ru, rup = inner ? ru + 1 : ru;
    const uint32_t offd = w.ru_off[rdn], off = w.ru_off[ru], offu = w.ru_off[ru + 1];
    const uint32_t endu = w.ru_off[inner ? ru + 2 : ru + 1];
    const GridParams Gd = w.grid[rdn], Gu = w.grid[rup];
    const uint32_t n = offu - off;
    // edge rows have no links; an over-full row unit (reported as an error) gets none either
    if (!inner || n > (uint32_t)kMaxRow) {
      for (uint32_t k = tid; k < n; k += TB) { w.up[off + k] = -1; w.dn[off + k] = -1; }
      return;
    }
    const uint32_t nd = off - offd, nu = endu - offu;
    const bool lds = nd <= kSlab && nu <= kSlab;
    // this thread's own clusters (grid order) for its first rounds, read now
    // so that they arrive with the staged rows
    constexpr int kOwn = 4;
    float4 mine[kOwn];
  #pragma unroll
    for (int i = 0; i < kOwn; ++i) {
      const uint32_t k = tid + TB * i;
      mine[i] = w.gbuf[off + (k < n ? k : 0u)];   // (used only if k < n)
    }
    const float WY = w.P.win_y, WZ = w.P.win_z;
    if (!lds) {
      auto link = [&](const float4& me) {
        int32_t bu, bd;
        find_pair(w, me.z, me.x, me.y, Gd, w.gbuf + offd, w.cell_off + Gd.cell_base, Gu, w.gbuf + offu,
                  w.cell_off + Gu.cell_base, bu, bd);
        const uint32_t p = __float_as_uint(me.w);
        w.up[p] = bu;
        w.dn[p] = bd;
      };
  #pragma unroll
      for (int i = 0; i < kOwn; ++i)
        if (tid + TB * i < n) link(mine[i]);
      for (uint32_t k = tid + TB * kOwn; k < n; k += TB) link(w.gbuf[off + k]);
      return;
    }
    // all of a thread's staging loads are issued before the first LDS store
    // (one memory round trip instead of one per loop iteration); slots past
    // a row's end load an entry known to exist (this row's first entry, the
    // row's first cell offset) and store it to the spare slot, so that
    // neither the loads nor the stores need a branch
    constexpr int kE = (int)((kSlab + TB - 1) / TB);                          // entries per thread
    constexpr int kC = (int)((kCellsPerCluster * kSlab + 1 + TB) / TB);      // cell offsets per thread
    const uint32_t ncd = Gd.nz() * Gd.ny(), ncu = Gu.nz() * Gu.ny();
  #pragma unroll
    for (int j = 0; j < kE; ++j) {
      const uint32_t i = tid + TB * (uint32_t)j;
      const float4 a = w.gbuf[i < nd ? offd + i : off];
      const float4 b = w.gbuf[i < nu ? offu + i : off];
      sd[i < nd ? i : kSpareE] = a;
      su[i < nu ? i : kSpareE] = b;
    }
  #pragma unroll
    for (int j = 0; j < kC; ++j) {
      const uint32_t i = tid + TB * (uint32_t)j;
      const uint16_t a = w.cell_off[Gd.cell_base + (i <= ncd ? i : 0u)];
      const uint16_t b = w.cell_off[Gu.cell_base + (i <= ncu ? i : 0u)];
      scd[i <= ncd ? i : kSpareC] = a;
      scu[i <= ncu ? i : kSpareC] = b;
    }
    __syncthreads();
    uint16_t* ld = s_ld + kCand * tid;
    uint16_t* lu = s_lu + kCand * tid;
    // rounds of the wave's 64 clusters: candidate lists per lane, then
    // the wave's pairs scored by all its lanes; a lane whose lists
    // overflow takes find_pair afterwards
    const uint32_t wb = tid & ~63u;
    const uint16_t* ld_w = s_ld + kCand * wb;
    const uint16_t* lu_w = s_lu + kCand * wb;
    unsigned long long* key_w = s_key + wb;
    // the prefetched clusters move down one slot per round (an array
    // indexed by the round would be placed in scratch memory)
    float4 m0 = mine[0], m1 = mine[1], m2 = mine[2], m3 = mine[3];
    for (uint32_t i = 0; wb + TB * i < n; ++i) {
      const uint32_t k = tid + TB * i;
      const bool has = k < n;
      float4 me = m0;
      if (i >= (uint32_t)kOwn) me = w.gbuf[off + (has ? k : 0u)];
      m0 = m1; m1 = m2; m2 = m3;
      const float xi = me.z, yi = me.x, zi = me.y;
      int cd = 0, cu = 0;
      if (has) {
        cd = collect<kCand>(Gd, sd, scd, yi, zi, WY, WZ, ld);
        cu = cd > 0 ? collect<kCand>(Gu, su, scu, yi, zi, WY, WZ, lu) : 0;
      }
      const bool fb = has && (cd > kCand || cu > kCand);
      int32_t bu, bd;
      wave_pairs(w, has && !fb, xi, yi, zi, (uint32_t)cd, (uint32_t)cu, (const float4*)sd, (const float4*)su,
                 ld_w, lu_w, key_w, offd, offu, bu, bd);
      if (fb)
        find_pair(w, xi, yi, zi, Gd, (const float4*)sd, (const uint16_t*)scd, Gu, (const float4*)su,
                  (const uint16_t*)scu, bu, bd);
      if (has) {
        const uint32_t p = __float_as_uint(me.w);
        w.up[p] = bu;
        w.dn[p] = bd;
      }
    }
  };
  const bool lists = ru_lists(w.RU);
  const uint32_t cnt = w.flags[F_LLINKS];
  for (uint32_t i = blockIdx.x; i < (lists || cnt == 0u ? cnt : (uint32_t)w.RU); i += gridDim.x) {
    const uint32_t ru = lists ? w.ru_links[i] : i;
    if (!lists) {
      const int r = (int)(ru % (uint32_t)w.R);
      const uint32_t a = w.ru_off[r > 0 ? ru - 1 : ru], b = w.ru_off[ru], c = w.ru_off[ru + 1];
      const uint32_t z = w.ru_off[r < w.R - 1 ? ru + 2 : ru + 1];
      if (b == c || (z - a <= cap && b - a <= kBandRow && z - c <= kBandRow)) continue;   // (k_links_band)
    }
    unit(ru);
    __syncthreads();   // LDS is reused by the next unit
  }
}

// ------------------------------------------------------- a3/a4: clean/start
// Keep a link only if reciprocated (from the raw arrays).  Start hit: kept up
// link, no kept down link.  Seed: start hit whose chain reaches
// min_seed_hits clusters.  Optional taps map positions to cluster ids.
// Invalid clusters have no row unit and so no position: the positions behind
// the last row unit hold what earlier calls left and are flagged only (the
// call reports the error at its end).
// Bound by memory: the up link goes into the record that the rows have
// written (4 bytes of its 16; records written here as well took 55 us
// instead of 43 on 3.8 M clusters, a link array of its own 36 but 15 more in
// the tracklets' chains, which then wait for two loads a step).
__global__ __launch_bounds__(TB) void k_clean(Ws w) {
  __shared__ uint32_t s_cnt[2][TB / 64];
  const int64_t p = (int64_t)blockIdx.x * TB + threadIdx.x;
  bool start = false, seed = false;
  if (p < (int64_t)w.ru_off[w.RU]) {
    // both links, then both reciprocity gathers together
    // (a missing link reads the cluster's own entry, which is not used)
    const int32_t u = w.up[p], d = w.dn[p];
    const int32_t du = w.dn[u >= 0 ? u : (int32_t)p];
    const int32_t ud = w.up[d >= 0 ? d : (int32_t)p];
    const int32_t cu = (u >= 0 && du == (int32_t)p) ? u : -1;
    const int32_t cd = (d >= 0 && ud == (int32_t)p) ? d : -1;
    w.cpk[p].w = __int_as_float(cu);
    start = cu >= 0 && cd < 0;
    if (start) {
      int L = 2;
      int32_t q = cu;
      while (L < w.P.min_seed_hits) {
        const int32_t nu = w.up[q];
        if (nu < 0 || w.dn[nu] != q) break;
        q = nu;
        ++L;
      }
      seed = L >= w.P.min_seed_hits;
    }
    w.flag[p] = (uint8_t)((start ? 1 : 0) | (seed ? 2 : 0));
    if (w.taps) {
      const int e = (int)(w.cru[p] / ((uint32_t)w.S * (uint32_t)w.R));
      const EventOut& O = w.out[e];
      const uint32_t id = w.cid[p];
      if (O.dbg_up) O.dbg_up[id] = u >= 0 ? (int32_t)w.cid[u] : -1;
      if (O.dbg_dn) O.dbg_dn[id] = d >= 0 ? (int32_t)w.cid[d] : -1;
      if (O.dbg_cup) O.dbg_cup[id] = cu >= 0 ? (int32_t)w.cid[cu] : -1;
      if (O.dbg_cdn) O.dbg_cdn[id] = cd >= 0 ? (int32_t)w.cid[cd] : -1;
    }
  } else if (p < w.N) {
    w.flag[p] = 0;
  }
  const uint64_t bs = __ballot(start), bq = __ballot(seed);
  if (lane_id() == 0) { s_cnt[0][threadIdx.x >> 6] = (uint32_t)__popcll(bs); s_cnt[1][threadIdx.x >> 6] = (uint32_t)__popcll(bq); }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t a = 0, b = 0;
    for (int i = 0; i < TB / 64; ++i) { a += s_cnt[0][i]; b += s_cnt[1][i]; }
    w.blk_start[blockIdx.x] = a;
    w.blk_seed[blockIdx.x] = b;
  }
}

// Ordered compaction: block offset (scanned) + wave offset + ballot rank.
__global__ __launch_bounds__(TB) void k_compact(Ws w) {
  __shared__ uint32_t s_cnt[2][TB / 64];
  const int64_t p = (int64_t)blockIdx.x * TB + threadIdx.x;
  const uint8_t f = p < w.N ? w.flag[p] : (uint8_t)0;
  const bool start = f & 1, seed = (f >> 1) & 1;
  const uint64_t bs = __ballot(start), bq = __ballot(seed);
  const int wid = threadIdx.x >> 6;
  if (lane_id() == 0) { s_cnt[0][wid] = (uint32_t)__popcll(bs); s_cnt[1][wid] = (uint32_t)__popcll(bq); }
  __syncthreads();
  uint32_t os = w.blk_start[blockIdx.x], oq = w.blk_seed[blockIdx.x];
  for (int i = 0; i < wid; ++i) { os += s_cnt[0][i]; oq += s_cnt[1][i]; }
  const uint64_t lt = lanemask_lt();
  if (start) w.starts[os + (uint32_t)__popcll(bs & lt)] = (uint32_t)p;
  if (seed) w.seeds[oq + (uint32_t)__popcll(bq & lt)] = (uint32_t)p;
}

// Counts and per-event (and, for seeds, per-sector) ranges of the start and
// seed lists: entry i of a list writes the boundaries between its
// predecessor's unit and its own (all entries in parallel).
__global__ __launch_bounds__(TB) void k_ev_offsets(Ws w) {
  const uint32_t ns = w.blk_seed[w.nb], nst = w.blk_start[w.nb];
  const int64_t g0 = (int64_t)blockIdx.x * TB + threadIdx.x, gs = (int64_t)gridDim.x * TB;
  if (g0 == 0) { w.flags[F_NSEEDS] = ns; w.flags[F_NSTARTS] = nst; }
  const int64_t nsu = (int64_t)w.E * w.S;
  for (int64_t i = g0; i <= ns; i += gs) {
    const int64_t cur = i < ns ? (int64_t)(w.cru[w.seeds[i]] / (uint32_t)w.R) : nsu;
    const int64_t prev = i > 0 ? (int64_t)(w.cru[w.seeds[i - 1]] / (uint32_t)w.R) : -1;
    for (int64_t u = prev + 1; u <= cur; ++u) w.seed_su_off[u] = (uint32_t)i;
    const int64_t ce = i < ns ? cur / w.S : w.E, pe = i > 0 ? prev / w.S : -1;
    for (int64_t e = pe + 1; e <= ce; ++e) w.seed_ev_off[e] = (uint32_t)i;
  }
  const uint32_t per = (uint32_t)w.S * (uint32_t)w.R;
  for (int64_t i = g0; i <= nst; i += gs) {
    const int64_t ce = i < nst ? (int64_t)(w.cru[w.starts[i]] / per) : w.E;
    const int64_t pe = i > 0 ? (int64_t)(w.cru[w.starts[i - 1]] / per) : -1;
    for (int64_t e = pe + 1; e <= ce; ++e) w.start_ev_off[e] = (uint32_t)i;
  }
}

__global__ __launch_bounds__(TB) void k_start_tap(Ws w) {
  const uint32_t nst = w.flags[F_NSTARTS];
  const uint32_t per = (uint32_t)w.S * (uint32_t)w.R;
  for (int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x; i < nst; i += (int64_t)gridDim.x * TB) {
    const uint32_t p = w.starts[i];
    const int e = (int)(w.cru[p] / per);
    const EventOut& O = w.out[e];
    if (O.dbg_start) O.dbg_start[i - w.start_ev_off[e]] = w.cid[p];
  }
}

// ----------------------------------------------------------- a5: tracklets
struct Found { int32_t pos; float y, z, x; };


template <int G, class F>
__device__ __forceinline__ void group_steps(F&& f) {
  if constexpr (G >= 2) f(std::integral_constant<int, kDppXor1>{});
  if constexpr (G >= 4) f(std::integral_constant<int, kDppXor2>{});
  if constexpr (G >= 8) f(std::integral_constant<int, kDppMirror8>{});
}

// Closest cluster of a row unit (grid Q) to the predicted (y, z):
// d = dy^2/(Cyy + sy^2) + dz^2/(Czz + sz^2) <= chi2_ext, minimum (d, id).
// The box's first two z rows are two ranges of the grid-ordered array whose
// bounds are read together; then their entries, the first ones of both
// ranges issued before any is tested, so a step waits for memory twice
// rather than once per candidate.  With one lane per seed (G = 1) a lane
// loads two entries of each range at once and two more where a range holds
// them; with a group of G lanes per seed half of the lanes take the entries
// of each range, and the group's minimum is the result.  Loads may pass the
// range's end (kGridPad entries beyond the array): those entries are masked.
// The result does not depend on the order the candidates are visited in.
template <int G>
__device__ __forceinline__ Found search_row(const Ws& w, const GridParams& Q, const float p[5],
                                            const float C[15], int gl) {
  const float sy2 = C[0] + w.m.vy, sz2 = C[5] + w.m.vz;
  float isy = rcp_rn(sy2), isz = rcp_rn(sz2);
  if (__builtin_expect(max(rcp_key(sy2), rcp_key(sz2)) > kRcpKey, 0)) { isy = 1.0f / sy2; isz = 1.0f / sz2; }
  // the window only bounds the cells scanned: the hardware square root
  // (1 ulp) is enough under the 1e-4 relative and 1e-3 cm margins; the
  // bounds are taken in cells, with 2e-3 cells for the rounding inside the
  // grid (coordinates of at most 4097 cells; of a query further out, by the
  // window, it is 4e-7 of the window in cells, within the relative margin),
  // so the scanned cells stay a superset of those of every cluster passing
  // the cut
  const float wy = fmaf(w.ext_w, __builtin_amdgcn_sqrtf(sy2), 1e-3f);
  const float wz = fmaf(w.ext_w, __builtin_amdgcn_sqrtf(sz2), 1e-3f);
  const uint32_t nz = Q.nz(), ny = Q.ny();
  const float fz = (float)(nz - 1u), fy = (float)(ny - 1u);
  const float tz = (p[1] - Q.z0) * Q.inv_bz, hz = fmaf(wz, Q.inv_bz, 2e-3f);
  const float ty = (p[0] - Q.y0) * Q.inv_by, hy = fmaf(wy, Q.inv_by, 2e-3f);
  // (a NaN bound takes cell 0)
  const uint32_t iz0 = (uint32_t)fminf(fmaxf(tz - hz, 0.0f), fz), iz1 = (uint32_t)fminf(fmaxf(tz + hz, 0.0f), fz);
  const uint32_t iy0 = (uint32_t)fminf(fmaxf(ty - hy, 0.0f), fy), iy1 = (uint32_t)fminf(fmaxf(ty + hy, 0.0f), fy) + 1u;
  // (bd, pos) starts at (CUT, INT32_MAX): the first candidate with d <= CUT
  // replaces it, later ones must beat the best so far, so no separate test
  // of the cut (a NaN distance fails every comparison)
  Found best{INT32_MAX, 0.f, 0.f, 0.f};
  float bd = w.P.chi2_ext;
  auto consider = [&](const float4& c, bool in) {
    const float dY = c.x - p[0], dZ = c.y - p[1];
    const float d = fmaf(dZ * dZ, isz, (dY * dY) * isy);
    const int32_t pos = (int32_t)__float_as_uint(c.w);
    const bool take = in & ((d < bd) | ((d == bd) & (pos < best.pos)));
    best.pos = take ? pos : best.pos;
    best.y = take ? c.x : best.y;
    best.z = take ? c.y : best.z;
    best.x = take ? c.z : best.x;
    bd = take ? d : bd;
  };
  const uint32_t nzr = iz1 - iz0 + 1u;
  const uint16_t* ca = w.cell_off + (Q.cell_base + iz0 * ny);
  const uint16_t* cb = ca + (nzr > 1u ? ny : 0u);
  const float4* g = w.gbuf + Q.base;
  const uint32_t a0 = ca[iy0], a1 = ca[iy1], b0 = cb[iy0], b1 = cb[iy1];
  const uint32_t na = a1 - a0, nb = nzr > 1u ? b1 - b0 : 0u;
  if constexpr (G == 1) {
    // entries k .. n - 1 of e, four loads at a time (wide windows, most of a
    // seed's first steps, hold many: one load per trip kept whole waves
    // waiting, 64 small events 773 us instead of 716)
    auto rest = [&](const float4* e, uint32_t k, uint32_t n) {
      for (; k < n; k += 4u) {
        const float4 c0 = e[k], c1 = e[k + 1u], c2 = e[k + 2u], c3 = e[k + 3u];
        consider(c0, true); consider(c1, k + 1u < n); consider(c2, k + 2u < n); consider(c3, k + 3u < n);
      }
    };
    const float4* ga = g + a0;
    const float4* gb = g + b0;
    const float4 A0 = ga[0], A1 = ga[1], B0 = gb[0], B1 = gb[1];
    if (max(na, nb) > 2u) {
      const float4 A2 = ga[2], A3 = ga[3], B2 = gb[2], B3 = gb[3];
      consider(A2, na > 2u); consider(A3, na > 3u);
      consider(B2, nb > 2u); consider(B3, nb > 3u);
      rest(ga, 4u, na);
      rest(gb, 4u, nb);
    }
    consider(A0, na > 0u); consider(A1, na > 1u);
    consider(B0, nb > 0u); consider(B1, nb > 1u);
    for (uint32_t iz = 2; iz < nzr; iz += 2) {
      const uint16_t* cz = ca + iz * ny;
      const uint16_t* cy = cz + (iz + 1u < nzr ? ny : 0u);
      const uint32_t k0 = cz[iy0], k1 = cz[iy1], m0 = cy[iy0], m1 = cy[iy1];
      rest(g, k0, k1);
      if (iz + 1u < nzr) rest(g, m0, m1);
    }
  } else {
    constexpr uint32_t H = G / 2;
    const bool side = gl >= (int)H;
    const uint32_t n = side ? nb : na, j = (uint32_t)gl & (H - 1u);
    const float4* gs = g + ((side ? b0 : a0) + j);
    const float4 c0 = gs[0];
    if (n > j + H) {
      const float4 c1 = gs[H];
      consider(c1, true);
      for (uint32_t k = j + 2u * H; k < n; k += H) consider(g[(side ? b0 : a0) + k], true);
    }
    consider(c0, j < n);
    for (uint32_t iz = 2; iz < nzr; ++iz) {
      const uint16_t* cz = ca + iz * ny;
      const uint32_t k0 = cz[iy0], k1 = cz[iy1];
      for (uint32_t k = k0 + (uint32_t)gl; k < k1; k += G) consider(g[k], true);
    }
    // the group's minimum (d, pos), then the winner's coordinates (one lane
    // of the group holds it: or over the group)
    const int32_t mine = best.pos;
    group_steps<G>([&](auto ctl) {
      const float od = dpp_f32<ctl.value>(bd);
      const int32_t op = (int32_t)dpp_u32<ctl.value>((uint32_t)best.pos);
      const bool take = (od < bd) | ((od == bd) & (op < best.pos));
      bd = take ? od : bd;
      best.pos = take ? op : best.pos;
    });
    const bool won = mine == best.pos;
    uint32_t uy = won ? __float_as_uint(best.y) : 0u, uz = won ? __float_as_uint(best.z) : 0u;
    uint32_t ux = won ? __float_as_uint(best.x) : 0u;
    group_steps<G>([&](auto ctl) {
      uy |= dpp_u32<ctl.value>(uy);
      uz |= dpp_u32<ctl.value>(uz);
      ux |= dpp_u32<ctl.value>(ux);
    });
    best.y = __uint_as_float(uy);
    best.z = __uint_as_float(uz);
    best.x = __uint_as_float(ux);
  }
  if (best.pos == INT32_MAX) best.pos = -1;
  return best;
}

struct Acc { float tan_a, z_max; };

__device__ __forceinline__ bool accepted(float X, const Acc& a, const float p[5]) {
  const float lim = X * a.tan_a;
  return !(fabsf(p[0]) > lim || fabsf(p[1]) > a.z_max);
}

// Tracklet construction as a per-lane state machine: every loop iteration
// advances each lane by one row step, whatever phase it is in, so the lanes
// of a wave stay converged on the common transport.  Phases:
//   CHAIN  fit the next cluster of the seed's chain (no search);
//   UP     transport to the next row plane, acceptance, search, update;
//   BACK   transport back to the seed's first row, at most kBackRows rows
//          per step, no updates;
//   DOWN   as UP, downward from the row below the seed.
// Bound by the dependent chain of a seed: about 162 steps, each the scalar
// chain of a transport, two memory round trips of the search (cell offsets,
// entries) and an update.  What is not on that chain is kept short: the next
// step's plane, grid and chain record are loaded before the update, which
// covers their latency; phase changes are settled in one place; quotients
// and roots take the short sequences.  On one sector's 17 k clusters the
// kernel takes 277 us (476 with one lane per seed, a test per loaded entry
// and no L2 warming), on 0.77 M clusters 345 (494), on 3.8 M, where three
// waves per SIMD share the issue slots, 708 (805).
// With several lanes per seed, groups that have finished wait until a quarter
// of the wave does (or the whole wave has): then they write their tracklets
// and take the next seeds from a device counter (one atomic per wave).  The
// seed list is split into kXcd contiguous ranges with a counter each; a
// workgroup starts on the range of its XCD and moves on to the others once
// that one is used up.
enum : int { ST_CHAIN = 0, ST_UP = 1, ST_BACK = 2, ST_DOWN = 3, ST_DONE = 4, ST_IDLE = 5 };

// With one lane per seed the workgroup's waves are regrouped as lanes finish:
// every kRegroupEvery steps the live lanes are counted, and once fewer waves
// can hold them the lanes of the others move, through LDS, into the idle
// lanes of these (which waves go turns with the chunk, as a workgroup's
// waves lie on different SIMDs).  Seeds last between 17 and 167 steps, so
// waves that keep their lanes to the end run with 0.62 to 0.76 of them; lanes
// that take new seeds instead bring the steps of all phases (and the three
// long updates of a seed's start) into every step of the wave.  3.8 M
// clusters 775 -> 711 us, 64 small events 783 -> 773; counting every 4 steps
// 733 and 791, every 8 steps 716 and 780.
struct Regroup {
  static constexpr int kMoved = 128;   // lanes moved at once, at most
  static constexpr int kWords = 28;    // words of a lane's state
  uint32_t cnt[2][TB / 64];
  uint32_t state[kWords * kMoved];
};
constexpr uint32_t kRegroupEvery = 16;
// chunks of TB seeds of the largest of kXcd ranges
__device__ __forceinline__ uint32_t regroup_chunks(uint32_t ns) {
  return ((ns + kXcd - 1u) / kXcd + TB - 1u) / TB;
}

// G lanes per seed: every lane of a group holds the same state (the same
// expressions of the same values), the row search is shared out.
template <int G>
__device__ __forceinline__ void tracklets_wave(const Ws& w, const float* sX, const uint32_t ns, Regroup& grp) {
  const Acc acc{w.tan_a, w.z_max};
  const int R = w.R;
  const int gl = lane_id() & (G - 1);
  const uint64_t groups_before = (1ull << (lane_id() & ~(G - 1))) - 1ull;
  int phase = ST_IDLE;
  bool more = true;   // (wave-uniform) seeds may be left
  uint32_t s = 0;
  int32_t h0 = 0, nxt = -1;
  int r0 = 0, r = 0, rstate = 0, rlo = 0, rhi = 0, nhits = 0, gap = 0;
  uint32_t rubase = 0;
  float p[5], C[15], xc = 0.f;
  uint32_t iters = 0;
  int nupd = 0;   // Kalman updates of the current seed (the first three are compensated)
  // loaded one step ahead: the record of the next chain cluster (nxt), or
  // the plane and grid of the next row r
  float4 cn = make_float4(0.f, 0.f, 0.f, 0.f);
  float Xr = 0.f;
  GridParams Q{};
  // hit slots: with one lane per seed they go through a four-row buffer
  // (rows are visited in order within a phase), one 16-byte store per full
  // group of four rows -- the wave's lanes store to 64 lines, and single
  // stores cost the central event 60 us more; groups store each hit as it
  // comes (few lanes store, and a step is 25 instructions shorter)
  int32_t* hits = nullptr;   // the seed's slots of the first band
  int32_t wb0 = 0, wb1 = 0, wb2 = 0, wb3 = 0;
  int wbase = -1;
  uint32_t wmask = 0;
  auto slot = [&](int row) { return hits + ((int64_t)(row >> 3) * ((int64_t)w.seed_cap * 8) + (row & 7)); };
  auto flush = [&]() {
    int32_t* q = slot(wbase);
    if (wmask == 0xFu) {
      *(int4*)q = make_int4(wb0, wb1, wb2, wb3);
    } else {
      if (wmask & 1u) q[0] = wb0;
      if (wmask & 2u) q[1] = wb1;
      if (wmask & 4u) q[2] = wb2;
      if (wmask & 8u) q[3] = wb3;
    }
    wmask = 0;
  };
  auto put = [&](int row, int32_t v) {
    if constexpr (G > 1) {
      if (gl == 0) *slot(row) = v;
    } else {
      const int b = row & ~3;
      if (b != wbase && wmask != 0u) flush();
      wbase = b;
      const int q = row & 3;
      // value selects, not a store through a selected pointer: the latter
      // would put the buffer in scratch memory
      wb0 = q == 0 ? v : wb0;
      wb1 = q == 1 ? v : wb1;
      wb2 = q == 2 ? v : wb2;
      wb3 = q == 3 ? v : wb3;
      wmask |= 1u << q;
    }
  };
  // writes the finished tracklet
  auto finish = [&]() {
    if (G == 1 && wmask) flush();
    if (gl == 0) {
      float* st = w.tl_state + (int64_t)s * kTl;
#pragma unroll
      for (int i = 0; i < 5; ++i) st[i] = p[i];
#pragma unroll
      for (int i = 0; i < 15; ++i) st[5 + i] = C[i];
      w.tl_nhits[s] = nhits;
      w.tl_range[s] = rlo | (rhi << 16);
      w.tl_key[s] = ((uint64_t)(uint32_t)nhits << 40) | ((uint64_t)(255 - r0) << 32) |
                    (uint64_t)(0xFFFFFFFFu - w.cid[h0]);
    }
    phase = ST_IDLE;
  };
  // sets the lane up for seed s
  auto begin = [&]() {
    h0 = (int32_t)w.seeds[s];
    const uint32_t ru0 = w.cru[h0];
    r0 = (int)(ru0 % (uint32_t)R);
    rubase = ru0 - (uint32_t)r0;
    const float4 a0 = w.cpk[h0];
    const int32_t h1 = __float_as_int(a0.w);
    const float4 a1 = w.cpk[h1];
    const int32_t h2 = __float_as_int(a1.w);
    const float4 a2 = w.cpk[h2];
    float sdir, tdir;
    const float x0 = a0.x, y0 = a0.y, z0 = a0.z;
    chord_dir(x0, y0, z0, a2.x, a2.y, a2.z, sdir, tdir);
    p[0] = y0; p[1] = z0; p[2] = sdir; p[3] = tdir; p[4] = 0.0f;
    init_cov(C, w.m.vy, w.m.vz);
    nupd = 0;
    rlo = rhi = rstate = r0;
    xc = x0;
    hits = w.tl_hits + (int64_t)s * 8;
    wbase = -1;
    if (fabsf(sdir) < w.m.sin_max) {
      put(r0, h0);
      nhits = 1;
      nxt = h1;
      cn = a1;
      phase = ST_CHAIN;
    } else {
      nhits = 0;
      phase = ST_DONE;
    }
  };
  // the next step's inputs
  auto ahead = [&]() {
    if (phase == ST_CHAIN) {
      cn = w.cpk[nxt];
    } else if (phase < ST_DONE) {
      Xr = sX[r];
      Q = w.grid[rubase + (uint32_t)r];
    }
  };
  auto step = [&]() {
    // one row step: every active lane transports once (the target plane
    // depends on the phase), then the phase's own work follows
    const bool chain = phase == ST_CHAIN;
    const float X = chain ? cn.x : Xr;
    float my = cn.y, mz = cn.z;
    bool go = transport(p, C, xc, X, w.m);
    bool upd = false, wr = false;
    int prow = r;
    int32_t pval = nxt;
    // whether the lane's phase ends with this step (chain used up, no
    // further row, too many rows without a cluster, a refused transport) or
    // is on its way back: settled in one place below
    bool turn;
    if (chain) {
      nxt = __float_as_int(cn.w);
      wr = upd = go;
      rstate += go ? 1 : 0;
      nhits = go ? nhits + 1 : 0;
      prow = rstate;
      xc = go ? X : xc;
      turn = !go || nxt < 0;
    } else {
      const bool back = phase == ST_BACK;
      xc = go ? X : xc;
      turn = back;
      if (!back) {
        rstate = go ? r : rstate;
        go = go && accepted(X, acc, p);
        if (go) {
          const Found h = search_row<G>(w, Q, p, C, gl);
          pval = h.pos;
          my = h.y; mz = h.z;
          upd = h.pos >= 0;
          if (upd && h.x != X) {   // a cluster off its row's plane
            upd = go = transport(p, C, X, h.x, w.m);
            xc = go ? h.x : xc;
          }
          wr = go;
          nhits += upd ? 1 : 0;
          gap = upd ? 0 : gap + 1;
          go = go && gap <= w.P.max_gap;
        }
        const bool up = phase == ST_UP;
        rhi = wr && up ? r : rhi;
        rlo = wr && !up ? r : rlo;
        const int rn = up ? r + 1 : r - 1;
        turn = !go || (uint32_t)rn >= (uint32_t)R;
        r = turn ? r : rn;
      }
    }
    if (turn) {
      if (chain && !go) {
        rlo = rhi = r0;
        phase = ST_DONE;
      } else if (phase == ST_DOWN || (phase == ST_BACK && !go)) {
        phase = ST_DONE;
      } else {
        // the next row above the chain, the next stop on the way back to the
        // first row, or the first row below it
        if (chain) rhi = rstate;
        gap = 0;
        const int at = phase == ST_BACK ? r : rstate;
        if (chain && at + 1 < R) {
          r = at + 1;
          phase = ST_UP;
        } else if (at > r0 || chain) {
          r = max(r0, at - kBackRows);
          phase = ST_BACK;
        } else {
          r = r0 - 1;
          phase = r >= 0 ? ST_DOWN : ST_DONE;
        }
      }
    }
    ahead();   // (in flight during the update)
    if (wr) put(prow, pval);
    if (upd) {
      float dummy = 0.0f;
      if (nupd < TPCCA_GRAD_C2_UPDATES) update_c2(p, C, my, mz, w.m, dummy);
      else update(p, C, my, mz, w.m, dummy);
      ++nupd;
    }
  };
  if constexpr (G == 1) {
    // a workgroup's 256 consecutive seeds at a time, the chunks of an XCD's
    // range on that XCD
    const int wv = threadIdx.x >> 6;
    const uint32_t nchunk = kXcd * regroup_chunks(ns);
    uint32_t par = 0;
    for (uint32_t c = blockIdx.x; c < nchunk; c += gridDim.x) {
      const uint32_t x = c % kXcd, hi = (uint32_t)(((uint64_t)ns * (x + 1)) / kXcd);
      s = (uint32_t)(((uint64_t)ns * x) / kXcd) + c / kXcd * TB + threadIdx.x;
      phase = ST_IDLE;
      if (s < hi) begin();
      const int rot = (int)(c / kXcd + c / (32 * kXcd)) & 3;
      const int pw = (wv - rot) & 3;   // the wave's turn to be given up is last for 0
      int kept = TB / 64;
      iters = 0;
      while (true) {
        // (at most 2 R + 16 steps; a defect is an error instead of a hang)
        if (++iters > (1u << 22)) { atomicOr(&w.flags[F_ERR], ERR_STUCK); return; }
        if (phase < ST_DONE) step();
        if (iters % kRegroupEvery != 0u) continue;
        if (phase == ST_DONE) finish();
        const uint64_t live = __ballot(phase < ST_DONE);
        par ^= 1u;
        if (lane_id() == 0) grp.cnt[par][pw] = (uint32_t)__popcll(live);
        __syncthreads();
        uint32_t cnt[TB / 64], total = 0;
#pragma unroll
        for (int q = 0; q < TB / 64; ++q) { cnt[q] = grp.cnt[par][q]; total += cnt[q]; }
        if (total == 0u) break;
        const int need = (int)((total + 63u) >> 6);
        if (need >= kept) continue;
        kept = need;
        uint32_t first = 0, moved = 0;
#pragma unroll
        for (int q = 0; q < TB / 64; ++q) {
          if (q >= kept) moved += cnt[q];
          if (q < pw && (q < kept) == (pw < kept)) first += q < kept ? 64u - cnt[q] : cnt[q];
        }
        const bool keep = pw < kept;
        const uint32_t at = first + (uint32_t)__popcll((keep ? ~live : live) & lanemask_lt());
        if (!keep && phase < ST_DONE) {
          if (wmask) flush();
          uint32_t* q = grp.state + at;
          auto put_u = [&](int i, uint32_t v) { q[i * Regroup::kMoved] = v; };
          put_u(0, s); put_u(1, (uint32_t)h0); put_u(2, (uint32_t)nxt); put_u(3, rubase);
          put_u(4, (uint32_t)r0 | ((uint32_t)r & 255u) << 8 | (uint32_t)rstate << 16 | (uint32_t)phase << 24);
          put_u(5, (uint32_t)rlo | (uint32_t)rhi << 8 | (uint32_t)gap << 16);
          put_u(6, (uint32_t)nhits | (uint32_t)nupd << 16);
          put_u(7, __float_as_uint(xc));
#pragma unroll
          for (int i = 0; i < 5; ++i) put_u(8 + i, __float_as_uint(p[i]));
#pragma unroll
          for (int i = 0; i < 15; ++i) put_u(13 + i, __float_as_uint(C[i]));
          phase = ST_IDLE;
        }
        __syncthreads();
        if (keep && phase >= ST_DONE && at < moved) {
          const uint32_t* q = grp.state + at;
          auto get_u = [&](int i) { return q[i * Regroup::kMoved]; };
          s = get_u(0); h0 = (int32_t)get_u(1); nxt = (int32_t)get_u(2); rubase = get_u(3);
          const uint32_t a = get_u(4), b = get_u(5), d = get_u(6);
          r0 = (int)(a & 255u); r = (int)(a >> 8 & 255u); rstate = (int)(a >> 16 & 255u); phase = (int)(a >> 24);
          rlo = (int)(b & 255u); rhi = (int)(b >> 8 & 255u); gap = (int)(b >> 16);
          nhits = (int)(d & 0xFFFFu); nupd = (int)(d >> 16);
          xc = __uint_as_float(get_u(7));
#pragma unroll
          for (int i = 0; i < 5; ++i) p[i] = __uint_as_float(get_u(8 + i));
#pragma unroll
          for (int i = 0; i < 15; ++i) C[i] = __uint_as_float(get_u(13 + i));
          hits = w.tl_hits + (int64_t)s * 8;
          wbase = -1;
          wmask = 0;
          ahead();
        }
      }
    }
    return;
  }
  // seed range of this workgroup's XCD (workgroups are dispatched to the
  // XCDs round-robin), so that each XCD's L2 holds the grids of its sectors
  int rx = (int)(blockIdx.x % kXcd), tries = 0;
  while (true) {
    // every lane's steps are bounded (rows only move one way per phase), so
    // this cap is never reached by a correct kernel; it turns a defect into
    // an error instead of a hang
    if (++iters > (1u << 22)) { atomicOr(&w.flags[F_ERR], ERR_STUCK); break; }
    const uint64_t act = __ballot(phase < ST_DONE);
    // refills stall the whole wave (counter, atomic, seed set-up): take new
    // seeds only once a quarter of the lanes wait, or no lane is working
    if (act == 0ull || (more && 64 - __popcll(act) >= kRefillMin)) {
      if (phase == ST_DONE) {
        finish();
      }
      bool want = phase == ST_IDLE;
      uint64_t wm = more ? __ballot(want) : 0ull;
      while (wm) {
        const uint32_t lo = (uint32_t)(((uint64_t)ns * (uint32_t)rx) / kXcd);
        const uint32_t hi = (uint32_t)(((uint64_t)ns * (uint32_t)(rx + 1)) / kXcd);
        uint32_t* ctr = &w.flags[F_SEEDCTR + rx];
        // a fresh (L2-bypassing) read first: exhausted ranges cost no atomic
        uint32_t base = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (base < hi - lo) {
          const int leader = __ffsll((unsigned long long)wm) - 1;
          if (lane_id() == leader) base = atomicAdd(ctr, (uint32_t)__popcll(wm) / G);
          base = __shfl(base, leader, 64);
          if (want) {
            const uint64_t mine = (uint64_t)lo + base + (uint32_t)__popcll(wm & groups_before) / G;
            if (mine < hi) {
              want = false;
              s = (uint32_t)mine;
              begin();
            }
          }
        }
        wm = __ballot(want);
        if (wm) {
          // this range is used up: take seeds from the next one
          if (++tries >= kXcd) { more = false; break; }   // every range is used up
          rx = (rx + 1) % kXcd;
        }
      }
      if (__ballot(phase != ST_IDLE) == 0ull) break;
    }
    if (phase >= ST_DONE) continue;
    step();
  }
}

// Lanes per seed.  A launch with few seeds lasts as long as one seed's chain
// of about 162 dependent steps, so lanes that would idle shorten the step:
// with eight lanes a search is one load and a group minimum instead of four
// to eight loads and tests in a row.  More lanes are more waves, each issuing
// the whole step: the lines are one wave per SIMD at eight lanes (1024 SIMDs
// x 64 / 8 seeds) and two at four.  Measured per launch with 1 / 4 / 8 lanes:
// 2,337 seeds 445 / 334 / 296 us, 14,124 seeds 428 / 343 / 373, 28,188 seeds
// 462 / 396 / 537, 65,263 seeds 490 / 574 / 1479 (two lanes were never the
// best).
constexpr uint32_t kSeeds8 = 8192, kSeeds4 = 32768;
__device__ __forceinline__ int tracklet_lanes(uint32_t ns) { return ns <= kSeeds8 ? 8 : ns <= kSeeds4 ? 4 : 1; }

// Reads one word of every 128-byte line of [p, p + bytes), the lines spread
// over nt threads of which this is thread t (p and bytes: multiples of 4).
__device__ __forceinline__ void touch_lines(const void* p, int64_t bytes, int64_t t, int64_t nt) {
  uint32_t acc = 0;
  for (int64_t i = t * 128; i < bytes; i += nt * 128) acc |= *(const uint32_t*)((const char*)p + i);
  asm volatile("" ::"v"(acc));   // (the loads are kept, the value is not used)
}

// Workgroups without seeds read the search data of their XCD's seed range
// (grids, cell offsets, entries: written by the binning on any XCD), if it
// fits the XCD's 4 MB L2 beside what else is there, so that the dependent
// loads of the search steps find it in that L2 instead of behind it (a
// sector's 17 k clusters: 339 -> 298 us).  kWarmGrid: launched at least, so
// that even the smallest events have such workgroups on every XCD.
constexpr int64_t kWarmBytes = (int64_t)3 << 20;
constexpr unsigned kWarmGrid = 512;

// (four waves per SIMD: with 129 registers, three, 3.8 M clusters take 1,056 us
// instead of 708)
__global__ __launch_bounds__(TB, 4) void k_tracklets(Ws w) {
  __shared__ float sX[256];
  __shared__ Regroup grp;
  for (int r = threadIdx.x; r < w.R; r += TB) sX[r] = w.row_x[r];
  __syncthreads();
  const uint32_t ns = w.flags[F_NSEEDS];
  const int G = tracklet_lanes(ns);
  // when the lanes of the lower workgroups already outnumber the seeds they
  // take (and, by refills, finish) them all: this one has no seeds to take
  const int64_t busy = G == 1 ? (int64_t)kXcd * regroup_chunks(ns) : ((int64_t)ns + TB / G - 1) / (TB / G);
  if ((int64_t)blockIdx.x >= busy) {
    const uint32_t x = blockIdx.x % kXcd;
    const uint32_t lo = (uint32_t)(((uint64_t)ns * x) / kXcd), hi = (uint32_t)(((uint64_t)ns * (x + 1)) / kXcd);
    if (lo >= hi) return;
    const uint32_t u0 = w.cru[w.seeds[lo]] / (uint32_t)w.R * (uint32_t)w.R;
    const uint32_t u1 = (w.cru[w.seeds[hi - 1]] / (uint32_t)w.R + 1u) * (uint32_t)w.R;
    const int64_t c0 = w.ru_off[u0], c1 = w.ru_off[u1], k0 = w.cell_base[u0], k1 = w.cell_base[u1];
    const int64_t bytes = (c1 - c0) * 16 + (k1 - k0) * 2 + (int64_t)(u1 - u0) * (int64_t)sizeof(GridParams);
    if (bytes > kWarmBytes) return;
    const int64_t b0 = (busy + kXcd - 1 - x) / kXcd;   // (first idle workgroup of this XCD, in its own numbering)
    const int64_t nt = ((int64_t)(gridDim.x + kXcd - 1 - x) / kXcd - b0) * TB;
    const int64_t t = ((int64_t)(blockIdx.x / kXcd) - b0) * TB + threadIdx.x;
    touch_lines(w.grid + u0, (int64_t)(u1 - u0) * (int64_t)sizeof(GridParams), t, nt);
    // (words of two offsets from an even one; the array has an entry more than it needs)
    const int64_t ka = k0 & ~(int64_t)1;
    touch_lines(w.cell_off + ka, (k1 - ka + 1) / 2 * 4, t, nt);
    touch_lines(w.gbuf + c0, (c1 - c0) * 16, t, nt);
    return;
  }
  if (G == 8) tracklets_wave<8>(w, sX, ns, grp);
  else if (G == 4) tracklets_wave<4>(w, sX, ns, grp);
  else tracklets_wave<1>(w, sX, ns, grp);
}

// ----------------------------------------------------------- a6: selection
// Ownership by bands of kBandRows pad rows of one (event, sector): tracklets
// of different sectors never share a cluster, so the workgroup of a band
// scans its sector's tracklets (a thread per tracklet and band) and
// takes the key maximum of each of the band's clusters with LDS atomics,
// then writes the mask of each tracklet's owned rows.  A band with more than
// kBandCap clusters uses global atomics on the (zeroed) owner array instead.
constexpr int kBandRows = 8;
constexpr int kBandCap = 6144;
// threads of an ownership workgroup: 1024 where the sectors hold many
// tracklets (short chains of dependent loads per thread), TB for smaller
// events
constexpr int TBO = 1024;

struct Band {
  int64_t su;        // (event, sector)
  int r_lo, r_hi;    // rows
  uint32_t c0, nc;   // canonical positions
};
__device__ __forceinline__ Band band_of(const Ws& w, uint32_t b) {
  const uint32_t nband = (uint32_t)((w.R + kBandRows - 1) / kBandRows);
  Band d;
  d.su = b / nband;
  d.r_lo = (int)(b % nband) * kBandRows;
  d.r_hi = min(d.r_lo + kBandRows, w.R) - 1;
  d.c0 = w.ru_off[d.su * w.R + d.r_lo];
  d.nc = w.ru_off[d.su * w.R + d.r_hi + 1] - d.c0;
  return d;
}

// One band by the nt threads of the workgroup; s_own: LDS words for cap
// clusters.
__device__ __forceinline__ void own_band(const Ws& w, const Band& d, unsigned long long* s_own, uint32_t cap,
                                         uint32_t nt) {
  const int64_t su = d.su;
  const int r_lo = d.r_lo, r_hi = d.r_hi;
  const uint32_t c0 = d.c0, nc = d.nc;
  const bool lds = nc <= cap;
  // every cluster lies in one band, whose workgroup alone takes its
  // maxima: in LDS or, for bands above the LDS capacity, by global atomics
  // on entries this workgroup clears
  if (lds)
    for (uint32_t i = threadIdx.x; i < nc; i += nt) s_own[i] = 0ull;
  else
    for (uint32_t i = threadIdx.x; i < nc; i += nt) w.owner[c0 + i] = 0ull;
  __syncthreads();
  // one thread per tracklet: the band's eight hit slots are two aligned
  // 16-byte loads, and the band's slots of consecutive tracklets are
  // contiguous (hit_slot), so a wave reads them in whole lines
  static_assert(kBandRows == 8, "two int4 of hit slots per band");
  const uint32_t s0 = w.seed_su_off[su], s1 = w.seed_su_off[su + 1];
  constexpr int kUn = 2;   // passes whose loads are issued together
  for (uint32_t sb = s0; sb < s1; sb += nt * kUn) {
    int32_t rg[kUn], nh[kUn];
    int4 hh[kUn], hh2[kUn];
    unsigned long long key[kUn];
    bool ok[kUn];
#pragma unroll
    for (int u = 0; u < kUn; ++u) {
      const uint32_t s = sb + u * nt + threadIdx.x;
      ok[u] = s < s1;
      const uint32_t sc = ok[u] ? s : s0;
      rg[u] = w.tl_range[sc];
      nh[u] = w.tl_nhits[sc];
      const int32_t* hb = w.tl_hits + hit_slot(w.seed_cap, sc, r_lo);   // (r_lo: a band's first row)
      hh[u] = *(const int4*)hb;
      hh2[u] = *(const int4*)(hb + 4);
      key[u] = w.tl_key[sc];
    }
#pragma unroll
    for (int u = 0; u < kUn; ++u) {
      if (!ok[u] || nh[u] < w.P.min_hits) continue;
      const int rlo = rg[u] & 0xFFFF, rhi = rg[u] >> 16;
      const int32_t hq[8] = {hh[u].x, hh[u].y, hh[u].z, hh[u].w, hh2[u].x, hh2[u].y, hh2[u].z, hh2[u].w};
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int r = r_lo + q;
        const int32_t h = hq[q];
        if (r > r_hi || r < rlo || r > rhi || h < 0) continue;
        if (lds) atomicMax(&s_own[(uint32_t)h - c0], key[u]);
        else if (w.owner[h] < key[u]) atomicMax((unsigned long long*)&w.owner[h], key[u]);
      }
    }
  }
  __syncthreads();
  // the band's maxima are final: every tracklet of the sector gets the mask
  // of the band's rows whose hit it owns (its key is the maximum there),
  // written beside those of the neighbouring tracklets
  uint8_t* mk = w.own_mask + (int64_t)(r_lo >> 3) * w.seed_cap;
  for (uint32_t s = s0 + threadIdx.x; s < s1; s += nt) {
    const int32_t rg = w.tl_range[s];
    const int nh = w.tl_nhits[s];
    const int32_t* hb = w.tl_hits + hit_slot(w.seed_cap, s, r_lo);
    const int4 a = *(const int4*)hb, b = *(const int4*)(hb + 4);
    const unsigned long long key = w.tl_key[s];
    uint32_t m = 0;
    if (nh >= w.P.min_hits) {
      const int rlo = rg & 0xFFFF, rhi = rg >> 16;
      const int32_t hq[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int r = r_lo + q;
        const int32_t h = hq[q];
        if (r > r_hi || r < rlo || r > rhi || h < 0) continue;
        // (bands above the LDS capacity: the maxima are this workgroup's
        // atomics, read past the compute unit's cache)
        const unsigned long long mx =
            lds ? s_own[(uint32_t)h - c0] : __hip_atomic_load(&w.owner[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (mx == key) m |= 1u << q;
      }
    }
    mk[s] = (uint8_t)m;
  }
}

// Every band a workgroup, or the bands that k_owner_small has listed.
__global__ __launch_bounds__(TBO) void k_owner(Ws w) {
  __shared__ unsigned long long s_own[kBandCap];
  if (!ru_lists(w.RU)) {
    own_band(w, band_of(w, blockIdx.x), s_own, kBandCap, blockDim.x);
    return;
  }
  const uint32_t cnt = w.flags[F_LBANDS];
  for (uint32_t i = blockIdx.x; i < cnt; i += gridDim.x) {
    own_band(w, band_of(w, w.ru_big[i]), s_own, kBandCap, blockDim.x);
    __syncthreads();   // LDS is reused by the next band
  }
}

// Batches of events: two waves and 16 KB of LDS per band, so that ten bands
// share a compute unit (a band of a small event is a chain of four dependent
// memory trips; workgroups with LDS for the largest bands leave three on a
// unit: 64 small events 223 -> 96 us).  Larger bands are listed for k_owner,
// which takes them with TBO threads (24-collision frame: 60 -> 34 and 30).
constexpr uint32_t kSmallBand = 2048;
constexpr uint32_t kSmallBandNT = 128;
__global__ __launch_bounds__(kSmallBandNT) void k_owner_small(Ws w) {
  __shared__ unsigned long long s_own[kSmallBand];
  const Band d = band_of(w, blockIdx.x);
  if (d.nc > kSmallBand) {
    // (the list of large row units has been used up by the row kernels)
    if (threadIdx.x == 0) w.ru_big[atomicAdd(&w.flags[F_LBANDS], 1u)] = blockIdx.x;
    return;
  }
  own_band(w, d, s_own, kSmallBand, kSmallBandNT);
}

// ------------------------------------------------ a6/a7: accept + final fit
// Acceptance: count the hits a tracklet owns (outermost first), keep them as
// a compact list tl_own[s][0..cnt) and flag the tracklet if it owns at least
// min_hits and owned_num/owned_den of its hits.  One wave per tracklet: 64
// rows per pass from the outermost down, compacted with a ballot.
__global__ __launch_bounds__(TB) void k_accept(Ws w) {
  // half a wave (32 lanes) per tracklet, two tracklets per wave in flight;
  // the tracklets of one XCD's seed range go to that XCD's workgroups
  const uint32_t ns = w.flags[F_NSEEDS];
  const int lane = lane_id(), hl = lane & 31;
  const uint64_t half = (lane < 32) ? 0x00000000FFFFFFFFull : 0xFFFFFFFF00000000ull;
  const uint32_t x = blockIdx.x % kXcd;
  const int64_t lo = (int64_t)(((uint64_t)ns * x) / kXcd), hi = (int64_t)(((uint64_t)ns * (x + 1)) / kXcd);
  const int64_t first = lo + (int64_t)(blockIdx.x / kXcd) * (TB / 32) + (threadIdx.x >> 5);
  const int64_t stride = (int64_t)(gridDim.x / kXcd) * (TB / 32);
  for (int64_t s = first; s < hi; s += stride) {
    uint32_t acc = 0, cnt = 0;
    // the two are loaded together (one memory round trip): no branch
    // around the rest, whose loads and stores are predicated on ok instead
    const int nh = w.tl_nhits[s];
    const int32_t rg = w.tl_range[s];
    const bool ok = nh >= w.P.min_hits;
    const int rlo = rg & 0xFFFF, rhi = rg >> 16;
    const int32_t* hits = w.tl_hits + s * 8;
    const int64_t bstride = (int64_t)w.seed_cap * 8;
    const uint8_t* mk = w.own_mask + s;
    int32_t* own = w.tl_own + s * w.R;
    // a list spans at most eight passes of 32 rows (<= 255 rows): read all
    // hit slots and the owned-row masks of their bands, then compact pass
    // by pass
    constexpr int kPass = 8;
    int32_t h[kPass];
    uint32_t mb[kPass];
#pragma unroll
    for (int c = 0; c < kPass; ++c) {
      const int r = rhi - hl - 32 * c;
      const bool in = ok && r >= rlo;
      h[c] = in ? hits[(int64_t)(r >> 3) * bstride + (r & 7)] : -1;
      mb[c] = in ? ((uint32_t)mk[(int64_t)(r >> 3) * w.seed_cap] >> (r & 7)) & 1u : 0u;
    }
#pragma unroll
    for (int c = 0; c < kPass; ++c) {
      const bool mine = h[c] >= 0 && mb[c] != 0u;
      const uint64_t m = __ballot(mine) & half;
      if (mine) own[cnt + (uint32_t)__popcll(m & lanemask_lt())] = h[c];
      cnt += (uint32_t)__popcll(m);
    }
    acc = (ok && (int)cnt >= w.P.min_hits && (int64_t)w.P.owned_den * cnt >= (int64_t)w.P.owned_num * nh) ? 1u : 0u;
    if (hl == 0) {
      w.acc_flag[s] = acc;
      w.own_cnt[s] = acc ? cnt : 0u;
    }
  }
  // slots past the seed count (scanned with the others)
  for (int64_t s = (int64_t)ns + (int64_t)blockIdx.x * TB + threadIdx.x; s < w.seed_cap;
       s += (int64_t)gridDim.x * TB) {
    w.acc_flag[s] = 0u;
    w.own_cnt[s] = 0u;
  }
}

__global__ __launch_bounds__(TB) void k_acc_list(Ws w) {
  for (int64_t s = (int64_t)blockIdx.x * TB + threadIdx.x; s < w.seed_cap; s += (int64_t)gridDim.x * TB) {
    const uint32_t a = w.acc_off[s];
    if (w.acc_off[s + 1] != a) w.acc_list[a] = (uint32_t)s;
  }
}

// Final fit of every accepted tracklet (dense over the accepted list):
// outermost owned hit first, direction from the chord to the hit two
// positions inward, q/pT prior from following.  One lane per track: bound by
// the chain of at most 158 dependent steps, about 270 instructions each (70 %
// of its time is their issue).  The first steps, whose updates are
// compensated (1,200 instructions), have a loop of their own, so that the
// code of the others, unrolled by four, stays short (0.77 M clusters: 122 ->
// 107 us with the shorter quotients, 24-collision frame 195 -> 154).
__global__ __launch_bounds__(64) void k_refit(Ws w) {
  const uint32_t na = w.acc_off[w.seed_cap];
  for (int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x; i < na; i += (int64_t)gridDim.x * 64) {
    const int64_t s = w.acc_list[i];
    const int32_t* own = w.tl_own + s * w.R;
    const uint32_t cnt = w.own_cnt[s];   // (>= min_hits >= 3)
    float p[5], C[15], sdir, tdir;
    const int32_t o0 = own[0];
    const float4 c0 = w.cpk[o0];
    float4 c1 = w.cpk[own[1]], c2 = w.cpk[own[2]], c3 = w.cpk[3 < cnt ? own[3] : o0];
    // hit records are read four steps ahead of their use and hit indices
    // eight steps ahead, so loads overlap the filter steps: one register slot
    // per step of the unrolled loop, refilled right after its use, and no
    // register moves (which would wait for the loads in flight)
    auto index = [&](uint32_t k) { return own[k < cnt ? k : 0u]; };   // (past the end: the first hit, never used)
    constexpr uint32_t kc = TPCCA_GRAD_C2_UPDATES + 1;
    float4 q0 = w.cpk[index(kc)], q1 = w.cpk[index(kc + 1)], q2 = w.cpk[index(kc + 2)], q3 = w.cpk[index(kc + 3)];
    int32_t j0 = index(kc + 4), j1 = index(kc + 5), j2 = index(kc + 6), j3 = index(kc + 7);
    chord_dir(c2.x, c2.y, c2.z, c0.x, c0.y, c0.z, sdir, tdir);
    const float kpr = w.tl_state[s * kTl + 4];
    p[0] = c0.y; p[1] = c0.z; p[2] = sdir; p[3] = tdir; p[4] = kpr;
    init_cov(C, w.m.vy, w.m.vz);
    float chi2 = 0.0f;
    bool ok = fabsf(sdir) < w.m.sin_max;
    float xc = c0.x;
    for (uint32_t k = 1; ok && k < kc && k < cnt; ++k) {
      ok = transport(p, C, xc, c1.x, w.m);
      if (ok) {
        update_c2(p, C, c1.y, c1.z, w.m, chi2);
        xc = c1.x;
      }
      c1 = c2;
      c2 = c3;
    }
    auto step = [&](float4& q, int32_t& j, uint32_t k) {
      if (ok && k < cnt) {
        ok = transport(p, C, xc, q.x, w.m);
        if (ok) {
          update(p, C, q.y, q.z, w.m, chi2);
          xc = q.x;
        }
      }
      q = w.cpk[j];
      j = index(k + 8);
    };
    for (uint32_t k = kc; ok && k < cnt; k += 4) {
      step(q0, j0, k);
      step(q1, j1, k + 1);
      step(q2, j2, k + 2);
      step(q3, j3, k + 3);
    }
    if (ok) {
      float* rf = w.rf + s * kRf;
      rf[0] = xc;
#pragma unroll
      for (int q = 0; q < 5; ++q) rf[1 + q] = p[q];
#pragma unroll
      for (int q = 0; q < 15; ++q) rf[6 + q] = C[q];
      rf[21] = chi2;
      rf[22] = kpr;
    } else {
      w.own_cnt[s] = 0u;          // a failed fit produces no track
    }
  }
}


// Per-event totals and the capacity check.
__global__ __launch_bounds__(TB) void k_totals(Ws w) {
  __shared__ int s_fit;
  if (threadIdx.x == 0) s_fit = 1;
  __syncthreads();
  for (int e = threadIdx.x; e < w.E; e += TB) {
    const uint32_t b = w.seed_ev_off[e], en = w.seed_ev_off[e + 1];
    const int64_t nt = (int64_t)w.trk_flag[en] - (int64_t)w.trk_flag[b];
    const int64_t nh = (int64_t)w.hit_cnt[en] - (int64_t)w.hit_cnt[b];
    w.ev_res[e * 4 + 0] = nt;
    w.ev_res[e * 4 + 1] = nh;
    w.ev_res[e * 4 + 2] = (int64_t)w.start_ev_off[e + 1] - (int64_t)w.start_ev_off[e];
    const EventOut& O = w.out[e];
    const bool fit = nt <= O.cap_tracks && nh <= O.cap_hits;
    w.ev_res[e * 4 + 3] = fit ? 1 : 0;
    if (!fit) atomicAnd(&s_fit, 0);
  }
  __syncthreads();
  const bool go = s_fit && w.flags[F_ERR] == 0u;
  if (threadIdx.x == 0) w.flags[F_FITS] = go ? 1u : 0u;
  if (go)
    for (int e = threadIdx.x; e < w.E; e += TB)
      w.out[e].hit_off[w.ev_res[e * 4 + 0]] = (int32_t)w.ev_res[e * 4 + 1];
}

// Half a wave per accepted tracklet (the ordered accepted list; those whose
// fit failed are skipped), two in flight per wave, the tracks of one XCD's
// range on that XCD (neighbouring tracks share the lines of their clusters'
// ids).  A lane stores one scalar and every 32nd hit, innermost first.  Bound
// by a chain of dependent memory trips: everything indexed by the tracklet
// is read in the first, the hits before their count is known; a wave per
// tracklet, its hits read after the count, took 154 us, this way 117
// (64 small events; 3.8 M clusters 47 and 35).
constexpr unsigned kWriteGrid = 2048;   // workgroups resident at once (a multiple of kXcd)
__global__ __launch_bounds__(TB) void k_write(Ws w) {
  if (w.flags[F_FITS] == 0u) return;
  const uint32_t na = w.acc_off[w.seed_cap];
  const int hl = lane_id() & 31;
  // the lane's scalar: its value's place in the fit record, its output array
  // and its place in the track's entry there
  int rfi = hl, at = 0, per = 1;
  const auto field = [](size_t o) { return (int)o; };
  int fo = 0;
  if (hl < 5) { rfi = 1 + hl; fo = field(offsetof(EventOut, p)); at = hl; per = 5; }
  else if (hl < 20) { rfi = 1 + hl; fo = field(offsetof(EventOut, cov)); at = hl - 5; per = 15; }
  else if (hl == 20) { rfi = 0; fo = field(offsetof(EventOut, x_ref)); }
  else if (hl == 21) fo = field(offsetof(EventOut, chi2));
  else if (hl == 22) fo = field(offsetof(EventOut, k_prior));
  else if (hl == 23) fo = field(offsetof(EventOut, ndf));
  else if (hl == 24) fo = field(offsetof(EventOut, hit_off));
  else fo = field(offsetof(EventOut, sector));
  if (hl > 22) rfi = 0;
  const uint32_t x = blockIdx.x % kXcd;
  const int64_t lo = (int64_t)(((uint64_t)na * x) / kXcd), hi = (int64_t)(((uint64_t)na * (x + 1)) / kXcd);
  const int64_t stride = (int64_t)(gridDim.x / kXcd) * (TB / 32);
  for (int64_t i = lo + (int64_t)(blockIdx.x / kXcd) * (TB / 32) + (threadIdx.x >> 5); i < hi; i += stride) {
    const int64_t s = w.acc_list[i];
    const uint32_t t0 = w.trk_flag[s], t1 = w.trk_flag[s + 1];
    const uint32_t c0 = w.hit_cnt[s], c1 = w.hit_cnt[s + 1];
    const int32_t h0 = (int32_t)w.seeds[s];
    const float v = w.rf[s * kRf + rfi];
    const int32_t* own = w.tl_own + s * w.R;
    constexpr int kPass = 8;   // (at most 255 rows)
    int32_t h[kPass];
#pragma unroll
    for (int c = 0; c < kPass; ++c)
      if (32 * c < w.R) h[c] = own[min(hl + 32 * c, w.R - 1)];
    if (t1 == t0) continue;
    const uint32_t n = c1 - c0;
    const uint32_t vsec = w.cru[h0] / (uint32_t)w.R;
    uint32_t id[kPass];
#pragma unroll
    for (int c = 0; c < kPass; ++c)
      if ((uint32_t)(hl + 32 * c) < n) id[c] = w.cid[h[c]];
    const int e = (int)(vsec / (uint32_t)w.S);
    const EventOut& O = w.out[e];
    // offsets within the event (a single event starts at zero)
    uint32_t j = t0, o = c0;
    if (w.E > 1) {
      const uint32_t sb = w.seed_ev_off[e];
      j = t0 - w.trk_flag[sb];
      o = c0 - w.hit_cnt[sb];
    }
    char* out = *(char* const*)((const char*)&O + fo);
    uint32_t* hid = O.hit_id;
    if (hl < 25) {
      const uint32_t b = hl < 23 ? __float_as_uint(v) : hl == 23 ? 2u * n - 5u : o;
      if (out) ((uint32_t*)out)[(int64_t)j * per + at] = b;
    } else if (hl == 25) {
      ((uint8_t*)out)[j] = (uint8_t)(vsec % (uint32_t)w.S);
    }
#pragma unroll
    for (int c = 0; c < kPass; ++c) {
      const uint32_t q = (uint32_t)(hl + 32 * c);
      if (q < n) hid[o + (n - 1u - q)] = id[c];
    }
  }
}

}  // namespace

// Exclusive scan of n values into out[0 .. n] (out[n] = total); part holds
// 2 (n / 1024 + 2) values.
hipError_t scan_exclusive_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* part, hipStream_t st) {
  return scan_u32(in, out, n, part, st);
}

// Persistent grid of the tracklet kernel: one lane per possible seed (the
// workgroups past the actual seed count leave at once), or the tuned value.
unsigned tracklet_grid(const Ws& w) {
  if (w.tracklet_grid > 0) return (unsigned)w.tracklet_grid;
  return std::max(blocks_for(w.seed_cap, 1 << 16), kWarmGrid);
}

namespace {
// FP32 building blocks of the bit-exact contract, elementwise, compiled with
// the flags of the tracking kernels: op 0 sqrt_rn_normal(a), 1 a / b,
// 2 1 / a and 3 sqrt(a), each by the kernels' short sequence in its range
// and the general one outside.  Where both reciprocal sequences apply a
// difference between them gives NaN.
__global__ __launch_bounds__(TB) void k_fp32_probe(int op, int64_t n, const float* __restrict__ a,
                                                   const float* __restrict__ b, float* __restrict__ out) {
  for (int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x; i < n; i += (int64_t)gridDim.x * TB) {
    const float x = a[i];
    float r;
    if (op == 0) r = sqrt_rn_normal(x);
    else if (op == 1) r = x / b[i];
    else if (op == 2) {
      const float q = rcp_rn_special(x);
      r = x == 0.0f || isinf(x) ? q : rcp_rn_any(x);
      if (rcp_key(x) <= kRcpKey && f32_bits(q) != f32_bits(r)) r = __int_as_float(0x7fc00000);
    }
    else r = x >= 0x1p-96f && x <= 0x1p+97f ? sqrt_rn_pos(x) : sqrtf(x);
    out[i] = r;
  }
}
}  // namespace

hipError_t fp32_probe(int op, int64_t n, const float* a, const float* b, float* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_fp32_probe<<<blocks_for(n, 1 << 14), TB, 0, st>>>(op, n, a, b, out);
  return hipGetLastError();
}

hipError_t fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_fill<<<blocks_for(n, 4096), TB, 0, st>>>(p, v, n);
  return hipGetLastError();
}

hipError_t run_pipeline(const Ws& w, hipStream_t st, const PhaseEvents* pe) {
  hipError_t e;
#define TPCCA_CHECK(x) do { if ((e = (x)) != hipSuccess) return e; } while (0)
#define TPCCA_MARK(i) do { if (pe) TPCCA_CHECK(hipEventRecord(pe->ev[i], st)); } while (0)
  TPCCA_MARK(PH_ZERO);
  k_zero2<<<blocks_for(F_COUNT + w.RU, 4096), TB, 0, st>>>(w.flags, F_COUNT, w.ru_count, w.RU);
  TPCCA_CHECK(hipGetLastError());
  TPCCA_MARK(PH_COUNT);
  const unsigned nchunk = (unsigned)chunk_cap(w.N, w.E);
  k_count<<<nchunk, TBB, 0, st>>>(w);
  TPCCA_CHECK(hipGetLastError());
  TPCCA_MARK(PH_SCAN);
  if (w.RU <= kScanSmall) {
    k_scan_rows<<<1, kScanNT, 0, st>>>(w);
    TPCCA_CHECK(hipGetLastError());
  } else {
    k_cell_caps<<<blocks_for(w.RU), TB, 0, st>>>(w);
    TPCCA_CHECK(scan_u32x2(w.ru_count, w.ru_off, w.cell_cap, w.cell_base, w.RU, w.scan_tmp, st));
    TPCCA_CHECK(fill_u32(w.ru_count, 0u, w.RU, st));
  }
  TPCCA_MARK(PH_SCATTER);
  k_scatter<<<nchunk, TBB, 0, st>>>(w);
  TPCCA_MARK(PH_ROWS);
  const bool lists = ru_lists(w.RU);
  const unsigned g_all = (unsigned)w.RU;
  const unsigned g_mid = lists ? std::min(g_all, kListGrid) : g_all, g_big = lists ? std::min(g_all, kListGridBig) : g_all;
  const unsigned g_wave = (unsigned)((w.RU + TB / 64 - 1) / (TB / 64));
  k_rows_tiny<<<g_wave, TB, 0, st>>>(w);
  k_rows_wave<<<lists ? std::min(g_wave, kListGrid) : g_wave, TB, 0, st>>>(w);
  k_rows<false><<<g_mid, TB, 0, st>>>(w);
  k_rows<true><<<g_big, TB, 0, st>>>(w);
  TPCCA_CHECK(hipGetLastError());
  const unsigned nbN = (unsigned)w.nb;
  TPCCA_MARK(PH_LINKS);
  // Rows of a band: with many row units eight (64 small events 315 us, with
  // six 338, with ten 333; a 24-collision frame 93, 88 and 111); with few (one
  // event) two, for more workgroups (0.77 M clusters 42 us with four, 36 with
  // two; one sector's 22 k 14.5 and 10.7).  LDS for one and a half times the
  // band that an average row would make, within limits (a single event:
  // fixed, as one sector may hold all of it).
  const int lr = lists ? kLinkRows : 2;
  const int64_t want = lists ? (3 * (lr + 2) * (w.N / w.RU + 1) / 2 + 63) / 64 * 64 : 768;
  const uint32_t lcap = (uint32_t)std::min<int64_t>(std::max<int64_t>(want, kLinkEMin), kLinkE);
  k_links_band<<<(unsigned)((int64_t)w.E * w.S * ((w.R + lr - 1) / lr)), TB,
                 lcap * sizeof(float4) + link_words(lcap) * sizeof(uint32_t), st>>>(w, lr, lcap);
  k_links<<<g_big, TB, 0, st>>>(w, lcap);
  TPCCA_MARK(PH_CLEAN);
  k_clean<<<nbN, TB, 0, st>>>(w);
  TPCCA_MARK(PH_COMPACT);
  TPCCA_CHECK(scan_u32x2(w.blk_start, w.blk_start, w.blk_seed, w.blk_seed, w.nb, w.scan_tmp, st));
  k_compact<<<nbN, TB, 0, st>>>(w);
  k_ev_offsets<<<blocks_for(w.N / 2 + 2, 4096), TB, 0, st>>>(w);
  if (w.taps) k_start_tap<<<blocks_for(w.N / 2 + 1, 2048), TB, 0, st>>>(w);
  TPCCA_CHECK(hipGetLastError());
  TPCCA_MARK(PH_TRACKLETS);
  k_tracklets<<<tracklet_grid(w), TB, 0, st>>>(w);
  TPCCA_CHECK(hipGetLastError());
  TPCCA_MARK(PH_OWNER);
  const unsigned nbands = (unsigned)((int64_t)w.E * w.S * ((w.R + kBandRows - 1) / kBandRows));
  if (lists) k_owner_small<<<nbands, kSmallBandNT, 0, st>>>(w);
  k_owner<<<lists ? std::min(nbands, kListGrid) : nbands,
            lists || w.N / std::max(w.E, 1) >= ((int64_t)1 << 20) ? TBO : TB, 0, st>>>(w);
  TPCCA_MARK(PH_REFIT);
  k_accept<<<xcd_blocks(w.seed_cap * 32), TB, 0, st>>>(w);
  TPCCA_CHECK(scan_u32(w.acc_flag, w.acc_off, w.seed_cap, w.scan_tmp, st));
  k_acc_list<<<blocks_for(w.seed_cap, 4096), TB, 0, st>>>(w);
  k_refit<<<blocks_for(w.seed_cap + 1, 16384), 64, 0, st>>>(w);
  TPCCA_MARK(PH_OUTPUT);
  // track offsets (indicator of a fitted track) and hit offsets (owned
  // count) from the owned counts, by the same launches
  TPCCA_CHECK(scan_u32x2(w.own_cnt, w.trk_flag, w.own_cnt, w.hit_cnt, w.seed_cap, w.scan_tmp, st, 1));
  k_totals<<<1, TB, 0, st>>>(w);
  k_write<<<std::min(xcd_blocks(w.seed_cap * 32), kWriteGrid), TB, 0, st>>>(w);
  TPCCA_CHECK(hipGetLastError());
  TPCCA_MARK(PH_N);
#undef TPCCA_MARK
#undef TPCCA_CHECK
  return hipSuccess;
}

}  // namespace tpcca
