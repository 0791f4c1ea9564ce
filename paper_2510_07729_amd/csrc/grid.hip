// grid.hip - probe grid, point ordering and k-nearest-probe search (ComGS Sec. 3.1.2,
// efficient querying through SOPs: FRNN search then KNN weights of Eq. 10-11).
//
// Positions are quantised to a 2^15 lattice in FP32; distances are exact integers. Probes
// are counting-sorted into a cube of 2^bits cells per axis addressed by the Morton index of
// the cell, so that cells close in space are close in memory. Points are counting-sorted by
// the same cell index into a processing order, so that consecutive wavefronts shade points
// that share probes. The search visits cells in growing Chebyshev shells and stops when the
// K-th best squared distance is below the squared distance to the nearest unvisited cell.
#include "sop_device.hpp"
#include "sop_internal.hpp"

namespace sopk {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr int kScanTile = kScanThreads * kScanItems;

size_t scan_tmp_elems(size_t n) { return (n + kScanTile - 1) / kScanTile + 1; }

__global__ __launch_bounds__(256) void k_fill_i32(int32_t* p, int32_t v, size_t n) {
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

// inclusive block scan of one value per thread; returns the exclusive prefix, *total = sum
__device__ __forceinline__ int32_t block_exclusive(int32_t v, int32_t* buf, int32_t* total) {
  const int t = threadIdx.x;
  buf[t] = v;
  __syncthreads();
  for (int off = 1; off < kScanThreads; off <<= 1) {
    int32_t x = t >= off ? buf[t - off] : 0;
    __syncthreads();
    buf[t] += x;
    __syncthreads();
  }
  const int32_t incl = buf[t];
  *total = buf[kScanThreads - 1];
  __syncthreads();
  return incl - v;
}

__global__ __launch_bounds__(kScanThreads) void k_tile_sums(const int32_t* in, size_t n,
                                                            int32_t* sums) {
  __shared__ int32_t buf[kScanThreads];
  const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
  int32_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i)
    if (base + i < n) s += in[base + i];
  int32_t total;
  block_exclusive(s, buf, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// single workgroup: exclusive scan of sums[0..nb) in place, sums[nb] = total
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(int32_t* sums, int32_t nb) {
  __shared__ int32_t buf[kScanThreads];
  int32_t carry = 0;
  for (int32_t base = 0; base < nb; base += kScanThreads) {
    const int32_t i = base + (int32_t)threadIdx.x;
    const int32_t v = i < nb ? sums[i] : 0;
    int32_t total;
    const int32_t ex = block_exclusive(v, buf, &total);
    if (i < nb) sums[i] = carry + ex;
    carry += total;
  }
  if (threadIdx.x == 0) sums[nb] = carry;
}

__global__ __launch_bounds__(kScanThreads) void k_tile_scan(const int32_t* in, int32_t* out,
                                                            size_t n, const int32_t* sums,
                                                            int32_t nb) {
  __shared__ int32_t buf[kScanThreads];
  const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)threadIdx.x * kScanItems;
  int32_t v[kScanItems];
  int32_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    v[i] = base + i < n ? in[base + i] : 0;
    s += v[i];
  }
  int32_t total;
  int32_t run = block_exclusive(s, buf, &total) + sums[blockIdx.x];
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (base + i < n) out[base + i] = run;
    run += v[i];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = sums[nb];
}

hipError_t launch_exclusive_scan(const int32_t* in, int32_t* out, size_t n, int32_t* tmp,
                                 hipStream_t s) {
  const int32_t nb = (int32_t)((n + kScanTile - 1) / kScanTile);
  if (nb == 0) {
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(256), 0, s, out, 0, (size_t)1);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_tile_sums, dim3(nb), dim3(kScanThreads), 0, s, in, n, tmp);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kScanThreads), 0, s, tmp, nb);
  hipLaunchKernelGGL(k_tile_scan, dim3(nb), dim3(kScanThreads), 0, s, in, out, n, tmp, nb);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// probe grid
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t cell_of(int qx, int qy, int qz, int shift) {
  return morton3((uint32_t)(qx >> shift), (uint32_t)(qy >> shift), (uint32_t)(qz >> shift));
}

__global__ __launch_bounds__(256) void k_probe_quant(const float* pos, int32_t P, float lo0,
                                                     float lo1, float lo2, float sc,
                                                     int32_t shift, int4* qtmp,
                                                     int32_t* counts, float* pos_copy) {
  const int32_t p = blockIdx.x * 256 + threadIdx.x;
  if (p >= P) return;
  const float x = pos[3 * p], y = pos[3 * p + 1], z = pos[3 * p + 2];
  const int qx = quantize1(x, lo0, sc), qy = quantize1(y, lo1, sc), qz = quantize1(z, lo2, sc);
  const uint32_t m = cell_of(qx, qy, qz, shift);
  qtmp[p] = make_int4(qx, qy, qz, (int)m);
  atomicAdd(&counts[m], 1);
  pos_copy[3 * p] = x;
  pos_copy[3 * p + 1] = y;
  pos_copy[3 * p + 2] = z;
}

__global__ __launch_bounds__(256) void k_probe_scatter(const int4* qtmp, int32_t P,
                                                       const int32_t* cell_start,
                                                       int32_t* cursor, int4* qsorted) {
  const int32_t p = blockIdx.x * 256 + threadIdx.x;
  if (p >= P) return;
  const int4 q = qtmp[p];
  const int32_t slot = cell_start[q.w] + atomicAdd(&cursor[q.w], 1);
  qsorted[slot] = make_int4(q.x, q.y, q.z, p);
}

hipError_t launch_probe_grid_build(const float* pos, int32_t P, const float lo[3], float sc,
                                   int32_t bits, int4* qtmp, int32_t* counts,
                                   int32_t* cell_start, int32_t* cursor, int4* qsorted,
                                   float* pos_copy, int32_t* scan_tmp, hipStream_t s) {
  const size_t C = (size_t)1 << (3 * bits);
  hipError_t e = launch_fill_i32(counts, 0, C, s);
  if (e != hipSuccess) return e;
  if ((e = launch_fill_i32(cursor, 0, C, s)) != hipSuccess) return e;
  if (P > 0) {
    hipLaunchKernelGGL(k_probe_quant, dim3((P + 255) / 256), dim3(256), 0, s, pos, P, lo[0],
                       lo[1], lo[2], sc, 15 - bits, qtmp, counts, pos_copy);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if ((e = launch_exclusive_scan(counts, cell_start, C, scan_tmp, s)) != hipSuccess) return e;
  if (P > 0) {
    hipLaunchKernelGGL(k_probe_scatter, dim3((P + 255) / 256), dim3(256), 0, s, qtmp, P,
                       cell_start, cursor, qsorted);
    e = hipGetLastError();
  }
  return e;
}

// ------------------------------------------------------------------------------------------
// point ordering: counting sort by Morton cell
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t point_cell(const ProbeGrid& g, const float* pts, int64_t i) {
  return cell_of(quantize1(pts[3 * i], g.lo[0], g.sc), quantize1(pts[3 * i + 1], g.lo[1], g.sc),
                 quantize1(pts[3 * i + 2], g.lo[2], g.sc), g.shift);
}

// Counts the points of every cell and keeps each point's rank in its cell, so that the
// scatter needs no atomics of its own. An atomic costs its request at memory, ~10 G/s, so
// there is one per run of lanes in the same cell (neighbouring pixels mostly are: a
// 1920x1080 frame takes 21 us and its scatter 8, against 562 and 822 us with one atomic per
// point in each) ...
__global__ __launch_bounds__(256) void k_point_rank(ProbeGrid g, const float* pts, int64_t N,
                                                    int32_t* counts, int32_t* rank) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const int32_t m = i < N ? (int32_t)point_cell(g, pts, i) : -1;
  const int32_t before = __shfl_up(m, 1);
  const bool head = lane == 0 || before != m;
  const uint64_t heads = __ballot(head);
  const uint64_t upto = heads & (~0ull >> (63 - lane));       // heads at or below the lane
  const int first = 63 - __builtin_clzll(upto);
  int32_t base = 0;
  if (head && m >= 0) {
    const uint64_t after = lane == 63 ? 0 : heads >> (lane + 1);
    const int len = after ? __builtin_ctzll(after) + 1 : 64 - lane;
    base = atomicAdd(&counts[m], len);
  }
  base = __shfl(base, first);
  if (i < N) rank[i] = base + lane - first;
}

// ... and, for grids of up to kTableCells cells, one per cell and chunk of kTablePoints
// points, counted in LDS first (points in no order: 500k over 900 cells 22 + 7 us, against 70
// + 96).
constexpr int kTableCells = 32768;
constexpr int kTablePer = 4;
constexpr int kTablePoints = 1024 * kTablePer;
__global__ __launch_bounds__(1024) void k_point_rank_table(ProbeGrid g, const float* pts,
                                                           int64_t N, int32_t* counts,
                                                           int32_t* rank) {
  extern __shared__ int32_t cnt[];                            // [cells], a multiple of 4
  const int cells = 1 << (3 * g.bits), tid = threadIdx.x;
  for (int c = 4 * tid; c < cells; c += 4096)
    *reinterpret_cast<int4*>(cnt + c) = make_int4(0, 0, 0, 0);
  __syncthreads();
  int32_t m[kTablePer], r[kTablePer];
#pragma unroll
  for (int u = 0; u < kTablePer; ++u) {
    const int64_t i = (int64_t)blockIdx.x * kTablePoints + u * 1024 + tid;
    m[u] = i < N ? (int32_t)point_cell(g, pts, i) : -1;
    r[u] = m[u] >= 0 ? atomicAdd(&cnt[m[u]], 1) : -1;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kTablePer; ++u)
    if (r[u] == 0) cnt[m[u]] = atomicAdd(&counts[m[u]], cnt[m[u]]);   // the chunk's first rank
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kTablePer; ++u) {
    const int64_t i = (int64_t)blockIdx.x * kTablePoints + u * 1024 + tid;
    if (i < N) rank[i] = cnt[m[u]] + r[u];
  }
}

__global__ __launch_bounds__(256) void k_point_scatter(ProbeGrid g, const float* pts, int64_t N,
                                                       const int32_t* start,
                                                       const int32_t* rank, int32_t* out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= N) return;
  out[start[point_cell(g, pts, i)] + rank[i]] = (int32_t)i;
}

// Orders the points of each grid cell by the Morton code of their lattice position inside
// the cell (10 bits per axis), ties by point index: consecutive points of the order then
// lie close together at the scale of a few points, not only of a cell, so a batch of them
// shares more neighbouring probes (the adjoint adds each batch's texture gradient once per
// distinct probe). A cell of more than kRefineMax points keeps the counting sort's order.
// Also makes the order deterministic. Most cells of a grid are empty, so a workgroup looks at
// up to 64 of them, spread over the grid. It places each point of a cell by counting the
// smaller keys: of the whole cell up to 256 points, and above that of its bin, the top 12
// bits of the code (a bitonic sort of every cell is bound by its LDS passes: 99 us on 500k
// points in 900 cells, 35 us this way); a cell with a bin of more than kBinMax
// points, whose counts would grow with the square of it, is still sorted.
constexpr int kRefineMax = 4096;
constexpr int kRefineBlocks = 4096;
constexpr int kBins = 4096;
constexpr int kBinMax = 128;
constexpr int kRefinePer = kRefineMax / 256;

// the number of keys below k among key[a, b)
template <int UNROLL>
__device__ __forceinline__ int count_below(const uint64_t* key, int a, int b, uint64_t k) {
  int c = 0;
#pragma unroll UNROLL
  for (int j = a; j < b; ++j) c += key[j] < k ? 1 : 0;
  return c;
}

__device__ __forceinline__ void bitonic_sort(uint64_t* key, int n) {
  int m = 1;
  while (m < n) m <<= 1;
  for (int i = n + (int)threadIdx.x; i < m; i += 256) key[i] = ~0ull;
  __syncthreads();
  for (int size = 2; size <= m; size <<= 1)
    for (int step = size >> 1; step > 0; step >>= 1) {
      for (int t = threadIdx.x; t < m / 2; t += 256) {
        const int i = 2 * t - (t & (step - 1)), j = i + step;
        const uint64_t x = key[i], y = key[j];
        if ((x > y) == ((i & size) == 0)) {
          key[i] = y;
          key[j] = x;
        }
      }
      __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_point_refine(ProbeGrid g, const float* pts,
                                                      const int32_t* start, int32_t cells,
                                                      const int32_t* in, int32_t* order) {
  __shared__ uint64_t key[kRefineMax];
  __shared__ int32_t bin[kBins + 1];                      // count, then first place of each bin
  __shared__ int32_t sums[kScanThreads];
  const int tid = threadIdx.x;
  const int32_t stride = (int32_t)gridDim.x;
  const int fine = g.shift < 10 ? g.shift : 10;           // bits per axis inside the cell
  const int sh = g.shift - fine, bsh = 32 + (fine > 4 ? 3 * fine - 12 : 0);
  const uint32_t mask = (1u << g.shift) - 1u;
  auto key_of = [&](int32_t p) {
    const uint32_t qx = (uint32_t)quantize1(pts[3 * (int64_t)p], g.lo[0], g.sc) & mask;
    const uint32_t qy = (uint32_t)quantize1(pts[3 * (int64_t)p + 1], g.lo[1], g.sc) & mask;
    const uint32_t qz = (uint32_t)quantize1(pts[3 * (int64_t)p + 2], g.lo[2], g.sc) & mask;
    return ((uint64_t)morton3(qx >> sh, qy >> sh, qz >> sh) << 32) | (uint32_t)p;
  };
  for (int32_t c0 = blockIdx.x; c0 < cells; c0 += 64 * stride) {
    const int64_t mine = (int64_t)c0 + (int64_t)(tid & 63) * stride;
    int32_t b0 = 0, bn = 0;
    if (mine < cells) {
      b0 = start[mine];
      bn = start[mine + 1] - b0;
    }
    for (uint64_t some = __ballot(bn > 0); some != 0; some &= some - 1) {   // uniform
      const int l = __builtin_ctzll(some);
      const int32_t s0 = __builtin_amdgcn_readlane(b0, l), n = __builtin_amdgcn_readlane(bn, l);
      if (n == 1 || n > kRefineMax) {
        for (int i = tid; i < n; i += 256) order[s0 + i] = in[s0 + i];
        continue;
      }
      __syncthreads();                                     // the cell before is done
      if (n <= 256) {
        uint64_t k = 0;
        if (tid < n) key[tid] = k = key_of(in[s0 + tid]);
        __syncthreads();
        if (tid < n) order[s0 + count_below<8>(key, 0, n, k)] = (int32_t)(uint32_t)k;
        continue;
      }
      for (int i = tid; i < kBins / 4; i += 256)
        reinterpret_cast<int4*>(bin)[i] = make_int4(0, 0, 0, 0);
      __syncthreads();
      uint64_t k[kRefinePer];
      int32_t r[kRefinePer];
#pragma unroll
      for (int u = 0; u < kRefinePer; ++u) {
        const int i = tid + 256 * u;
        if (i < n) {
          k[u] = key_of(in[s0 + i]);
          r[u] = atomicAdd(&bin[(int)(k[u] >> bsh)], 1);
        }
      }
      __syncthreads();
      int32_t cnt[kBins / 256], own = 0;
      bool large = false;
#pragma unroll
      for (int u = 0; u < kBins / 256; ++u) {
        cnt[u] = bin[tid * (kBins / 256) + u];
        own += cnt[u];
        large = large || cnt[u] > kBinMax;
      }
      int32_t total;
      int32_t at = block_exclusive(own, sums, &total);
#pragma unroll
      for (int u = 0; u < kBins / 256; ++u) {
        bin[tid * (kBins / 256) + u] = at;
        at += cnt[u];
      }
      if (tid == 255) bin[kBins] = n;
      const bool sort = __syncthreads_or(large) != 0;
#pragma unroll
      for (int u = 0; u < kRefinePer; ++u)
        if (tid + 256 * u < n) key[bin[(int)(k[u] >> bsh)] + r[u]] = k[u];
      __syncthreads();
      if (sort) {
        bitonic_sort(key, n);
        for (int i = tid; i < n; i += 256) order[s0 + i] = (int32_t)(uint32_t)key[i];
        continue;
      }
#pragma unroll
      for (int u = 0; u < kRefinePer; ++u)
        if (tid + 256 * u < n) {
          const int q = (int)(k[u] >> bsh), first = bin[q];
          order[s0 + first + count_below<1>(key, first, bin[q + 1], k[u])] =
              (int32_t)(uint32_t)k[u];
        }
    }
  }
}

// The same order for a call of up to kOrderSmall points in one kernel: every workgroup forms
// all the keys (cell, code inside it, index) in LDS and places kOrderPer of the points by
// counting the smaller ones, kOrderLanes lanes to a point. The seven launches above cost
// 16-22 us whatever they sort, and the gaps between them as much again; this one takes
// 3.4 us for 300 points and 12 us for 4096.
constexpr int kOrderSmall = 4096;
constexpr int kOrderLanes = 16;
constexpr int kOrderPer = 256 / kOrderLanes;
__global__ __launch_bounds__(256) void k_point_order_small(ProbeGrid g, const float* pts, int32_t N,
                                                           int32_t* order) {
  __shared__ uint64_t key[kOrderSmall];
  const int fine = g.shift < 10 ? g.shift : 10, sh = g.shift - fine;
  const uint32_t mask = (1u << g.shift) - 1u;
#pragma unroll 8
  for (int i = threadIdx.x; i < N; i += 256) {
    const uint32_t qx = (uint32_t)quantize1(pts[3 * i], g.lo[0], g.sc);
    const uint32_t qy = (uint32_t)quantize1(pts[3 * i + 1], g.lo[1], g.sc);
    const uint32_t qz = (uint32_t)quantize1(pts[3 * i + 2], g.lo[2], g.sc);
    const uint32_t cell = cell_of((int)qx, (int)qy, (int)qz, g.shift);          // 21 bits
    const uint32_t code = morton3((qx & mask) >> sh, (qy & mask) >> sh, (qz & mask) >> sh);
    key[i] = ((uint64_t)cell << 42) | ((uint64_t)code << 12) | (uint32_t)i;     // 30 + 12 bits
  }
  __syncthreads();
  const int slice = threadIdx.x % kOrderLanes;
  const int i = (int)blockIdx.x * kOrderPer + (int)threadIdx.x / kOrderLanes;
  const uint64_t k = i < N ? key[i] : 0;
  int c = 0;
#pragma unroll 8
  for (int j = slice; j < N; j += kOrderLanes) c += key[j] < k ? 1 : 0;
#pragma unroll
  for (int o = 1; o < kOrderLanes; o <<= 1) c += __shfl_xor(c, o);
  if (i < N && slice == 0) order[c] = i;
}
static_assert(kOrderSmall <= 1 << 12, "index bits of the key");

hipError_t launch_point_order(const ProbeGrid& g, const float* pts, int64_t N,
                              int32_t* by_cell, int32_t* counts, int32_t* offsets,
                              int32_t* scan_tmp, int32_t* order, hipStream_t s) {
  if (N == 0) return hipSuccess;
  if (N <= kOrderSmall) {
    hipLaunchKernelGGL(k_point_order_small, dim3((unsigned)((N + kOrderPer - 1) / kOrderPer)),
                       dim3(256), 0, s, g, pts, (int32_t)N, order);
    return hipGetLastError();
  }
  const size_t C = (size_t)1 << (3 * g.bits);
  hipError_t e = launch_fill_i32(counts, 0, C, s);
  if (e != hipSuccess) return e;
  const unsigned blocks = (unsigned)((N + 255) / 256);
  int32_t* rank = order;                       // until the order itself is written
  if (C <= (size_t)kTableCells) {
    const size_t lds = C * sizeof(int32_t);
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_point_rank_table),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(k_point_rank_table, dim3((unsigned)((N + kTablePoints - 1) / kTablePoints)),
                       dim3(1024), lds, s, g, pts, N, counts, rank);
  } else {
    hipLaunchKernelGGL(k_point_rank, dim3(blocks), dim3(256), 0, s, g, pts, N, counts, rank);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = launch_exclusive_scan(counts, offsets, C, scan_tmp, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_point_scatter, dim3(blocks), dim3(256), 0, s, g, pts, N, offsets, rank,
                     by_cell);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(k_point_refine, dim3((unsigned)std::min<size_t>(C, kRefineBlocks)), dim3(256),
                     0, s, g, pts, offsets, (int32_t)C, by_cell, order);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------
// k nearest probes
// ------------------------------------------------------------------------------------------
// A search grows a box of grid cells around its points (their own cells and the neighbours of
// those first) and stops when the K-th best squared
// distance is below that to the nearest cell outside the box. One load per lane fetches the
// ranges of 64 cells of the box, cells that are further off than the K-th best are dropped,
// and the probes of the rest are numbered across the lanes and fetched 64 at a time: two
// dependent loads for every 64 cells and 64 probes, where a thread that walks the cells of
// its own point pays two for every cell (it took 85-117 us, whatever the point count).
template <int CTRL, int BANKS = 0xF>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t old, uint64_t v) {
  const int lo = __builtin_amdgcn_update_dpp((int)(uint32_t)old, (int)(uint32_t)v, CTRL, 0xF,
                                             BANKS, false);
  const int hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(old >> 32), (int)(uint32_t)(v >> 32),
                                             CTRL, 0xF, BANKS, false);
  return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

// the key of lane l ^ X of the same row of 16 (X = 1, 2, 4, 8), or of its mirror image in a
// group of X + 1 lanes (X = 3, 7, 15)
template <int X>
__device__ __forceinline__ uint64_t row_partner(uint64_t v) {
  if constexpr (X == 1) return dpp_u64<0xB1>(v, v);
  else if constexpr (X == 2) return dpp_u64<0x4E>(v, v);
  else if constexpr (X == 3) return dpp_u64<0x1B>(v, v);
  else if constexpr (X == 7) return dpp_u64<0x141>(v, v);
  else if constexpr (X == 15) return dpp_u64<0x140>(v, v);
  else if constexpr (X == 8) return dpp_u64<0x128>(v, v);
  else return dpp_u64<0x114, 0xA>(dpp_u64<0x104, 0x5>(v, v), v);   // 4: shift by 4 either way
}

// one step of a sorting network over the lanes of a row: the lane whose bit BIT is clear
// keeps the smaller key
template <int X, int BIT>
__device__ __forceinline__ uint64_t row_step(uint64_t v, int lane) {
  const uint64_t o = row_partner<X>(v);
  return ((o < v) != ((lane & BIT) != 0)) ? o : v;
}

__device__ __forceinline__ uint64_t row_sort(uint64_t v, int lane) {
  v = row_step<1, 1>(v, lane);
  v = row_step<3, 2>(v, lane);
  v = row_step<1, 1>(v, lane);
  v = row_step<7, 4>(v, lane);
  v = row_step<2, 2>(v, lane);
  v = row_step<1, 1>(v, lane);
  v = row_step<15, 8>(v, lane);
  v = row_step<4, 4>(v, lane);
  v = row_step<2, 2>(v, lane);
  return row_step<1, 1>(v, lane);
}

// the 16 smallest keys of two sorted rows, sorted
__device__ __forceinline__ uint64_t row_merge(uint64_t a, uint64_t b, int lane) {
  const uint64_t o = row_partner<15>(b);
  uint64_t v = o < a ? o : a;
  v = row_step<8, 8>(v, lane);
  v = row_step<4, 4>(v, lane);
  v = row_step<2, 2>(v, lane);
  return row_step<1, 1>(v, lane);
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int o) {
  const uint32_t lo = __shfl_xor((uint32_t)v, o), hi = __shfl_xor((uint32_t)(v >> 32), o);
  return ((uint64_t)hi << 32) | lo;
}

// the 16 smallest of the wavefront's 64 keys and of the list `best` (sorted, one copy in
// every row of 16 lanes): the new list
__device__ __forceinline__ uint64_t list_merge(uint64_t best, uint64_t key, int lane) {
  key = row_sort(key, lane);
  key = row_merge(key, shfl_xor_u64(key, 16), lane);
  key = row_merge(key, shfl_xor_u64(key, 32), lane);
  return row_merge(best, key, lane);
}

// inclusive sum over the lanes (all 64 active)
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row 15 -> next row
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // lane 31 -> rows 2, 3
  return v;
}

// largest value over the lanes (all 64 active)
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  auto step = [](uint32_t x, int moved) { return max(x, (uint32_t)moved); };
  v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false));
  v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false));
  v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false));
  v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x140, 0xF, 0xF, false));
  v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xA, 0xF, false));
  v = step(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xC, 0xF, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// A box of cells [lo, hi] of the search and the box inside it that was visited before
// (empty at first: lo > hi); ql, qh bound the lattice positions of the points searched for.
// All wave-uniform.
struct CellBox {
  int lo[3], hi[3], plo[3], phi[3];
  int ql[3], qh[3];
};

// grows the box to r cells around the cells [c0, c1], clipped to the grid of n cells a side
__device__ __forceinline__ void box_grow(CellBox& b, const int c0[3], const int c1[3], int r,
                                         int n) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    b.plo[a] = b.lo[a];
    b.phi[a] = b.hi[a];
    b.lo[a] = max(c0[a] - r, 0);
    b.hi[a] = min(c1[a] + r, n - 1);
  }
}

// Calls use(m, pq) with up to 64 probes at a time, pq in lanes 0 .. m - 1, for every probe in
// a new cell of the box whose distance to the points is at most limit() (squared, lattice
// units); limit() is read again for every 64 cells. Every lane of the wavefront calls it.
template <typename Limit, typename Use>
__device__ __forceinline__ void visit_new_cells(const ProbeGrid& g, const CellBox& b, int lane,
                                                Limit limit, Use use) {
  const int nx = b.hi[0] - b.lo[0] + 1, ny = b.hi[1] - b.lo[1] + 1;
  const int ncell = nx * ny * (b.hi[2] - b.lo[2] + 1);
  for (int base = 0; base < ncell; base += 64) {
    const uint32_t most = limit();             // every lane takes part in it
    const int i = base + lane;
    const int row = i / nx;
    const int c[3] = {b.lo[0] + i - row * nx, b.lo[1] + row % ny, b.lo[2] + row / ny};
    bool inner = true;
    uint32_t d2 = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      inner = inner && c[a] >= b.plo[a] && c[a] <= b.phi[a];
      const int c0 = c[a] << g.shift, c1 = c0 + (1 << g.shift) - 1;
      const int d = max(max(c0 - b.qh[a], b.ql[a] - c1), 0);
      d2 += (uint32_t)(d * d);
    }
    int e0 = 0, cnt = 0;
    if (i < ncell && !inner && d2 <= most) {
      const uint32_t m = morton3((uint32_t)c[0], (uint32_t)c[1], (uint32_t)c[2]);
      e0 = g.cell_start[m];
      cnt = g.cell_start[m + 1] - e0;
    }
    const int incl = wave_scan(cnt);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const int src = e0 - (incl - cnt);        // entry of candidate j of this lane's cell: src + j
    for (int j0 = 0; j0 < total; j0 += 64) {
      // the lane whose cell holds candidate j: the number of lanes with incl <= j
      const int j = j0 + lane;
      int own = 0;
#pragma unroll
      for (int s = 32; s > 0; s >>= 1)
        if (__shfl(incl, own + s - 1) <= j) own += s;
      const int e = __shfl(src, own & 63) + j;
      const int m = min(total - j0, 64);
      int4 pq = make_int4(0, 0, 0, 0);
      if (lane < m) pq = g.qsorted[e];
      use(m, pq);
    }
  }
}

// The box grows by a cell at first, and by half its radius from 6 cells on (probes in a volume
// are found within 5): every growth scans the cells it has visited before as well, so that
// single steps up to radius r look at r / 4 times the final box. That is what bounds points far
// from all probes: 200k points of a sphere, 16,384 probes in one place beside it, 254 -> 37 ms
// (a thread per point that visits each cell once: 123); 300 points 39.7 -> 3.6 ms.
__device__ __forceinline__ int next_radius(int r) { return r < 6 ? r + 1 : r + r / 2; }

// squared distance from lattice position q to the nearest cell outside the box (~0: none)
__device__ __forceinline__ uint64_t outside_d2(const CellBox& b, const int q[3], int shift,
                                               int n) {
  uint64_t lb = ~0ull;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (b.lo[a] > 0) lb = min(lb, (uint64_t)(q[a] - (b.lo[a] << shift) + 1));
    if (b.hi[a] < n - 1) lb = min(lb, (uint64_t)(((b.hi[a] + 1) << shift) - q[a]));
  }
  return lb == ~0ull ? lb : lb * lb;
}

// weight of a neighbour before the division by the sum (Eq. 10-11)
__device__ __forceinline__ float knn_weight(const ProbeGrid& g, int p, v3 x, v3 n) {
  const v3 d = sub(mk3(g.pos[3 * p], g.pos[3 * p + 1], g.pos[3 * p + 2]), x);
  const float len = sqrtf(dot(d, d));
  const float inv = 1.0f / len;
  const float wb = 0.5f * (1.0f + dot(d, n) * inv) + 0.01f;
  return inv * wb;
}

// One wavefront per point: the lanes test 64 probes at once and merge them into the point's
// list by a sorting network. Bound by the latency of its few dependent loads until the points
// fill the chip: 300 points among 64 probes take 10 us (a thread per point: 117 us), 4096
// points 13 us (86).
template <int K>
__global__ __launch_bounds__(256) void k_knn_wave(ProbeGrid g, const float* pts,
                                                  const float* normals, int64_t N,
                                                  const int32_t* order, uint32_t lim,
                                                  int32_t* out_idx, float* out_w) {
  const int64_t t = (int64_t)blockIdx.x * 4 + wave_id_uniform();
  if (t >= N) return;
  const int lane = threadIdx.x & 63;
  int64_t i = t;
  if (order) {
    const int32_t o = __builtin_amdgcn_readfirstlane(order[t]);
    if ((uint64_t)o >= (uint64_t)N) return;
    i = o;
  }
  const v3 x = mk3(pts[3 * i], pts[3 * i + 1], pts[3 * i + 2]);
  const int G = 1 << g.bits;
  int q[3] = {quantize1(x.x, g.lo[0], g.sc), quantize1(x.y, g.lo[1], g.sc),
              quantize1(x.z, g.lo[2], g.sc)};
  CellBox b;
  int c[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    q[a] = __builtin_amdgcn_readfirstlane(q[a]);
    c[a] = q[a] >> g.shift;
    b.ql[a] = b.qh[a] = q[a];
    b.lo[a] = 0;
    b.hi[a] = -1;
  }
  uint64_t best = ~0ull;             // lane s of every row of 16: the s-th best key
  uint32_t kth = ~0u;                // d^2 of the K-th best
  for (int r = 1;; r = next_radius(r)) {
    box_grow(b, c, c, r, G);
    visit_new_cells(
        g, b, lane, [&]() { return min(kth, lim); },
        [&](int m, int4 pq) {
          const int dx = pq.x - q[0], dy = pq.y - q[1], dz = pq.z - q[2];
          const uint32_t d2 = (uint32_t)(dx * dx) + (uint32_t)(dy * dy) + (uint32_t)(dz * dz);
          const bool in = lane < m && d2 <= min(kth, lim);
          if (__ballot(in) == 0) return;
          best = list_merge(best, in ? ((uint64_t)d2 << 32) | (uint32_t)pq.w : ~0ull, lane);
          kth = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(best >> 32), K - 1);
        });
    const uint64_t lb2 = outside_d2(b, q, g.shift, G);
    if (lb2 == ~0ull || lb2 > (uint64_t)lim) break;
    // ~0 in the low half marks an empty entry (a probe index is below 2^31)
    const uint32_t kid = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)best, K - 1);
    if (kid != ~0u && (uint64_t)kth < lb2) break;
  }
  const bool found = (uint32_t)best != ~0u;
  // exact hit: that probe alone
  const bool hit = __builtin_amdgcn_readfirstlane((int)(uint32_t)best) != -1 &&
                   __builtin_amdgcn_readfirstlane((int)(uint32_t)(best >> 32)) == 0;
  const v3 n = mk3(normals[3 * i], normals[3 * i + 1], normals[3 * i + 2]);
  const int p = (int)(uint32_t)best;
  float wv = 0.0f;
  if (lane < K && found) wv = knn_weight(g, p, x, n);
  float sum = 0.0f;                  // added in list order
#pragma unroll
  for (int s = 0; s < K; ++s)
    sum += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wv), s));
  const float isum = 1.0f / sum;
  if (lane < K) {
    const bool keep = found && (!hit || lane == 0);
    out_idx[i * K + lane] = keep ? p : -1;
    out_w[i * K + lane] = keep ? (hit ? 1.0f : wv * isum) : 0.0f;
  }
}

template <int K>
__device__ __forceinline__ void insert_key(uint64_t (&best)[K], uint64_t key) {
  if (key < best[K - 1]) {
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const uint64_t lo = key < best[s] ? key : best[s];
      key = key < best[s] ? best[s] : key;
      best[s] = lo;
    }
  }
}

// One lane per point, in processing order: the points of a wavefront lie in a few
// neighbouring cells, so the wavefront searches for all its points within one cell of the
// first unfinished one together, and every lane tests every probe of their box (the probe's
// lattice position comes from a lane's register as a scalar). The points left over, across
// a jump of the order, are taken in turn. Bound by the vector ALUs (the insertions): 200k
// points among 4096 probes, K = 8, 52 us (a thread per point walking its own cells: 99 us),
// 2.07M points among 16,384 probes 133 us (357).
template <int K>
__global__ __launch_bounds__(256) void k_knn_dense(ProbeGrid g, const float* pts,
                                                   const float* normals, int64_t N,
                                                   const int32_t* order, uint32_t lim,
                                                   int32_t* out_idx, float* out_w) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  bool live = t < N;
  int64_t i = live ? t : 0;
  if (live && order) {
    const int32_t o = order[t];
    live = (uint64_t)o < (uint64_t)N;
    i = live ? o : 0;
  }
  const v3 x = mk3(pts[3 * i], pts[3 * i + 1], pts[3 * i + 2]);
  const int q[3] = {quantize1(x.x, g.lo[0], g.sc), quantize1(x.y, g.lo[1], g.sc),
                    quantize1(x.z, g.lo[2], g.sc)};
  const int G = 1 << g.bits;
  const int c[3] = {q[0] >> g.shift, q[1] >> g.shift, q[2] >> g.shift};
  uint64_t best[K];
#pragma unroll
  for (int s = 0; s < K; ++s) best[s] = ~0ull;

  uint64_t todo = __ballot(live);
  while (todo != 0) {                              // uniform
    const int first = __builtin_ctzll(todo);
    bool act = ((todo >> lane) & 1) != 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) act = act && abs(c[a] - __builtin_amdgcn_readlane(c[a], first)) <= 1;
    todo &= ~__ballot(act);
    CellBox b;
    int c0[3], c1[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      b.qh[a] = (int)wave_max_u32(act ? (uint32_t)q[a] : 0u);
      b.ql[a] = 32767 - (int)wave_max_u32(act ? (uint32_t)(32767 - q[a]) : 0u);
      c0[a] = b.ql[a] >> g.shift;
      c1[a] = b.qh[a] >> g.shift;
      b.lo[a] = 0;
      b.hi[a] = -1;
    }
    for (int r = 1;; r = next_radius(r)) {
      box_grow(b, c0, c1, r, G);
      visit_new_cells(
          g, b, lane,
          [&]() { return min(wave_max_u32(act ? (uint32_t)(best[K - 1] >> 32) : 0u), lim); },
          [&](int m, int4 pq) {
            for (int j = 0; j < m; ++j) {
              const int dx = __builtin_amdgcn_readlane(pq.x, j) - q[0];
              const int dy = __builtin_amdgcn_readlane(pq.y, j) - q[1];
              const int dz = __builtin_amdgcn_readlane(pq.z, j) - q[2];
              const uint32_t id = (uint32_t)__builtin_amdgcn_readlane(pq.w, j);
              const uint32_t d2 =
                  (uint32_t)(dx * dx) + (uint32_t)(dy * dy) + (uint32_t)(dz * dz);
              if (act && d2 <= lim) insert_key<K>(best, ((uint64_t)d2 << 32) | id);
            }
          });
      const uint64_t lb2 = outside_d2(b, q, g.shift, G);
      const bool more = act && lb2 != ~0ull && lb2 <= (uint64_t)lim &&
                        !(best[K - 1] != ~0ull && (best[K - 1] >> 32) < lb2);
      if (__ballot(more) == 0) break;
    }
  }
  if (!live) return;

  int32_t* oi = out_idx + i * K;
  float* ow = out_w + i * K;
  if (best[0] != ~0ull && (best[0] >> 32) == 0) {    // exact hit: that probe alone
    oi[0] = (int32_t)(best[0] & 0xFFFFFFFFu);
    ow[0] = 1.0f;
#pragma unroll
    for (int s = 1; s < K; ++s) {
      oi[s] = -1;
      ow[s] = 0.0f;
    }
    return;
  }
  const v3 n = mk3(normals[3 * i], normals[3 * i + 1], normals[3 * i + 2]);
  float wv[K];
  float sum = 0.0f;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    wv[s] = best[s] != ~0ull ? knn_weight(g, (int)(best[s] & 0xFFFFFFFFu), x, n) : 0.0f;
    sum += wv[s];
  }
  const float isum = 1.0f / sum;
#pragma unroll
  for (int s = 0; s < K; ++s) {
    const bool valid = best[s] != ~0ull;
    oi[s] = valid ? (int32_t)(best[s] & 0xFFFFFFFFu) : -1;
    ow[s] = valid ? wv[s] * isum : 0.0f;
  }
}

// The lines cross where a wavefront's 64 consecutive points begin to share cells. Whole
// sop_knn calls at K = 8, wavefront / lane per point: 64 probes (8 cells a side) 8192 points
// 45 / 53 us, 16,384 points 57 / 52; 512 probes (16) 16,384 points 55 / 67, 32,768 points
// 76 / 65; 4096 probes (32) 32,768 points 78 / 99, 65,536 points 113 / 99; 16,384 probes (64)
// 65,536 points 129 / 140, 131,072 points 213 / 159.
static bool knn_by_wave(const ProbeGrid& g, int64_t N) { return N <= (int64_t)1536 << g.bits; }

template <int K>
static hipError_t knn_k(const ProbeGrid& g, const float* pts, const float* normals, int64_t N,
                        const int32_t* order, uint32_t lim, int32_t* idx, float* w,
                        hipStream_t s) {
  if (knn_by_wave(g, N))
    hipLaunchKernelGGL(k_knn_wave<K>, dim3((unsigned)((N + 3) / 4)), dim3(256), 0, s, g, pts,
                       normals, N, order, lim, idx, w);
  else
    hipLaunchKernelGGL(k_knn_dense<K>, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, g,
                       pts, normals, N, order, lim, idx, w);
  return hipGetLastError();
}

hipError_t launch_knn(const ProbeGrid& g, const float* pts, const float* normals, int64_t N,
                      const int32_t* order, int32_t k, uint32_t lim, int32_t* idx, float* w,
                      hipStream_t s) {
  if (N == 0) return hipSuccess;
  switch (k) {
#define SOP_KNN_CASE(KK) \
  case KK:               \
    return knn_k<KK>(g, pts, normals, N, order, lim, idx, w, s);
    SOP_KNN_CASE(1) SOP_KNN_CASE(2) SOP_KNN_CASE(3) SOP_KNN_CASE(4) SOP_KNN_CASE(5)
    SOP_KNN_CASE(6) SOP_KNN_CASE(7) SOP_KNN_CASE(8) SOP_KNN_CASE(9) SOP_KNN_CASE(10)
    SOP_KNN_CASE(11) SOP_KNN_CASE(12) SOP_KNN_CASE(13) SOP_KNN_CASE(14) SOP_KNN_CASE(15)
    SOP_KNN_CASE(16)
#undef SOP_KNN_CASE
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace sopk
