// First kernel of a batched call: its first workgroups write the scan of the
// work counts that the tile kernel walks (k_batched, k_batched_oop), and the
// others permute every array short enough for LDS, which needs no scan.
#include <limits.h>

#include "bitrev_launch.hpp"
#include "bitrev_rows.hpp"

namespace bitrev {
namespace {

// Threads of a workgroup with 2^lb bytes of LDS: four 16-byte vectors each, 4
// KiB a wavefront.
constexpr int front_threads(int lb) { return 1 << (lb - 6); }
// Arrays per workgroup of the whole-array part, at most: short batches (32 KiB
// of LDS) 8 (20000 float32 arrays of 2^4-2^12: 4 per workgroup 34.9 us, 8 30.8,
// 16 33), longer arrays 2 (4 lost 1-2%).  Batches of fewer arrays than fill
// kMinFrontBlocks workgroups so take fewer each (50 float32 arrays of 2^0-2^14
// out of place by 8: 8.5 us, one by one 7.2).
constexpr int front_arrays(int lb) { return lb == 15 ? 8 : 2; }
constexpr int kMinFrontBlocks = 512;
// Arrays per scan workgroup.
constexpr int kArraysPerScan = 1024;
constexpr int kMaxScanBlocks = 32;
constexpr int kScanLoads = 8;  // arrays a scan thread reads at once

struct BatchMeta {
  const int64_t* offsets;
  const int32_t* log2n;
  int64_t num;
  int64_t data_elems;
  int b;      // tile width
  int whole;  // arrays of at most 2^whole elements move whole
  int oop;
  int per;    // arrays per workgroup of the whole-array part
};

// Whether array a's metadata hold together: 2^log2n elements between its
// offsets, inside the data, and a middle the tile kernels can index.
__device__ __forceinline__ bool array_ok(const BatchMeta& m, int k, int64_t o0, int64_t o1) {
  return k >= 0 && k <= 40 && o0 >= 0 && o1 >= o0 && (o1 - o0) == (1ll << k) &&
         o1 <= m.data_elems && (k <= m.whole || k - 2 * m.b <= 32);
}

// Tile work items of array a: one per tile pair (in place) or per tile (out
// of place), none where it moves whole.  Counts a rejected array.
__device__ __forceinline__ int64_t array_work(const BatchMeta& m, int64_t a, int k, int64_t o0,
                                              int64_t o1, int64_t* bad, int64_t* first) {
  const bool ok = array_ok(m, k, o0, o1);
  *bad += ok ? 0 : 1;
  *first = !ok && a < *first ? a : *first;
  if (!ok || k <= m.whole) return 0;
  return m.oop ? (int64_t)1 << (k - 2 * m.b) : (int64_t)pair_count(k - 2 * m.b);
}

__device__ __forceinline__ int64_t wave_sum(int64_t v) {
  for (int d = 32; d; d >>= 1) v += __shfl_xor(v, d);
  return v;
}

// Workgroup j of `blocks` writes the exclusive prefix sums of its own run of
// arrays: it adds up the work of every array before the run itself (a plain
// coalesced sum), so that the workgroups need nothing from each other.  The
// last one has then seen every array and writes the header.  ws[0] = rejected
// arrays, ws[1] = first rejected (or -1), ws[2 + a] = first work item of array
// a, ws[2 + num] = all work.
//
// Bound by latency: 1024 threads of one workgroup, each summing a contiguous
// run twice with one load in flight, took 56.8 us for 20000 arrays.
template <int NT>
__device__ void batched_scan(const BatchMeta& m, int64_t* ws, int block, int blocks) {
  constexpr int kWaves = NT / 64;
  __shared__ int64_t part[kWaves][3];
  const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t per = (m.num + blocks - 1) / blocks;
  const int64_t a0 = per * block < m.num ? per * block : m.num;
  const int64_t a1 = a0 + per < m.num ? a0 + per : m.num;
  int64_t sum = 0, bad = 0, first = LLONG_MAX;
  for (int64_t base = 0; base < a0; base += NT * kScanLoads) {
    int k[kScanLoads];
    int64_t o0[kScanLoads], o1[kScanLoads];
#pragma unroll
    for (int i = 0; i < kScanLoads; ++i) {  // all loads first: one latency
      const int64_t a = base + i * NT + t, c = a < a0 ? a : a0 - 1;
      k[i] = m.log2n[c];
      o0[i] = m.offsets[c];
      o1[i] = m.offsets[c + 1];
    }
#pragma unroll
    for (int i = 0; i < kScanLoads; ++i) {
      const int64_t a = base + i * NT + t;
      if (a < a0) sum += array_work(m, a, k[i], o0[i], o1[i], &bad, &first);
    }
  }
  sum = wave_sum(sum);
  if (lane == 0) part[wave][0] = sum;
  __syncthreads();
  int64_t run = 0;
  for (int w = 0; w < kWaves; ++w) run += part[w][0];
  for (int64_t base = a0; base < a1; base += NT) {
    const int64_t a = base + t;
    const int64_t work =
        a < a1 ? array_work(m, a, m.log2n[a], m.offsets[a], m.offsets[a + 1], &bad, &first) : 0;
    int64_t incl = work;
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t v = __shfl_up(incl, d);
      if (lane >= d) incl += v;
    }
    __syncthreads();  // the previous sums have been read
    if (lane == 63) part[wave][0] = incl;
    __syncthreads();
    int64_t before = run;
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) before += part[w][0];
      run += part[w][0];
    }
    if (a < a1) ws[2 + a] = before + incl - work;
  }
  if (block != blocks - 1) return;
  bad = wave_sum(bad);
  for (int d = 32; d; d >>= 1) {
    const int64_t v = __shfl_xor(first, d);
    first = v < first ? v : first;
  }
  __syncthreads();
  if (lane == 0) {
    part[wave][1] = bad;
    part[wave][2] = first;
  }
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < kWaves; ++w) {
      bad += part[w][1];
      first = part[w][2] < first ? part[w][2] : first;
    }
    ws[0] = bad;
    ws[1] = first == LLONG_MAX ? -1 : first;
    ws[2 + m.num] = run;
  }
}

// Orders a wavefront's LDS writes before its lanes' reads (the hardware runs
// one wavefront's LDS accesses in order; this holds the compiler to it).
struct WaveSync {
  __device__ __forceinline__ void operator()() const {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
};
struct BlockSync {
  __device__ __forceinline__ void operator()() const { __syncthreads(); }
};

// Lane i's v (i uniform).
__device__ __forceinline__ int64_t lane_value(int64_t v, int i) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)v, i);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), i);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// One array of 2^k elements through LDS by NT threads, t of them, each moving
// at most VPT vectors: k_rows' and k_rows_bytes' steps where a row has them,
// element by element for 1- and 2-byte elements off the 4-byte grid and for
// the rows of k < 2 c too long for a wavefront's lanes.  The element loops
// read eight at once, and the banks are spread (50 int16 arrays of 2^0-2^14:
// 17.3 us one by one, 12.5 by eight, 7.6 with the spread and a workgroup each).
template <int S, int NT, int VPT, int H, typename Sync>
__device__ __forceinline__ void whole_array(const char* in, char* out, int k, u32x4* lds,
                                            uint32_t t, Sync sync) {
  typedef typename Bytes<S>::T E;
  constexpr int C = vec_log2(S), CE = 1 << C;
  const bool vec = S >= 4 || ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 3u) == 0;
  if constexpr (S >= 2) {
    if (k >= 2 * C && vec) {
      constexpr int T = (VPT + CE - 1) / CE;
      const int w = k - 2 * C, lv = k - C;
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const uint32_t q = t + i * NT;
        if (q < (1u << w)) {
          u32x4 a[CE], r[CE];
#pragma unroll
          for (int e = 0; e < CE; ++e)
            a[e] = ld_vec<H>(in + q * 16u + ((uint32_t)e << (w + 4)));
          rows_transpose<S>(a, r);
          const uint32_t o = rev_bits(q, w);
#pragma unroll
          for (int j = 0; j < CE; ++j) lds[rows_slot(o + ((uint32_t)crev(j, C) << w))] = r[j];
        }
      }
      sync();
#pragma unroll
      for (int i = 0; i < VPT; ++i) {
        const uint32_t v = t + i * NT;
        if (v < (1u << lv)) st_vec<H>(out + v * 16u, lds[rows_slot(v)]);
      }
      return;
    }
  }
  if constexpr (S == 1) {
    if (k >= 8 && vec) {
      constexpr int T = (VPT + 3) / 4;
      const int w = k - 6, lv = k - 4;
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const uint32_t q = t + i * NT;
        if (q < (1u << w)) {
          uint32_t a[16];
          u32x4 r[4];
#pragma unroll
          for (int e = 0; e < 16; ++e)
            a[e] = *reinterpret_cast<const uint32_t*>(in + q * 4u + ((uint32_t)e << lv));
          bytes_transpose(a, r);
          const uint32_t o = rev_bits(q, w);
#pragma unroll
          for (int j = 0; j < 4; ++j) lds[rows_slot(o + ((uint32_t)crev(j, 2) << w))] = r[j];
        }
      }
      sync();
#pragma unroll
      for (int i = 0; i < VPT; ++i) {
        const uint32_t v = t + i * NT;
        if (v < (1u << lv)) st_vec<H>(out + v * 16u, lds[rows_slot(v)]);
      }
      return;
    }
  }
  E* le = reinterpret_cast<E*>(lds);
  const uint32_t n = 1u << k;
  if (S < 4 && k >= C && vec) {
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const uint32_t v = t + i * NT;
      if (v < n / CE) lds[v] = ld_vec<kHintPlain>(in + v * 16u);
    }
    sync();
#pragma unroll 1
    for (uint32_t v = t; v < n / CE; v += NT) {
      Chunk<S, 16> c;
#pragma unroll
      for (int e = 0; e < CE; ++e) c.e[e] = le[rev_bits(v * CE + e, k)];
      st_vec<kHintPlain>(out + v * 16u, c.v);
    }
    return;
  }
  // element i's place: the lanes of the reversed read differ in i's top bits,
  // which the XOR brings into the low ones, the banks
  const int sh = k > 6 ? k - 6 : 1;
  const auto at = [sh](uint32_t i) { return i ^ (i >> sh); };
  constexpr int kAtOnce = 8;
  const E* ein = reinterpret_cast<const E*>(in);
  E* eout = reinterpret_cast<E*>(out);
#pragma unroll 1
  for (uint32_t i0 = t; i0 < n; i0 += kAtOnce * NT) {
    E x[kAtOnce];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u)
      if (i0 + u * NT < n) x[u] = ein[i0 + u * NT];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u)
      if (i0 + u * NT < n) le[at(i0 + u * NT)] = x[u];
  }
  sync();
#pragma unroll 1
  for (uint32_t i0 = t; i0 < n; i0 += kAtOnce * NT) {
    E x[kAtOnce];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u)
      if (i0 + u * NT < n) x[u] = le[at(rev_bits(i0 + u * NT, k))];
#pragma unroll
    for (int u = 0; u < kAtOnce; ++u)
      if (i0 + u * NT < n) eout[i0 + u * NT] = x[u];
  }
}

// The scan workgroups, then workgroups of front_arrays consecutive arrays:
// each wavefront reads their metadata in its lanes (one latency for all); the
// arrays beyond 4 KiB take the whole workgroup, one after the other, and the
// others one wavefront each, in turn.
//
// Bound by latency: an array is one chain of metadata, load and store, and
// those beyond 4 KiB follow one another in their workgroup; the 95 registers
// of the 8-byte kernel leave two workgroups of 32 KiB per CU, four wavefronts
// per SIMD.  Measured on 20000 uneven complex64 arrays of 2^0-2^12 out of place
// (a copy of the bytes: 31 us), the two kernels of a call together: 188 us
// where a persistent kernel took each array with 1024 threads, after a search
// for it in the scan; 51 us.
template <int S, int LB, int H>
__global__ __launch_bounds__(front_threads(LB)) void k_batched_front(const void* src, void* data,
                                                                 BatchMeta m, int scan_blocks,
                                                                 int64_t* ws) {
  constexpr int NT = front_threads(LB), kWaves = NT / 64;
  if ((int)blockIdx.x < scan_blocks) {
    batched_scan<NT>(m, ws, (int)blockIdx.x, scan_blocks);
    return;
  }
  constexpr int kWaveBytes = 4096;
  __shared__ u32x4 lds[1 << (LB - 4)];
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
  const char* in = static_cast<const char*>(m.oop ? src : data);
  char* out = static_cast<char*>(data);
  const int64_t step = (int64_t)(gridDim.x - (uint32_t)scan_blocks) * m.per;
  for (int64_t a0 = (int64_t)(blockIdx.x - (uint32_t)scan_blocks) * m.per; a0 < m.num;
       a0 += step) {
    int k = -1;
    int64_t o0 = 0;
    if (lane < (uint32_t)m.per && a0 + lane < m.num) {
      k = m.log2n[a0 + lane];
      o0 = m.offsets[a0 + lane];
      if (!array_ok(m, k, o0, m.offsets[a0 + lane + 1]) || k > m.whole || (k <= 1 && !m.oop)) k = -1;
    }
    // (element by element, a wavefront alone would take 4 KiB in 32 or 64 steps)
    const bool steps = S < 4 && k > 9 && ((reinterpret_cast<uintptr_t>(in) + S * o0) |
                                          (reinterpret_cast<uintptr_t>(out) + S * o0)) & 3u;
    const bool one_wave = k >= 0 && ((int64_t)S << k) <= kWaveBytes && !steps;
    uint64_t small = __ballot(one_wave), large = __ballot(k >= 0 && !one_wave);
    while (large) {
      const int i = __builtin_ctzll(large);
      large &= large - 1;
      const int ki = __builtin_amdgcn_readlane(k, i);
      const int64_t off = S * lane_value(o0, i);
      whole_array<S, NT, 4, H>(in + off, out + off, ki, lds, t, BlockSync());
      __syncthreads();  // the array has left LDS
    }
    uint32_t turn = 0;
    while (small) {
      const int i = __builtin_ctzll(small);
      small &= small - 1;
      if ((turn++ & (kWaves - 1)) != wave) continue;
      const int ki = __builtin_amdgcn_readlane(k, i);
      const int64_t off = S * lane_value(o0, i);
      if (ki <= 6 && ki < 2 * vec_log2(S)) {
        typedef typename Bytes<S>::T E;
        wave_array<S>(reinterpret_cast<const E*>(in + off), reinterpret_cast<E*>(out + off), ki,
                      (int)lane);
      } else {
        WaveSync sync;
        whole_array<S, 64, 4, H>(in + off, out + off, ki, lds + wave * (kWaveBytes / 16), lane,
                                 sync);
        sync();
      }
    }
    __syncthreads();
  }
}

template <int S, int LB> hipError_t run_front(const BatchedLaunch& a, hipStream_t st) {
  BatchMeta m;
  m.offsets = a.offsets;
  m.log2n = a.log2n;
  m.num = a.num;
  m.data_elems = a.data_elems;
  m.b = a.b;
  m.whole = a.whole;
  m.oop = a.src != nullptr ? 1 : 0;
  const int64_t want = (a.num + kArraysPerScan - 1) / kArraysPerScan;
  const int scan = (int)(want < kMaxScanBlocks ? want : kMaxScanBlocks);
  const int64_t few = a.num / kMinFrontBlocks;
  m.per = few < 1 ? 1 : few < front_arrays(LB) ? (int)few : front_arrays(LB);
  const int64_t blocks = (a.num + m.per - 1) / m.per;
  const uint32_t grid = (uint32_t)scan + (uint32_t)(blocks < (1 << 20) ? blocks : (1 << 20));
  if (a.hints == kHintStreamWriteThrough) {
    hipLaunchKernelGGL((k_batched_front<S, LB, kHintStreamWriteThrough>), dim3(grid),
                       dim3(front_threads(LB)), 0, st, a.src, a.data, m, scan, a.ws);
  } else {
    hipLaunchKernelGGL((k_batched_front<S, LB, kHintPlain>), dim3(grid), dim3(front_threads(LB)), 0,
                       st, a.src, a.data, m, scan, a.ws);
  }
  return hipGetLastError();
}

template <int S> hipError_t run_front_s(const BatchedLaunch& a, hipStream_t st) {
  return ((uint64_t)S << a.whole) <= 16384 ? run_front<S, 14>(a, st) : run_front<S, 15>(a, st);
}

}  // namespace

hipError_t launch_batched_front(int s, const BatchedLaunch& a, hipStream_t st) {
  switch (s) {
    case 1: return run_front_s<1>(a, st);
    case 2: return run_front_s<2>(a, st);
    case 4: return run_front_s<4>(a, st);
    case 8: return run_front_s<8>(a, st);
    default: return run_front_s<16>(a, st);
  }
}

}  // namespace bitrev
