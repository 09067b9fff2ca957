// Whole rows in LDS: the bit reversal of many short arrays of equal length.
// A workgroup takes a run of whole rows, so both its reads and its writes are
// linear in memory whatever the row length, and nothing is shared between
// workgroups: in place, every row is read before the barrier and written
// after it.
//
// Bound by memory: one 16-byte LDS write and one read per 16 bytes moved is
// far below the LDS rate.  The tile kernels split a short row into 2^b x 2^b
// tiles of 2^b s bytes a row (k = 5, complex64: 32 bytes; 9, float32: 64), and
// the wavefront kernel for k <= 6 leaves 64 - 2^k lanes idle.  Measured,
// kernel time at 32 MiB, three arrays in turn (a copy of the bytes: 10.5 us):
// complex64 k = 2 67.7 -> 10.5 us, 5 16.5 -> 10.5, 7 15.9 -> 10.6, 11 11.3 ->
// 10.8; float32 3 59.1 -> 10.1, 9 20.9 -> 10.9; int16 9 21.2 -> 10.7; uint8 7
// 107 -> 13; rows at a pitch of n + 2: float64 9 31.9 -> 11.0, float32 13
// 17.5 -> 11.5.  Below 4 MiB both are launch-bound and equal.
#pragma once

#include "bitrev_device.hpp"

namespace bitrev {

// 16 bytes at any multiple of 4 bytes: gfx950's wide global accesses need
// dword alignment only, so rows at a padded pitch move as vectors too.  The
// accessors name the type: a template parameter deduced from it would be the
// vector without the attribute, and the access would claim 16.
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));

template <int H> __device__ __forceinline__ u32x4 ld_vec(const u32x4_a4* q) {
  if constexpr (H == kHintStreamLoads || H == kHintStreamWriteThrough) {
    return __builtin_nontemporal_load(q);
  } else {
    return *q;
  }
}

template <int H> __device__ __forceinline__ u32x4 ld_vec(const char* p) {
  return ld_vec<H>(reinterpret_cast<const u32x4_a4*>(p));
}

template <int H> __device__ __forceinline__ void st_vec(u32x4_a4* q, u32x4 v) {
  if constexpr (H == kHintStreamStores) {
    __builtin_nontemporal_store(v, q);
  } else if constexpr (H == kHintStreamWriteThrough) {
    st_through(reinterpret_cast<u32x4*>(q), v);  // one instruction: it claims nothing
  } else {
    *q = v;
  }
}

template <int H> __device__ __forceinline__ void st_vec(char* p, u32x4 v) {
  st_vec<H>(reinterpret_cast<u32x4_a4*>(p), v);
}

// log2 of the elements per 16-byte vector.
__host__ __device__ constexpr int vec_log2(int s) { return s == 16 ? 0 : s == 8 ? 1 : s == 4 ? 2 : s == 2 ? 3 : 4; }

// Transposed groups of CE = 16 / s vectors a thread moves per chunk of 2^lb
// bytes.  One group (two 16-byte accesses for complex64) ran 1-4% ahead of
// two from 64 MiB up and level below; wider chunks need more to stay within
// 1024 threads, and at 16 bytes 8 KiB chunks of one were 2% ahead of 16 KiB
// of two at 128-512 MiB.
__host__ __device__ constexpr int rows_groups(int s, int lb) {
  return (s == 16 && lb >= 14) || (s == 8 && lb >= 15) ? 2 : 1;
}

// Threads of a workgroup of k_rows whose chunk has 2^lb bytes.
__host__ __device__ constexpr int rows_threads(int s, int lb) {
  return (1 << (lb - 4)) / (rows_groups(s, lb) * (16 / s));
}

// Threads of a workgroup of k_rows_gather: four vectors each.
__host__ __device__ constexpr int gather_threads(int lb) { return 1 << (lb - 6); }

// Physical slot of 16-byte slot v: the low three bits (the eight slots of a
// 128-byte LDS line) XORed with the fold of all higher bits in groups of
// three.  The scatter's eight neighbouring lanes differ in three consecutive
// slot bits, which the fold maps onto the three low ones, and the linear
// reads stay permutations within aligned runs of eight.
__device__ __forceinline__ uint32_t rows_slot(uint32_t v) {
  return v ^ (((v >> 3) ^ (v >> 6) ^ (v >> 9)) & 7u);
}

// The CE vectors a[e] of CE elements, as CE vectors r[j] with
// r[j][rev(e)] = a[e][j] (e and j of vec_log2(S) bits).
template <int S> __device__ __forceinline__ void rows_transpose(const u32x4 (&a)[16 / S], u32x4 (&r)[16 / S]) {
  if constexpr (S == 16) {
    r[0] = a[0];
  } else if constexpr (S == 8) {
    r[0] = __builtin_shufflevector(a[0], a[1], 0, 1, 4, 5);
    r[1] = __builtin_shufflevector(a[0], a[1], 2, 3, 6, 7);
  } else if constexpr (S == 4) {
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = u32x4{a[0][j], a[2][j], a[1][j], a[3][j]};
  } else {
    static_assert(S == 2, "2-byte elements");
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int d = 0; d < 4; ++d)  // halves 2d and 2d + 1 of r[j]
        r[j][d] = __builtin_amdgcn_perm(a[crev(2 * d + 1, 3)][j >> 1], a[crev(2 * d, 3)][j >> 1],
                                        (j & 1) ? 0x07060302u : 0x05040100u);
  }
}

// Rows of 2^k elements, k >= 2 c (c = vec_log2(S)), 2^k S <= 2^LB bytes: a
// thread loads the CE vectors at one offset q of the CE equal parts of a row
// (part e holds the elements whose top c index bits are e), and their
// transpose in registers is CE whole output vectors: element (e, q, j) of the
// index [e | q | j] goes to [rev(j) | rev(q) | rev(e)], so output vector j is
// vector [rev(j) | rev(q)] of the row.  One 16-byte LDS write and read per
// vector turn the scattered vectors into linear runs.
// LH: the hint of the loads, H that of the stores (both streaming forms bypass
// the caches for a line the kernel touches once; a part of less than 64 bytes
// shares its line with the next).
template <int S, int LB, int H, int LH>
__global__ __launch_bounds__(rows_threads(S, LB)) void k_rows(const void* src, void* dst, int k,
                                                             uint64_t rows, uint64_t src_pitch,
                                                             uint64_t dst_pitch) {
  constexpr int C = vec_log2(S), CE = 1 << C;
  constexpr int NT = rows_threads(S, LB), T = rows_groups(S, LB), PT = T * CE;
  constexpr uint32_t CHV = 1u << (LB - 4);  // vectors per chunk
  __shared__ u32x4 lds[CHV];
  const int w = k - 2 * C, lv = k - C;
  const uint32_t wmask = (1u << w) - 1u, vmask = (1u << lv) - 1u;
  const uint64_t step = (uint64_t)gridDim.x * (CHV >> lv);
  for (uint64_t row0 = (uint64_t)blockIdx.x * (CHV >> lv); row0 < rows; row0 += step) {
    const uint32_t live = rows - row0 < (CHV >> lv) ? (uint32_t)(rows - row0) : CHV >> lv;
    const char* in = static_cast<const char*>(src) + row0 * src_pitch;
    char* out = static_cast<char*>(dst) + row0 * dst_pitch;
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const uint32_t u = threadIdx.x + i * NT;
      const uint32_t q = u & wmask, r = u >> w;
      if (r < live) {
        u32x4 a[CE], t[CE];
        const char* p = in + r * src_pitch + q * 16u;
#pragma unroll
        for (int e = 0; e < CE; ++e)
          a[e] = ld_vec<LH>(p + ((size_t)e << (w + 4)));
        rows_transpose<S>(a, t);
        const uint32_t o = (r << lv) + rev_bits(q, w);
#pragma unroll
        for (int j = 0; j < CE; ++j) lds[rows_slot(o + ((uint32_t)crev(j, C) << w))] = t[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const uint32_t v = threadIdx.x + i * NT;
      const uint32_t r = v >> lv;
      if (r < live)
        st_vec<H>(out + r * dst_pitch + (v & vmask) * 16u, lds[rows_slot(v)]);
    }
    __syncthreads();
  }
}

// Threads of a workgroup of k_rows_bytes: sixteen dwords each.
__host__ __device__ constexpr int bytes_threads(int lb) { return 1 << (lb - 6); }

// The sixteen dwords a[e] of four bytes, as the four vectors t[j] with byte
// t[j][rev(e)] = a[e][j] (e of four bits): 4 x 4 byte transposes.
__device__ __forceinline__ void bytes_transpose(const uint32_t (&a)[16], u32x4 (&t)[4]) {
#pragma unroll
  for (int d = 0; d < 4; ++d) {  // dword d of an output vector: bytes rev(4d + b), b = 0..3
    const int e = crev(d, 2);
    const uint32_t lo0 = __builtin_amdgcn_perm(a[8 + e], a[e], 0x05010400u);
    const uint32_t lo1 = __builtin_amdgcn_perm(a[12 + e], a[4 + e], 0x05010400u);
    const uint32_t hi0 = __builtin_amdgcn_perm(a[8 + e], a[e], 0x07030602u);
    const uint32_t hi1 = __builtin_amdgcn_perm(a[12 + e], a[4 + e], 0x07030602u);
    t[0][d] = __builtin_amdgcn_perm(lo1, lo0, 0x05040100u);
    t[1][d] = __builtin_amdgcn_perm(lo1, lo0, 0x07060302u);
    t[2][d] = __builtin_amdgcn_perm(hi1, hi0, 0x05040100u);
    t[3][d] = __builtin_amdgcn_perm(hi1, hi0, 0x07060302u);
  }
}

// Rows of 2^k bytes, k >= 8.  Whole vectors at one offset of sixteen parts
// would be 64 registers in and 64 out; a thread takes one dword of each part
// instead: byte (e, q, j) of the index [e(4) | q | j(2)] goes to [rev(j) |
// rev(q) | rev(e)], so the four bytes j of the sixteen dwords are four whole
// output vectors, made by 4 x 4 byte transposes (two v_perm a dword).  A
// wavefront reads 16 bytes of each part of a row at k = 8, 256 from k = 12 on;
// below k = 8 the gather is better.
// Bound by memory.  Against a gather of single bytes from LDS (64 byte reads
// for each four vectors), three arrays in turn, us: 2^8 12.9 MiB 8.2 -> 6.8,
// 2^9 29.5 MiB 13.4 -> 10.9, 2^11 34 MiB 12.9 -> 12.0 and 14.9 -> 11.6 out of
// place, 2^13 38 MiB 16.0 -> 13.1 and 17.6 -> 12.7 (a copy of 38 MiB: 12.5).
template <int LB, int H, int LH>
__global__ __launch_bounds__(bytes_threads(LB)) void k_rows_bytes(const void* src, void* dst, int k,
                                                                 uint64_t rows, uint64_t src_pitch,
                                                                 uint64_t dst_pitch) {
  constexpr int NT = bytes_threads(LB);
  constexpr uint32_t CHV = 1u << (LB - 4);
  __shared__ u32x4 lds[CHV];
  const int w = k - 6, lv = k - 4;
  const uint32_t vmask = (1u << lv) - 1u;
  const uint32_t q = threadIdx.x & ((1u << w) - 1u), r = threadIdx.x >> w;
  const uint32_t o = (r << lv) + rev_bits(q, w);
  const uint64_t step = (uint64_t)gridDim.x * (CHV >> lv);
  for (uint64_t row0 = (uint64_t)blockIdx.x * (CHV >> lv); row0 < rows; row0 += step) {
    const uint32_t live = rows - row0 < (CHV >> lv) ? (uint32_t)(rows - row0) : CHV >> lv;
    const char* in = static_cast<const char*>(src) + row0 * src_pitch;
    char* out = static_cast<char*>(dst) + row0 * dst_pitch;
    if (r < live) {
      const char* p = in + r * src_pitch + q * 4u;
      uint32_t a[16];
      u32x4 t[4];
#pragma unroll
      for (int e = 0; e < 16; ++e)
        a[e] = ld_hint<LH>(reinterpret_cast<const uint32_t*>(p + ((size_t)e << lv)));
      bytes_transpose(a, t);
#pragma unroll
      for (int j = 0; j < 4; ++j) lds[rows_slot(o + ((uint32_t)crev(j, 2) << w))] = t[j];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t v = threadIdx.x + i * NT;
      const uint32_t s = v >> lv;
      if (s < live)
        st_vec<H>(out + s * dst_pitch + (v & vmask) * 16u, lds[rows_slot(v)]);
    }
    __syncthreads();
  }
}

// Rows shorter than k = 2 c: a chunk of rows goes to LDS as it is, and each
// output vector gathers its elements one by one.  The data are `nrun` runs of
// 2^lr vectors, `pitch` bytes apart: the rows, or single vectors (lr = 0,
// pitch 16) of contiguous rows shorter than a vector; the `tail` elements
// after the last whole run move alone.
template <int S, int LB, int H>
__global__ __launch_bounds__(gather_threads(LB)) void k_rows_gather(
    const void* src, void* dst, int k, uint64_t nrun, int lr, uint32_t tail, uint64_t src_pitch,
    uint64_t dst_pitch) {
  typedef typename Bytes<S>::T E;
  constexpr int CE = 16 / S, NT = gather_threads(LB), PT = 4;
  constexpr uint32_t CHV = 1u << (LB - 4);
  __shared__ u32x4 lds[CHV];
  const E* le = reinterpret_cast<const E*>(lds);
  const uint32_t nmask = (1u << k) - 1u, rmask = (1u << lr) - 1u;
  const uint64_t step = (uint64_t)gridDim.x * (CHV >> lr);
  for (uint64_t run0 = (uint64_t)blockIdx.x * (CHV >> lr); run0 < nrun; run0 += step) {
    const uint32_t live = nrun - run0 < (CHV >> lr) ? (uint32_t)(nrun - run0) : CHV >> lr;
    const char* in = static_cast<const char*>(src) + run0 * src_pitch;
    char* out = static_cast<char*>(dst) + run0 * dst_pitch;
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const uint32_t v = threadIdx.x + i * NT;
      const uint32_t r = v >> lr;
      if (r < live)
        lds[v] = ld_vec<H>(in + r * src_pitch + (v & rmask) * 16u);
    }
    __syncthreads();
#pragma unroll 1
    for (int i = 0; i < PT; ++i) {
      const uint32_t v = threadIdx.x + i * NT;
      const uint32_t r = v >> lr;
      if (r < live) {
        Chunk<S, 16> c;
#pragma unroll
        for (int e = 0; e < CE; ++e) {
          const uint32_t o = v * CE + e;
          c.e[e] = le[(o & ~nmask) | rev_bits(o & nmask, k)];
        }
        st_vec<H>(out + r * dst_pitch + (v & rmask) * 16u, c.v);
      }
    }
    __syncthreads();
  }
  if (tail && blockIdx.x == 0 && threadIdx.x < 64) {  // less than a vector: one wavefront, in lanes
    const E* in = reinterpret_cast<const E*>(static_cast<const char*>(src) + nrun * src_pitch);
    E* out = reinterpret_cast<E*>(static_cast<char*>(dst) + nrun * dst_pitch);
    const uint32_t o = threadIdx.x;
    const uint32_t from = (o & ~nmask) | rev_bits(o & nmask, k);
    E x = (E)0u;
    if (o < tail) x = in[from];
    if (o < tail) out[o] = x;
  }
}

// Threads of a workgroup of k_rows_dit: eight 16-byte loads each.
__host__ __device__ constexpr int dit_rows_threads(int lb) { return 1 << (lb - 7); }

// The reversal of short complex rows fused with the first LV <= 3 levels: a
// thread loads the vectors at one offset q of a row's eight parts, element (e,
// q, j) of the index [e(3) | q | j]; the eight elements of one j go to the
// contiguous block [rev(j) | rev(q)] of eight outputs, whole blocks of every
// level, so the levels run in registers (dit_block_levels) and one pass
// through LDS makes the writes linear, as in k_rows.
// Bound by memory; the tile kernel's tiles are 2^(k / 2) elements wide (64
// bytes a row at k = 6).  Kernel us, three arrays in turn: complex64 33 MiB
// 2^4, two levels, 96 -> 14.0, 2^5 95 -> 12.6, 2^6, three levels, 29.7 -> 12.4,
// 75 MiB of 2^7 65.6 -> 26.3; complex128 32 MiB 2^4 50.2 -> 11.9, 2^6 16.5 ->
// 10.9 (a copy of 32 MiB: 10.7).
template <int S, int LB, int LV, int H, int LH>
__global__ __launch_bounds__(dit_rows_threads(LB)) void k_rows_dit(const void* src, void* dst, int k,
                                                                  uint64_t rows, int inverse) {
  typedef typename ComplexOf<S>::T F;
  constexpr int C = vec_log2(S), CE = 1 << C, NT = dit_rows_threads(LB);
  constexpr int VB = 8 / CE;  // vectors of a block
  constexpr uint32_t CHV = 1u << (LB - 4);
  __shared__ u32x4 lds[CHV];
  const int w = k - 3 - C, lv = k - C;
  const uint32_t vmask = (1u << lv) - 1u;
  const uint32_t q = threadIdx.x & ((1u << w) - 1u), r = threadIdx.x >> w;
  const F sg = inverse ? (F)-1 : (F)1;
  const uint64_t step = (uint64_t)gridDim.x * (CHV >> lv);
  for (uint64_t row0 = (uint64_t)blockIdx.x * (CHV >> lv); row0 < rows; row0 += step) {
    const uint32_t live = rows - row0 < (CHV >> lv) ? (uint32_t)(rows - row0) : CHV >> lv;
    const u32x4_a4* in = static_cast<const u32x4_a4*>(src) + (row0 << lv);
    u32x4_a4* out = static_cast<u32x4_a4*>(dst) + (row0 << lv);
    if (r < live) {
      Chunk<S, 16> a[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e].v = ld_vec<LH>(in + (r << lv) + q + ((uint32_t)e << w));
#pragma unroll
      for (int j = 0; j < CE; ++j) {
        F re[8], im[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          Cplx<F> x;
          __builtin_memcpy(&x, &a[e].e[j], sizeof(x));
          re[crev(e, 3)] = x.re;
          im[crev(e, 3)] = x.im;
        }
        dit_block_levels<F, 8, LV>(re, im, sg);
        const uint32_t o = (r << lv) + (rev_bits(q, w) + ((uint32_t)crev(j, C) << w)) * VB;
#pragma unroll
        for (int i = 0; i < VB; ++i) {
          Chunk<S, 16> y;
#pragma unroll
          for (int c = 0; c < CE; ++c) {
            const Cplx<F> x{re[i * CE + c], im[i * CE + c]};
            __builtin_memcpy(&y.e[c], &x, sizeof(x));
          }
          lds[rows_slot(o + i)] = y.v;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t v = threadIdx.x + i * NT;
      if ((v >> lv) < live) st_vec<H>(out + v, lds[rows_slot(v)]);
    }
    __syncthreads();
  }
}

}  // namespace bitrev
