// The whole-row kernels for every element size (see bitrev_rows.hpp) and
// their launcher.
#include "bitrev_launch.hpp"
#include "bitrev_rows.hpp"

namespace bitrev {
namespace {

template <int S, int LB, int H, int LH> hipError_t run_rows(const RowsLaunch& a, hipStream_t st) {
  hipLaunchKernelGGL((k_rows<S, LB, H, LH>), dim3(a.grid), dim3(rows_threads(S, LB)), 0, st, a.src,
                     a.dst, a.k, a.runs, a.src_pitch, a.dst_pitch);
  return hipGetLastError();
}

template <int LB, int H, int LH> hipError_t run_bytes(const RowsLaunch& a, hipStream_t st) {
  hipLaunchKernelGGL((k_rows_bytes<LB, H, LH>), dim3(a.grid), dim3(bytes_threads(LB)), 0, st, a.src,
                     a.dst, a.k, a.runs, a.src_pitch, a.dst_pitch);
  return hipGetLastError();
}

template <int S, int LB, int H> hipError_t run_gather(const RowsLaunch& a, hipStream_t st) {
  hipLaunchKernelGGL((k_rows_gather<S, LB, H>), dim3(a.grid), dim3(gather_threads(LB)), 0, st,
                     a.src, a.dst, a.k, a.runs, a.run_log2, a.tail, a.src_pitch, a.dst_pitch);
  return hipGetLastError();
}

template <int S, int H, int LH> hipError_t run_rows_s(const RowsLaunch& a, hipStream_t st) {
  if (a.gather) {
    if constexpr (S == 1) return run_gather<S, 12, H>(a, st);
    if constexpr (S == 2 || S == 4 || S == 8) return run_gather<S, 14, H>(a, st);
  } else if constexpr (S == 1) {
    if (a.chunk_log2 == 14) return run_bytes<14, H, LH>(a, st);
    if constexpr (H == kHintPlain) {  // longer rows only off the 16-byte grid, with plain stores
      if (a.chunk_log2 == 15) return run_bytes<15, H, LH>(a, st);
      if (a.chunk_log2 == 16) return run_bytes<16, H, LH>(a, st);
    }
  } else {
    if constexpr (S == 16)
      if (a.chunk_log2 == 13) return run_rows<S, 13, H, LH>(a, st);
    if (a.chunk_log2 == 14) return run_rows<S, 14, H, LH>(a, st);
    // (16-byte elements are always on the 16-byte grid: rows of 16 KiB at most)
    if constexpr (H == kHintPlain && S < 16) {
      if (a.chunk_log2 == 15) return run_rows<S, 15, H, LH>(a, st);
      if (a.chunk_log2 == 16) return run_rows<S, 16, H, LH>(a, st);
    }
  }
  return hipErrorInvalidValue;
}

// Write-through launches keep plain loads where the parts a wavefront reads
// of a row (16 / S parts) are shorter than 64 bytes: streaming loads fetch
// such a line once for each part (us per MiB moved, 140-180 MiB, streaming ->
// plain: uint8 2^8 0.57 -> 0.35, 2^9 0.36 -> 0.34; int16 2^6 0.53 -> 0.38, 2^7
// 0.41 -> 0.36; float32 2^4 and 2^5 0.39 -> 0.35).  8- and 16-byte elements
// have two parts or one and read their line at once.
template <int S> hipError_t run_rows_hint(const RowsLaunch& a, hipStream_t st) {
  constexpr int kThrough = kHintStreamWriteThrough;
  if (a.hints != kThrough) return run_rows_s<S, kHintPlain, kHintPlain>(a, st);
  if constexpr (S <= 4)
    if (!a.gather && ((uint64_t)S * S << a.k) < 16 * 64)
      return run_rows_s<S, kThrough, kHintPlain>(a, st);
  return run_rows_s<S, kThrough, kThrough>(a, st);
}

template <int S, int LV, int H, int LH>
hipError_t run_rows_dit(const RowsDitLaunch& a, hipStream_t st) {
  hipLaunchKernelGGL((k_rows_dit<S, kRowsDitLog2, LV, H, LH>), dim3(a.grid),
                     dim3(dit_rows_threads(kRowsDitLog2)), 0, st, a.src, a.dst, a.k, a.rows,
                     a.inverse);
  return hipGetLastError();
}

template <int S, int LV> hipError_t run_rows_dit_hint(const RowsDitLaunch& a, hipStream_t st) {
  constexpr int kThrough = kHintStreamWriteThrough;
  if (a.hints != kThrough) return run_rows_dit<S, LV, kHintPlain, kHintPlain>(a, st);
  // plain loads for parts shorter than a 128-byte line, as in run_rows_hint
  if (((uint64_t)S << a.k) < 8 * 128) return run_rows_dit<S, LV, kThrough, kHintPlain>(a, st);
  return run_rows_dit<S, LV, kThrough, kThrough>(a, st);
}

template <int S> hipError_t run_rows_dit_levels(const RowsDitLaunch& a, hipStream_t st) {
  switch (a.stages) {
    case 1: return run_rows_dit_hint<S, 1>(a, st);
    case 2: return run_rows_dit_hint<S, 2>(a, st);
    case 3: return run_rows_dit_hint<S, 3>(a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_rows_dit(int s, const RowsDitLaunch& a, hipStream_t st) {
  return s == 8 ? run_rows_dit_levels<8>(a, st) : run_rows_dit_levels<16>(a, st);
}

int rows_block_threads(int s, int chunk_log2, bool gather) {
  return gather ? gather_threads(chunk_log2)
         : s == 1 ? bytes_threads(chunk_log2)
                  : rows_threads(s, chunk_log2);
}

hipError_t launch_rows(int s, const RowsLaunch& a, hipStream_t st) {
  switch (s) {
    case 1: return run_rows_hint<1>(a, st);
    case 2: return run_rows_hint<2>(a, st);
    case 4: return run_rows_hint<4>(a, st);
    case 8: return run_rows_hint<8>(a, st);
    default: return run_rows_hint<16>(a, st);
  }
}

}  // namespace bitrev
