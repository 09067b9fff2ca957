// The whole-row kernels for every element size (see bitrev_rows.hpp) and
// their launcher.
#include "bitrev_launch.hpp"
#include "bitrev_rows.hpp"

namespace bitrev {
namespace {

template <int S, int LB, int H> hipError_t run_rows(const RowsLaunch& a, hipStream_t st) {
  hipLaunchKernelGGL((k_rows<S, LB, H>), dim3(a.grid), dim3(rows_threads(S, LB)), 0, st, a.src,
                     a.dst, a.k, a.runs, a.src_pitch, a.dst_pitch);
  return hipGetLastError();
}

template <int S, int LB, int H> hipError_t run_gather(const RowsLaunch& a, hipStream_t st) {
  hipLaunchKernelGGL((k_rows_gather<S, LB, H>), dim3(a.grid), dim3(gather_threads(LB)), 0, st,
                     a.src, a.dst, a.k, a.runs, a.run_log2, a.tail, a.src_pitch, a.dst_pitch);
  return hipGetLastError();
}

template <int S, int H> hipError_t run_rows_s(const RowsLaunch& a, hipStream_t st) {
  if (a.gather) {
    if constexpr (S == 1) {
      return a.chunk_log2 == 12 ? run_gather<S, 12, H>(a, st) : run_gather<S, 13, H>(a, st);
    } else if constexpr (S <= 8) {
      return run_gather<S, 14, H>(a, st);
    }
  } else if constexpr (S >= 2) {
    switch (a.chunk_log2) {
      case 13:
        if constexpr (S == 16) return run_rows<S, 13, H>(a, st);
        break;
      case 14: return run_rows<S, 14, H>(a, st);
      case 15:  // longer rows only off the 16-byte grid, with plain stores
        if constexpr (H == kHintPlain) return run_rows<S, 15, H>(a, st);
        break;
      case 16:
        if constexpr (H == kHintPlain) return run_rows<S, 16, H>(a, st);
        break;
    }
  }
  return hipErrorInvalidValue;
}

template <int S> hipError_t run_rows_hint(const RowsLaunch& a, hipStream_t st) {
  return a.hints == kHintStreamWriteThrough ? run_rows_s<S, kHintStreamWriteThrough>(a, st)
                                            : run_rows_s<S, kHintPlain>(a, st);
}

}  // namespace

int rows_block_threads(int s, int chunk_log2, bool gather) {
  return gather ? gather_threads(chunk_log2) : rows_threads(s, chunk_log2);
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
