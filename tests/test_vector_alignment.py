"""The whole-row kernels' 16-byte accesses start at any multiple of 4 bytes:
what the compiler is told of their alignment must be 4 (CPU: compiles a kernel
of the accessors to LLVM IR)."""
import re
import subprocess

from paper_1708_01873_amd import build

SOURCE = r'''
#include "bitrev_rows.hpp"
using namespace bitrev;
#define MOVE(H)                                                             \
  __global__ void move_##H(const char* a, char* b, int n) {                 \
    st_vec<H>(b + n, ld_vec<H>(a + n));                                     \
  }                                                                         \
  template __global__ void bitrev::k_rows<4, 14, H, H>(const void*, void*, int, uint64_t, \
                                                       uint64_t, uint64_t); \
  template __global__ void bitrev::k_rows_dit<8, 14, 2, H, H>(const void*, void*, int, uint64_t, int); \
  template __global__ void bitrev::k_rows_gather<2, 14, H>(const void*, void*, int, uint64_t, int, \
                                                           uint32_t, uint64_t, uint64_t);
MOVE(kHintPlain) MOVE(kHintStreamStores) MOVE(kHintStreamWriteThrough)
'''


def test_sixteen_byte_accesses_claim_four(tmp_path):
    src, ir = tmp_path / "probe.hip", tmp_path / "probe.ll"
    src.write_text(SOURCE)
    flags = [f for f in build.HIPCC_FLAGS if f != "-Wall"]
    p = subprocess.run([build.hipcc()] + flags + ["--cuda-device-only", "-S", "-emit-llvm",
                                                  str(src), "-o", str(ir)],
                       capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
    seen = {"load": 0, "store": 0}
    for line in ir.read_text().splitlines():
        m = re.search(r"\b(load|store)\b.*<4 x i32>.*addrspace\(1\).*align (\d+)", line)
        if m:
            seen[m[1]] += 1
            assert m[2] == "4", line
    assert min(seen.values()) >= 10, seen


