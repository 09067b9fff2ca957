"""Performance cases: the calls that programs make of this library, each
through its public entry points.

A bit-reversal library is used as the reordering step of radix-2 (and, with
digits, radix-4/8) FFTs: on one array of any length, on rows of equal length
(frames, channels, images), on packed arrays of uneven length, fused with the
first butterfly levels, and under autograd.  ``listed()`` names one case of
each; ``draw(rng)`` gives others of the same ranges.

A case is a dict of plain values.  ``kind`` selects the call:

    both        bitrev_inplace and bitrev_outofplace of two small arrays
    inplace     bitrev_inplace of one array
    outofplace  bitrev_outofplace of one array into a kept destination
    rows        bitrev_rows of a matrix, in place or out of place
    strided     bitrev_rows_strided in place: rows at a padded pitch
    autograd    the differentiable form, forward and backward
    batched     bitrev_batched / bitrev_batched_outofplace, uneven lengths
    dit         bitrev_dit_stages out of place: reversal and butterfly levels
    digit       bitrev_digitrev_inplace / bitrev_digitrev_outofplace
"""
from __future__ import annotations

import numpy as np
import torch

import paper_1708_01873_amd as br
from paper_1708_01873_amd.autograd import bitrev

DTYPES = {
    "uint8": torch.uint8,
    "int16": torch.int16,
    "int32": torch.int32,
    "float32": torch.float32,
    "float64": torch.float64,
    "complex64": torch.complex64,
    "complex128": torch.complex128,
}
SIZE = {"uint8": 1, "int16": 2, "int32": 4, "float32": 4, "float64": 8, "complex64": 8,
        "complex128": 16}


def listed():
    return [
        # one small array of 32-bit words, both forms: a program that
        # transforms single short vectors; launch and call latency
        {"name": "both_i32_2p10", "kind": "both", "dtype": "int32", "k": 10},
        # one complex64 array of 128 MiB in place: a long one-dimensional FFT
        {"name": "inplace_c64_2p24", "kind": "inplace", "dtype": "complex64", "k": 24},
        # the paper's own workload, complex doubles of 2^24, out of place
        {"name": "outofplace_c128_2p24", "kind": "outofplace", "dtype": "complex128", "k": 24},
        # the largest array, 4 GiB of float32 in place: nothing fits a cache
        {"name": "inplace_f32_2p30", "kind": "inplace", "dtype": "float32", "k": 30},
        # frames of a short-time transform: many rows of 2^10 complex64
        {"name": "rows_c64_8192x2p10", "kind": "rows", "dtype": "complex64", "k": 10, "rows": 8192,
         "inplace": False},
        # very short rows in place, an odd count: small FFTs of one dimension
        # of an array (blocks of 32)
        {"name": "rows_c64_99991x2p5", "kind": "rows", "dtype": "complex64", "k": 5, "rows": 99991,
         "inplace": True},
        # real rows at the padded pitch of an in-place real FFT (n + 2 floats)
        {"name": "strided_f32_3000x2p12", "kind": "strided", "dtype": "float32", "k": 12,
         "rows": 3000, "pad": 2},
        # the differentiable form on a batch of 256 rows of 2^16 float32
        {"name": "autograd_f32_256x2p16", "kind": "autograd", "dtype": "float32", "k": 16,
         "rows": 256},
        # thousands of arrays of uneven length in one call, in place
        {"name": "batched_c64_4096", "kind": "batched", "dtype": "complex64", "num": 4096,
         "kmin": 8, "kmax": 20, "inplace": True},
        # a ragged batch of short arrays out of place, single elements among
        # them, so that later arrays start off the 16-byte grid
        {"name": "batched_oop_c64_ragged", "kind": "batched", "dtype": "complex64", "num": 20000,
         "kmin": 0, "kmax": 12, "inplace": False},
        # bit reversal fused with six butterfly levels, rows of 2^16 complex64
        {"name": "dit6_c64_256x2p16", "kind": "dit", "dtype": "complex64", "k": 16, "rows": 256,
         "stages": 6, "inverse": False},
        # radix-4 digit reversal in place, complex64 of 2^22
        {"name": "digit4_c64_2p22", "kind": "digit", "dtype": "complex64", "k": 22,
         "digit_bits": 2, "inplace": True},
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _rows_for(rng, k, size, lo_bytes, hi_bytes):
    """A row count that puts the matrix between the two footprints."""
    lo = max(1, lo_bytes // (size << k))
    return _log_uniform(rng, lo, max(lo, hi_bytes // (size << k)))


def draw(rng):
    kind = rng.choice(["both", "inplace", "inplace", "outofplace", "outofplace", "rows", "rows",
                       "strided", "autograd", "batched", "batched", "dit", "dit", "digit"])
    any_type = ["uint8", "int16", "int32", "float32", "float64", "complex64", "complex128"]
    if kind == "both":
        return {"kind": kind, "dtype": rng.choice(any_type), "k": rng.randint(5, 18)}
    if kind in ("inplace", "outofplace"):
        # 512 KiB to 4 GiB (out of place 2 GiB)
        dtype = rng.choice(any_type)
        shift = SIZE[dtype].bit_length() - 1
        return {"kind": kind, "dtype": dtype,
                "k": rng.randint(19, 32 if kind == "inplace" else 31) - shift}
    if kind == "rows":
        dtype = rng.choice(["int16", "float32", "complex64", "complex64", "complex128"])
        k = rng.randint(2, 15)
        return {"kind": kind, "dtype": dtype, "k": k,
                "rows": _rows_for(rng, k, SIZE[dtype], 1 << 19, 1 << 28),
                "inplace": rng.random() < 0.5}
    if kind == "strided":
        dtype = rng.choice(["int16", "float32", "float64"])
        k = rng.randint(6, 15)
        return {"kind": kind, "dtype": dtype, "k": k,
                "rows": _rows_for(rng, k, SIZE[dtype], 1 << 19, 1 << 28),
                "pad": rng.choice([2, 2, 16, 64])}
    if kind == "autograd":
        dtype = rng.choice(["float32", "float32", "float64"])
        k = rng.randint(6, 18)
        return {"kind": kind, "dtype": dtype, "k": k,
                "rows": _rows_for(rng, k, SIZE[dtype], 1 << 20, 1 << 28)}
    if kind == "batched":
        dtype = rng.choice(["float32", "complex64", "complex64", "complex128"])
        kmin = rng.randint(0, 10)
        kmax = rng.randint(kmin + 2, 20)
        # the expected footprint stays under 2 GiB
        most = (1 << 31) * (kmax - kmin + 1) // (SIZE[dtype] << (kmax + 1))
        return {"kind": kind, "dtype": dtype, "num": _log_uniform(rng, 64, max(64, min(20000, most))),
                "kmin": kmin, "kmax": kmax, "inplace": rng.random() < 0.5}
    if kind == "dit":
        dtype = rng.choice(["complex64", "complex64", "complex128"])
        k = rng.randint(6, 24)
        rows = 1 if k > 20 else _rows_for(rng, k, SIZE[dtype], 1 << 20, 1 << 28)
        return {"kind": kind, "dtype": dtype, "k": k, "rows": rows,
                "stages": rng.randint(1, min(6, k // 2)), "inverse": rng.random() < 0.5}
    d = rng.choice([2, 3])
    dtype = rng.choice(["float32", "complex64", "complex64", "complex128"])
    return {"kind": kind, "dtype": dtype, "k": d * rng.randint(-(-12 // d), 26 // d),
            "digit_bits": d, "inplace": rng.random() < 0.5}


def _values(n, dtype, seed):
    """n values on the GPU: N(0, 1) for the floating types (both parts of the
    complex ones), uniform over all bit patterns for the integers."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    t = DTYPES[dtype]
    if t.is_complex:
        part = torch.float32 if t == torch.complex64 else torch.float64
        return torch.randn(2 * n, dtype=part, device="cuda", generator=g).view(t)
    if t.is_floating_point:
        return torch.randn(n, dtype=t, device="cuda", generator=g)
    info = torch.iinfo(t)
    return torch.randint(info.min, info.max + 1, (n,), dtype=t, device="cuda", generator=g)


def _layout(case, seed):
    """log2 lengths uniform in [kmin, kmax], arrays packed back to back: the
    case's own set of lengths, in an order drawn from the seed."""
    rng = np.random.default_rng(case["num"])
    log2n = rng.integers(case["kmin"], case["kmax"] + 1, size=case["num"]).astype(np.int32)
    np.random.default_rng(seed).shuffle(log2n)
    offsets = np.zeros(case["num"] + 1, dtype=np.int64)
    np.cumsum(np.left_shift(np.int64(1), log2n.astype(np.int64)), out=offsets[1:])
    return offsets, log2n


def prepare(case, seed):
    kind, dtype = case["kind"], case["dtype"]
    s = {"case": case}
    if kind == "both":
        s["a"] = _values(1 << case["k"], dtype, seed)
        s["b"] = _values(1 << case["k"], dtype, seed + 500009)
        s["out"] = torch.empty_like(s["b"])
    elif kind in ("inplace", "outofplace", "digit"):
        s["x"] = _values(1 << case["k"], dtype, seed)
        if kind == "outofplace" or not case.get("inplace", True):
            s["out"] = torch.empty_like(s["x"])
    elif kind in ("rows", "dit"):
        s["x"] = _values(case["rows"] << case["k"], dtype, seed).view(case["rows"], -1)
        s["out"] = s["x"] if case.get("inplace") else torch.empty_like(s["x"])
    elif kind == "strided":
        pitch = (1 << case["k"]) + case["pad"]
        s["x"] = _values(case["rows"] * pitch, dtype, seed)
        s["pitch"] = pitch
    elif kind == "autograd":
        s["x"] = _values(case["rows"] << case["k"], dtype, seed).view(case["rows"], -1)
        s["x"].requires_grad_()
        s["w"] = _values(case["rows"] << case["k"], dtype, seed + 500009).view(case["rows"], -1)
    else:
        offsets, log2n = _layout(case, seed)
        s["x"] = _values(int(offsets[-1]), dtype, seed)
        s["offsets"] = torch.from_numpy(offsets).cuda()
        s["log2n"] = torch.from_numpy(log2n).cuda()
        s["workspace"] = torch.empty(br.bitrev_batched_workspace_size(case["num"]),
                                     dtype=torch.uint8, device="cuda")
        if not case["inplace"]:
            s["out"] = torch.empty_like(s["x"])
    return s


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "both":
        return [br.bitrev_inplace(state["a"]), br.bitrev_outofplace(state["b"], state["out"])]
    if kind == "inplace":
        return br.bitrev_inplace(state["x"])
    if kind == "outofplace":
        return br.bitrev_outofplace(state["x"], state["out"])
    if kind == "rows":
        return br.bitrev_rows(state["x"], state["out"])
    if kind == "strided":
        return br.bitrev_rows_strided(state["x"], state["x"], case["k"], case["rows"],
                                      state["pitch"], state["pitch"])
    if kind == "autograd":
        y = bitrev(state["x"])
        (gx,) = torch.autograd.grad(y, state["x"], state["w"])
        return [y, gx]
    if kind == "batched":
        if case["inplace"]:
            return br.bitrev_batched(state["x"], state["offsets"], state["log2n"],
                                     state["workspace"])
        return br.bitrev_batched_outofplace(state["x"], state["out"], state["offsets"],
                                            state["log2n"], state["workspace"])
    if kind == "dit":
        return br.bitrev_dit_stages(state["x"], state["out"], case["stages"],
                                    inverse=case["inverse"])
    if case["inplace"]:
        return br.bitrev_digitrev_inplace(state["x"], case["digit_bits"])
    return br.bitrev_digitrev_outofplace(state["x"], state["out"], case["digit_bits"])


def work(case):
    """Each element read once and written once (the elements the permutation
    leaves in place count too: a pass moves whole cache lines)."""
    kind, size = case["kind"], SIZE[case["dtype"]]
    flops = 0
    if kind in ("both", "autograd"):
        elems = 2 * case.get("rows", 1) << case["k"]
    elif kind == "batched":
        # the mean length of the layout's arrays
        elems = case["num"] * ((2 << case["kmax"]) - (1 << case["kmin"])) // (
            case["kmax"] - case["kmin"] + 1)
    else:
        elems = case.get("rows", 1) << case["k"]
    if kind == "dit":
        flops = 5 * case["stages"] * elems  # ten per butterfly, half as many butterflies
    return {"bytes": 2 * size * elems, "flops": flops}


def _rev_index(k, d=1):
    """The reversal of the d-bit digits of 0 .. 2^k - 1: a new top digit e of
    the index becomes the lowest digit of its reversal."""
    r = torch.zeros(1, dtype=torch.int64, device="cuda")
    for _ in range(k // d):
        r = torch.cat([(r << d) + e for e in range(1 << d)])
    return r


def _wide(x):
    if x.dtype.is_complex:
        return x.to(torch.complex128)
    return x.to(torch.float64) if x.dtype.is_floating_point else x


def exact(case, seed):
    """What ``run`` returns for a new state, by indexing and a 64-bit FFT."""
    kind, dtype, k = case["kind"], case["dtype"], case.get("k", 0)
    if kind == "both":
        rev = _rev_index(k)
        return [_wide(_values(1 << k, dtype, seed)[rev]),
                _wide(_values(1 << k, dtype, seed + 500009)[rev])]
    if kind in ("inplace", "outofplace"):
        return _wide(_values(1 << k, dtype, seed)[_rev_index(k)])
    if kind == "digit":
        return _wide(_values(1 << k, dtype, seed)[_rev_index(k, case["digit_bits"])])
    if kind == "rows":
        return _wide(_values(case["rows"] << k, dtype, seed).view(case["rows"], -1)[:, _rev_index(k)])
    if kind == "strided":
        x = _values(case["rows"] * ((1 << k) + case["pad"]), dtype, seed)
        m = x.view(case["rows"], -1)
        m[:, :1 << k] = m[:, _rev_index(k)]
        return _wide(x)
    if kind == "autograd":
        rev = _rev_index(k)
        shape = (case["rows"], -1)
        return [_wide(_values(case["rows"] << k, dtype, seed).view(shape)[:, rev]),
                _wide(_values(case["rows"] << k, dtype, seed + 500009).view(shape)[:, rev])]
    if kind == "batched":
        offsets, log2n = _layout(case, seed)
        x = _values(int(offsets[-1]), dtype, seed)
        out = torch.empty_like(x)
        for k in range(case["kmin"], case["kmax"] + 1):
            first = torch.from_numpy(offsets[:-1][log2n == k]).cuda()[:, None]
            span = torch.arange(1 << k, device="cuda")[None, :]
            out[(first + span).view(-1)] = x[(first + _rev_index(k)[None, :]).view(-1)]
        return _wide(out)
    # the first L levels after the reversal leave each block of 2^L outputs as
    # the DFT of that block's elements in their order before the reversal
    rows, L = case["rows"], case["stages"]
    x = _values(rows << k, dtype, seed).view(rows, -1)[:, _rev_index(k)].to(torch.complex128)
    blocks = x.view(-1, 1 << L)[:, _rev_index(L)]
    if case["inverse"]:
        y = torch.fft.ifft(blocks, norm="forward")
    else:
        y = torch.fft.fft(blocks)
    return y.reshape(rows, -1)
