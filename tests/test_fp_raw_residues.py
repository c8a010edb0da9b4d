"""Residues as a caller passes them, 0 .. 2^32 - 1: values that are no residue go
through the kernels' arithmetic, whose sums then pass every bound, so each sum,
difference and negation on their way has to be defined for any operands
(csrc/field_fp.h).  The header itself is compiled for the host and evaluated at
compile time, where a signed overflow is an error."""
import os
import shutil
import subprocess

import pytest

from paper_2502_07060_amd import build as B

CLANG = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")) if c and os.path.exists(c)), None)

STUB = """#pragma once
#include <cstdint>
#define __device__ constexpr
#define __forceinline__ inline
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
"""


def s32(x):
    return (x + 2**31) % 2**32 - 2**31


def s64(x):
    return (x + 2**63) % 2**64 - 2**63


def lit(x):
    return f"({x + 1}LL - 1)"   # INT64_MIN has no literal of its own


@pytest.mark.skipif(CLANG is None, reason="no clang++")
@pytest.mark.parametrize("p", [3, 5, 65537, 998244353, 2147483629, 2147483647])
def test_any_operands(tmp_path, p):
    shutil.copy(os.path.join(B.CSRC, "field_fp.h"), tmp_path / "field_fp.h")
    (tmp_path / "bg_common.h").write_text(STUB)
    h, pinv, c64 = (p - 1) // 2, pow(p, -1, 2**32), 2**64 % p
    c64 -= p if c64 > h else 0
    text = f'#include "field_fp.h"\nconstexpr bg::FpConst F{{{p}, {h}, {pinv}u, {-p}, 0, {c64}}};\n'
    for x in sorted({0, 1, h, h + 1, p - 1, p, p + 1, 2**31 - 1, 2**31, 2**31 + h, 2**32 - 2, 2**32 - 1}):
        want = f" == {x if x <= h else x - p}" if x < p else " != INT64_MIN"
        text += f"static_assert((int64_t)bg::fp_from_canonical({x}u, F){want});\n"
    ends = [-2**31, -2**31 + 1, -p, -h, -1, 0, 1, h, p, 2**31 - 1]
    for a in ends:
        for b in ends:
            for c in (-2**63, -2**62, 0, 2**62, 2**63 - 1):
                text += f"static_assert(bg::mad64({lit(a)}, {lit(b)}, {lit(c)}) == {lit(s64(a * b + c))});\n"
            for name, r in (("add", a + b), ("sub", a - b)):
                r = s32(r) % p
                text += f"static_assert(bg::fp_{name}({lit(a)}, {lit(b)}, F) == {r if r <= h else r - p});\n"
    (tmp_path / "t.cc").write_text(text)
    r = subprocess.run([CLANG, "-std=c++17", "-fsyntax-only", "-w", "t.cc"], cwd=tmp_path, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[:3000]
