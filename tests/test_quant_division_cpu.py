"""The compression kernel divides by a product with the reciprocal and two FMA corrections; that equals the IEEE division for
every finite fp16 value and every scale that an fp16 channel can have (a dense sample of them), and so do the codes."""
import ctypes
import os
import re
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

C = r"""
#include <math.h>
static float divide_by(float x, float lam, float inv)
{
    float q = x * inv;
    q = fmaf(fmaf(-q, lam, x), inv, q);
    return fmaf(fmaf(-q, lam, x), inv, q);
}
long long differences(const float *x, int n, const float *lam, int m)
{
    long long bad = 0;
    for (int j = 0; j < m; ++j) {
        const float inv = 1.0f / lam[j];
        for (int i = 0; i < n; ++i)
            if (divide_by(x[i], lam[j], inv) != x[i] / lam[j]) ++bad;
    }
    return bad;
}
"""


def test_reciprocal_division_rounds_correctly(tmp_path):
    # the three lines above are the kernel's
    src = open(os.path.join(ROOT, "paper_2403_17312_amd", "csrc", "swa_quant.hip")).read()
    body = re.search(r"float divide_by\(.*?\n\{(.*?)\n\}", src, flags=re.S).group(1)
    assert re.sub(r"\s+", "", body.replace("__builtin_fmaf", "fmaf")) in re.sub(r"\s+", "", C)
    (tmp_path / "d.c").write_text(C)
    lib = str(tmp_path / "d.so")
    # -ffp-contract=off: the multiplication stays one
    subprocess.check_call(["gcc", "-O2", "-ffp-contract=off", "-shared", "-fPIC", "-o", lib, str(tmp_path / "d.c"), "-lm"])
    x = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16).view(np.float16)
    x = np.ascontiguousarray(x[np.isfinite(x)].astype(np.float32))
    rng = np.random.default_rng(1)
    ends = rng.choice(x, (2, 400))
    spread = np.concatenate([np.abs(ends[0] - ends[1]), 2.0 ** np.arange(-7.0, 17.0), np.exp(rng.uniform(np.log(2.0 ** -7), np.log(131008.0), 300)),
                             np.float32([2.0 ** -7, 131008.0])]).astype(np.float32)
    lam = np.ascontiguousarray(np.maximum(spread, np.float32(2.0 ** -7)) / np.float32(255.0))
    L = ctypes.CDLL(lib)
    L.differences.restype = ctypes.c_longlong
    fp = ctypes.POINTER(ctypes.c_float)
    assert L.differences(x.ctypes.data_as(fp), len(x), lam.ctypes.data_as(fp), len(lam)) == 0
