"""The GELU of the GEMM epilogues: its polynomial, read from the source and evaluated in fp32, against the closed form in
fp64; and that it hides no NaN."""
import os
import re
from dataclasses import replace

import numpy as np
import pytest
from scipy.special import erfc

from paper_2603_12118_amd import workloads as wl

HEADER = os.path.join(os.path.dirname(wl.__file__), "csrc", "common.h")


def test_polynomial():
    body = re.search(r"float gelu_erf\(float z\) \{(.*?)\n\}", open(HEADER).read(), re.S).group(1)
    f32 = np.float32
    top = f32(re.search(r"fabsf\(z\), ([0-9.]+)f\)", body).group(1))
    first = re.search(r"float p = (\S+)f;", body).group(1)
    coeff = [f32(c) for c in [first] + re.findall(r"fmaf\(p, x, (\S+)f\);", body)]
    assert len(coeff) == 9 and coeff[-1] == -1
    fma = lambda a, b, c: (np.float64(a) * np.float64(b) + np.float64(c)).astype(f32)   # (a product of two fp32 values is exact in fp64)
    z = np.concatenate([np.linspace(-12, 12, 200_001), np.random.default_rng(0).standard_normal(100_000)]).astype(f32)
    x = np.minimum(np.abs(z), top)
    p = np.full_like(x, coeff[0])
    for c in coeff[1:]:
        p = fma(p, x, c)
    y = fma(-x, np.exp2(p.astype(np.float64)).astype(f32), np.maximum(z, f32(0))).astype(np.float64)
    z = z.astype(np.float64)
    ref = z * 0.5 * erfc(-z / np.sqrt(2))
    err = np.abs(y - ref)
    # half an ulp of a result of 8 - 12 is 4.8e-7 and of 4 - 8 2.4e-7 (y is a multiple of its ulp); the rest is the
    # polynomial's: x h(x) <= 0.17 times ln 2 times 1e-6, and its last additions in fp32, 2^-24 |log2 h|
    assert err[np.abs(z) < 8].max() < 2.4e-7 + 1.5e-7 and err.max() < 4.8e-7 + 1e-8
    assert np.sqrt((err[200_001:] ** 2).mean()) < 3.5e-8
    assert err[z < -6].max() < 6.5 * 4.1e-11 + 6.1e-9   # 6 h(6) is 5.9e-9
    for lo, hi, rel in [(0, 1, 6e-7), (1, 2, 1.2e-6), (2, 3, 1e-5), (3, 4, 1.5e-4), (4, 5, 1e-3), (5, 6, 3e-3)]:
        m = (z < -lo) & (z >= -hi)
        assert (err[m] <= rel * np.abs(ref[m])).all(), (lo, hi, (err[m] / np.abs(ref[m])).max())


@pytest.mark.gpu
def test_nan_stays_in_its_clip_and_stays_nan():
    import torch

    from paper_2603_12118_amd import binding as B
    from tests.test_gpu_batch_sizes import dev_bf16

    w = wl.audio_workload("nan", replace(wl.audio_config(1), hidden=320, n_heads=5, mlp_dim=1280, out_hidden=256), 2, 400, seq_len=512, data_seed=1)
    enc = B.Encoder(w.cfg, w.weights)
    clean, _ = enc.cs_encode(dev_bf16(w.patches), w.cu_seqlens, w.grid_thw)
    mel = dev_bf16(w.patches)
    mel[100] = float("nan")
    out, _ = enc.cs_encode(mel, w.cu_seqlens, w.grid_thw)
    torch.cuda.synchronize()
    assert torch.isfinite(clean).all()
    assert torch.isnan(out[:100]).all() and torch.equal(out[100:], clean[100:])
