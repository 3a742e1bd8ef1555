"""LayerNorm of rows whose mean is thousands of spreads: the variance must come from the distances to the mean.  (As the
difference of two sums it keeps the digits that the mean leaves it: at this ratio of 4000, fp32 sums of squares of 4e6 are
off by more than the variance of 0.25.)"""
import numpy as np
import pytest

import workloads as wl
from harness import LockStep, gpu_context

pytestmark = pytest.mark.gpu

OFFSET = 2000.0


# decoder blocks and sources of one row tile (LayerNorm inside the GEMM and inside the cross-attention); of more rows, with a LayerNorm
# kernel that finds the rows whole or as K slices; every width of the kernels with a constant K; fp32 in one workgroup, launch by launch beyond d = 256
@pytest.mark.parametrize("d,F,k,B,S,dtype", [(128, 512, 4, 1, 5, "bf16"), (256, 1024, 5, 3, 7, "bf16"), (512, 2048, 8, 2, 9, "bf16"), (512, 2048, 10, 33, 12, "bf16"), (768, 3072, 11, 4, 10, "bf16"),
                                             (1024, 4096, 10, 1, 3, "bf16"), (1024, 4096, 16, 4, 11, "bf16"), (256, 512, 9, 70, 3, "bf16"), (64, 256, 4, 2, 17, "f32"), (96, 384, 4, 1, 5, "f32")])
def test_rows_far_from_zero(d, F, k, B, S, dtype):
    cfg = wl.Config("far", 90, 1, 1, d, d // (64 if dtype == "bf16" else 16), F, 272, k, B, S, 2 * k + 4, dtype, 2, src_len_kind="lognormal")
    weights = wl.make_weights(cfg)
    for name in ("pos_src", "pos_tgt"):                    # (kept in fp32: not rounded to bf16 like the matrices)
        weights[name] = (weights[name] + OFFSET).astype(np.float32)
    ctx = gpu_context(cfg, weights)
    src, n = wl.make_sources(cfg)
    ls = LockStep(cfg, weights, ctx, src, n, np.full(B, cfg.max_out, np.int32), sample=sorted({0, B // 2, B - 1}))
    if dtype == "f32":                                     # the rows themselves are rounded to 2^-13 here, 2.5e-4 of their spread
        ls.tol = 2e-3
    for _ in range(2):
        ls.step(imposed=np.full(B, k, np.int32))
    print(f"d {d} rows {B * k}: worst logit error {ls.max_logit_err:.2e}")
