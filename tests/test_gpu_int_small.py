"""GPU: the INT family's kernel for few tokens (16 rows of W and 16 or 32 tokens
per workgroup) at the sizes where it can go wrong, against the fp64 oracle:
one token past the decode kernel's, full and ragged token tiles, several
token blocks, ragged rows (half a tile with no row in use), one chunk of K, fewer chunks
than waves, a partial chunk, every scale format and outlier type, both output
types and an output that is only 4-byte aligned."""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import sdq as S
from tests.gpu_util import say, torch_cuda

import paper_2406_13868_amd as sdq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(9, 33, 128), (16, 48, 96), (16, 4100, 1152), (17, 15, 2176), (32, 130, 320),
                                   (33, 96, 1024), (64, 2048, 256), (24, 12288, 160)])
@pytest.mark.parametrize("fmt_o,sfmt_i,qv,n_i", [("e4m3", "", 0, 3), ("int8", "", 32, 2), ("e4m3", "e4m3", 16, 3),
                                                  ("int8", "ue6m2", 32, 1), ("e4m3", "e4m3", 64, 2), ("int8", "", 64, 3)])
def test_few_tokens_match_oracle(M, N, K, fmt_o, sfmt_i, qv, n_i):
    if qv == 64 and K % 64:
        K += 32
    torch = torch_cuda()
    cfg = sdq.Config("int", 1, 8, fmt_o, n_i, 8, "int4", "int8", sfmt_i=sfmt_i, qv_i=qv)
    cfg_o = S.Config("int", 1, 8, fmt_o, n_i, 8, "int4", "int8", sfmt_i=sfmt_i, qv=qv)
    X, W = synth.make_x(2, M, K), synth.make_w(2, 0, N, K)
    say("int small", M, N, K, fmt_o, sfmt_i, qv)
    blob = torch.from_numpy(sdq.pack(W, cfg)).cuda()
    Xq, s_a = sdq.quantize_act(torch.from_numpy(X).cuda(), cfg)
    Y = sdq.gemm(Xq, s_a, blob, N, K, cfg, path=sdq.PATH_MFMA)
    buf = torch.full((M * N + 2,), 7.0, device="cuda")
    Y1 = sdq.gemm(Xq, s_a, blob, N, K, cfg, path=sdq.PATH_MFMA, out=buf[1:1 + M * N].view(M, N))
    Yb = sdq.gemm(Xq, s_a, blob, N, K, dataclasses.replace(cfg, y_dtype="bf16"), path=sdq.PATH_MFMA)
    torch.cuda.synchronize()
    Yref, Xr, s_r, L = S.reference(X, W, cfg_o)
    A = Xr.view(np.int8).astype(np.float64) * s_r[:, None]
    T = np.abs(A) @ (np.abs(S.dequant_outliers(L)) + np.abs(S.dequant_inliers(L))).T
    # exact products; each output's fp32 sums round at most about once per 8
    # products of a wave, and a few times at the end, each by 2^-24 of sum |terms|
    err = np.abs(Y.cpu().numpy().astype(np.float64) - Yref)
    assert (err <= (K / 8 + 16) * 2.0 ** -24 * T + 1e-30).all(), f"worst {np.max(err / np.maximum(T, 1e-30)):.2e} of sum |terms|"
    assert torch.equal(Y, Y1) and float(buf[0]) == 7.0 and float(buf[-1]) == 7.0
    assert torch.equal(Yb, Y.to(torch.bfloat16))
