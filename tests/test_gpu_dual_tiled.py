"""GPU: the dual family's tiled kernel at the sizes where it can go wrong, for
each of its workgroup shapes, against the fp64 oracle.

The launcher picks the shape by grid: 32 tokens x 128 outputs (two K groups
per workgroup), 64 x 128, 64 x 256 and 128 x 256 (and leaves few tokens on
short rows to the split-K form).  For each: ragged tokens
and outputs, one chunk of K, an odd number of chunks, more chunks than the
buffers of the staging loop hold, K that is not a whole chunk (with rows of
scales that are not whole dwords), one and two outlier planes, fp32 and bf16 outputs, an output that is not 16-byte aligned.  The
tolerance is that of test_gpu_dual (fp32 sums of exact products; a bf16
output adds its half ulp).
"""
import numpy as np
import pytest

import synth
from oracle import sdq as S
from tests.gpu_util import dual_term_tol, kernel_of, rel_errors, say, torch_cuda

import paper_2406_13868_amd as sdq

pytestmark = pytest.mark.gpu

SHAPES = [  # M, N, K, form
    (9, 8225, 160, "splitk"), (16, 8224, 32, "splitk"), (32, 8200, 416, "splitk"),  # (few tokens on short rows)
    (33, 8225, 160, "32x128"), (34, 8224, 32, "32x128"), (64, 8200, 416, "32x128"), (33, 8193, 128, "32x128"),
    (25, 8225, 544, "32x128"), (40, 8200, 1152, "32x128"),
    (130, 8196, 96, "64x128"), (321, 4129, 288, "64x128"), (384, 4096, 640, "64x128"), (1100, 8193, 96, "64x128"),
    (2049, 4100, 416, "64x128"), (321, 4129, 128, "64x128"), (321, 4129, 1152, "64x128"),
    (700, 4100, 256, "64x256"), (700, 4100, 96, "64x256"), (700, 4100, 288, "64x256"), (700, 4100, 416, "64x256"),
    (700, 4100, 128, "64x256"), (700, 4100, 1152, "64x256"),
    (513, 8225, 160, "128x256"), (513, 8225, 96, "128x256"), (513, 8225, 128, "128x256"), (513, 8225, 416, "128x256"),
    (513, 8225, 1152, "128x256"),
]


def kernel_name(form):
    return "dual_splitk" if form == "splitk" else f"dual_tiled {form}"


@pytest.mark.parametrize("n_o,n_i", [(1, 6), (2, 4)])
@pytest.mark.parametrize("y_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K,form", SHAPES)
def test_tiled_shapes_match_oracle(M, N, K, form, n_o, n_i, y_dtype):
    torch = torch_cuda()
    cfg = sdq.Config("dual", n_o, 8, "int8", n_i, 8, "e2m1", "int8", y_dtype=y_dtype)
    assert kernel_of(cfg, M, N, K) == kernel_name(form)
    cfg_o = S.Config("dual", n_o, 8, "int8", n_i, 8, "e2m1", "int8+e2m1")
    X, W = synth.make_x(2, M, K), synth.make_w(2, 0, N, K)
    X[M // 2] = 0.0  # an all-zero token
    say("dual tiled", M, N, K, n_o, y_dtype)
    blob = torch.from_numpy(sdq.pack(W, cfg)).cuda()
    q = sdq.quantize_act_dual(torch.from_numpy(X).cuda(), cfg)
    # an output one element into its allocation: 4-byte (bf16: 4 of 8) aligned only
    buf = torch.full((M * N + 4,), 7.0, dtype=cfg.y_torch_dtype(), device="cuda")
    skip = 1 if y_dtype == "f32" else 2
    outs = [sdq.gemm_dual(*q, blob, N, K, cfg),
            sdq.gemm_dual(*q, blob, N, K, cfg, out=buf[skip:skip + M * N].view(M, N))]
    torch.cuda.synchronize()
    Yref, (Ao, Ai), (s_ao, Ea), L = S.reference(X, W, cfg_o)
    A_o, A_i = S.dequant_act_dual(Ao, s_ao, Ai, Ea)
    T = np.abs(A_o) @ np.abs(S.dequant_outliers(L)).T + np.abs(A_i) @ np.abs(S.dequant_inliers(L)).T
    for Y in outs:
        Yn = Y.float().cpu().numpy().astype(np.float64)
        tol = dual_term_tol(K) * T + (np.abs(Yref) * 2.0 ** -8 if y_dtype == "bf16" else 0.0)
        bad = np.abs(Yn - Yref) > tol + 1e-30
        assert not bad.any(), f"{bad.sum()} outputs off, first at {np.argwhere(bad)[0]}, {rel_errors(Yn, Yref)}"
    assert torch.equal(outs[0], outs[1])
    # nothing is written outside the output
    assert (buf[:skip] == 7.0).all() and (buf[skip + M * N:] == 7.0).all()


NAN_SHAPES = [  # M, N, K, kernel
    (16, 256, 160, "dual_splitk"),
    (32, 8200, 160, "dual_splitk"), (32, 8200, 384, "dual_splitk"),
    (40, 8200, 160, "dual_tiled 32x128"), (40, 8200, 384, "dual_tiled 32x128"),  # (384: an odd number of chunks)
    (32, 8200, 1152, "dual_tiled 32x128"), (32, 8200, 1408, "dual_tiled 32x128"), (40, 8200, 1184, "dual_tiled 32x128"),
    (321, 4129, 160, "dual_tiled 64x128"), (700, 4100, 160, "dual_tiled 64x256"), (513, 8225, 160, "dual_tiled 128x256"),
    (321, 4129, 672, "dual_tiled 64x128"), (700, 4100, 672, "dual_tiled 64x256"), (513, 8225, 1184, "dual_tiled 128x256"),
]


@pytest.mark.parametrize("n_o,n_i", [(1, 6), (2, 4)])
@pytest.mark.parametrize("M,N,K,kernel", NAN_SHAPES)
def test_a_nan_activation_scale_stays_in_its_token(M, N, K, kernel, n_o, n_i):
    """The e8m0 NaN (0xFF, which a caller's own scales may hold) in the first
    block of a token follows the last blocks of the token before it: with K no
    whole number of chunks, or a second K group's chunk past K, that token's
    scale reads reach it, and it must not reach the token's outputs."""
    torch = torch_cuda()
    cfg = sdq.Config("dual", n_o, 8, "int8", n_i, 8, "e2m1", "int8")
    assert kernel_of(cfg, M, N, K) == kernel
    blob = torch.from_numpy(sdq.pack(synth.make_w(2, 0, N, K), cfg)).cuda()
    Xo, s_a, Xi, Ea = sdq.quantize_act_dual(torch.from_numpy(synth.make_x(2, M, K)).cuda(), cfg)
    say("dual nan scale", M, N, K, n_o)
    clean = sdq.gemm_dual(Xo, s_a, Xi, Ea, blob, N, K, cfg)
    nan = torch.zeros(M, dtype=torch.bool, device="cuda")
    nan[1::5] = True
    bad = Ea.clone()
    bad[nan, 0] = 0xFF
    Y = sdq.gemm_dual(Xo, s_a, Xi, bad, blob, N, K, cfg)
    torch.cuda.synchronize()
    assert torch.isnan(Y[nan]).all()
    assert torch.equal(Y[~nan], clean[~nan]), f"{int((Y[~nan] != clean[~nan]).any(1).sum())} other tokens changed"
