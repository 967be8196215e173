"""GPU: the MX family's kernel for few tokens (16 rows of W per workgroup, K
split over its waves) at the sizes where it can go wrong, against the fp64
oracle: one token, full and ragged token tiles, ragged rows (half a tile with no
row in use), one chunk of K, fewer and more chunks than are in flight, a partial
chunk, blocks whose inliers do not merge, no outliers, both output types and an
output that is only 4-byte aligned."""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import sdq as S
from tests.gpu_util import assert_close_terms, kernel_of, say, torch_cuda

import paper_2406_13868_amd as sdq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(1, 33, 128), (9, 48, 96), (16, 4100, 4096), (17, 15, 2176), (32, 130, 4768),
                                   (33, 96, 1024), (64, 2048, 256), (50, 100, 8160), (50, 1640, 9344), (5, 64, 5120),
                                   (65, 72, 1184), (130, 512, 640)])
@pytest.mark.parametrize("n_o,n_i,split", [(1, 2, False), (1, 3, True), (0, 3, False), (1, 1, False)])
def test_few_tokens_match_oracle(M, N, K, n_o, n_i, split):
    torch = torch_cuda()
    cfg = sdq.Config("mx", n_o, 8, "e4m3", n_i, 8, "e2m1", "e4m3")
    cfg_o = S.Config("mx", n_o, 8, "e4m3", n_i, 8, "e2m1", "e4m3")
    assert kernel_of(cfg, M, N, K, sdq.PATH_SPLITK) == "mx_small"
    X, W = synth.make_x(2, M, K), synth.make_w(2, 0, N, K)
    if split:  # a few blocks whose outliers are far above their inliers
        W[::3, 0:8 * (K // 8):40] = 60000.0
    L = S.pack_logical(W, cfg_o)
    if split:
        d = L["scale_i"].astype(int) - L["scale_o"].astype(int)
        assert np.any((d < -5) | (d > 6))
    say("mx small", M, N, K, n_o, n_i, split)
    blob = torch.from_numpy(sdq.pack(W, cfg)).cuda()
    Xq, s_a = sdq.quantize_act(torch.from_numpy(X).cuda(), cfg)
    nb = sdq.gemm_workspace_size(cfg, M, N, K, sdq.PATH_SPLITK)
    ws = torch.full((nb,), 0x5A, dtype=torch.uint8, device="cuda")
    Y = sdq.gemm(Xq, s_a, blob, N, K, cfg, path=sdq.PATH_SPLITK, workspace=ws)
    buf = torch.full((M * N + 2,), 7.0, device="cuda")
    Y1 = sdq.gemm(Xq, s_a, blob, N, K, cfg, path=sdq.PATH_SPLITK, workspace=ws, out=buf[1:1 + M * N].view(M, N))
    Yb = sdq.gemm(Xq, s_a, blob, N, K, dataclasses.replace(cfg, y_dtype="bf16"), path=sdq.PATH_SPLITK, workspace=ws)
    torch.cuda.synchronize()
    Yref, Xr, s_r, _ = S.reference(X, W, cfg_o)
    A = np.abs(S.dequant_act(Xr, s_r, cfg_o))
    T = A @ (np.abs(S.dequant_outliers(L)) + np.abs(S.dequant_inliers(L))).T
    assert_close_terms(Y.cpu().numpy(), Yref, T, K, f"M={M} N={N} K={K}")
    assert torch.equal(Y, Y1) and float(buf[0]) == 7.0 and float(buf[-1]) == 7.0
    assert torch.equal(Yb, Y.to(torch.bfloat16))
