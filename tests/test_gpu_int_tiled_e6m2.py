"""GPU: the INT tiled kernel with ufp8-e6m2 inlier scales over many rows of W,
against the fp64 oracle (a decode that branched on the lane left a few rows in
a thousand non-finite), on its own grid and over K ranges."""
import numpy as np
import pytest

import synth
from oracle import sdq as S
from tests.gpu_util import assert_close, say, torch_cuda

import paper_2406_13868_amd as sdq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("qv", [0, 32, 64])
@pytest.mark.parametrize("fmt_o,n_i", [("e4m3", 3), ("int8", 2)])
def test_many_rows_match_oracle(fmt_o, n_i, qv):
    torch = torch_cuda()
    M, N, K = 1024, 4096, 512
    cfg = sdq.Config("int", 1, 8, fmt_o, n_i, 8, "int4", "int8", sfmt_i="ue6m2", qv_i=qv)
    cfg_o = S.Config("int", 1, 8, fmt_o, n_i, 8, "int4", "int8", sfmt_i="ue6m2", qv=qv)
    X, W = synth.make_x(2, M, K), synth.make_w(2, 0, N, K)
    Yref, _, _, _ = S.reference(X, W, cfg_o)
    blob = torch.from_numpy(sdq.pack(W, cfg)).cuda()
    Xq, s_a = sdq.quantize_act(torch.from_numpy(X).cuda(), cfg)
    for path in (sdq.PATH_MFMA, sdq.PATH_SPLITK):
        say("int tiled e6m2", M, N, K, fmt_o, n_i, qv, path)
        nb = sdq.gemm_workspace_size(cfg, M, N, K, path)
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda") if nb else None
        out = torch.full((M, N), float("nan"), device="cuda")
        Y = sdq.gemm(Xq, s_a, blob, N, K, cfg, path=path, workspace=ws, out=out)
        torch.cuda.synchronize()
        assert_close(Y.cpu().numpy(), Yref, f"{fmt_o} {n_i} {qv} path={path}")
