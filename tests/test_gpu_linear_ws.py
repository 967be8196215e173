"""GPU: sdq.linear (one library call, with or without a workspace) equals
quantize_act followed by gemm bit for bit on every path sdq_linear_ws can
take, and refuses a workspace that does not serve."""
import copy
import pickle

import numpy as np
import pytest

import synth
from tests.gpu_util import say, torch_cuda

import paper_2406_13868_amd as sdq

pytestmark = pytest.mark.gpu
INT, MX = sdq.Config.int_family(), sdq.Config.mx_family()


@pytest.mark.parametrize("cfg,M,N,K", [(INT, 1, 256, 512), (INT, 16, 256, 512), (INT, 64, 8192, 256),
                                       (INT, 33, 96, 8192), (INT, 16, 96, 8704), (INT, 20, 96, 8192), (MX, 1, 96, 256), (MX, 5, 96, 1024),
                                       (MX, 48, 96, 8192), (MX, 600, 10240, 256)])
def test_linear_equals_quantize_then_gemm(cfg, M, N, K):
    torch = torch_cuda()
    say("linear ws", cfg.label, M, N, K)
    X = torch.from_numpy(synth.make_x(2, M, K)).cuda()
    blob = torch.from_numpy(sdq.pack(synth.make_w(2, 0, N, K), cfg)).cuda()
    Xq, s_a = sdq.quantize_act(X, cfg)
    Y = sdq.gemm(Xq, s_a, blob, N, K, cfg)
    nb = sdq.gemm_workspace_size(cfg, M, N, K)
    for ws in (None, torch.empty(max(nb, 16), dtype=torch.uint8, device="cuda")):
        Y2, Xq2, s2 = sdq.linear(X, blob, N, K, cfg, workspace=ws)
        assert torch.equal(Xq, Xq2) and torch.equal(s_a, s2)
        fused = nb == 0 and sdq.gemm_path(cfg, M, N, K) == sdq.PATH_DECODE
        assert torch.equal(Y, Y2), "fused" if fused else "two calls"
    if nb:
        with pytest.raises(ValueError, match="workspace holds"):
            sdq.linear(X, blob, N, K, cfg, workspace=torch.empty(nb - 16, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("call", ["linear", "gemm"])
def test_a_calls_own_workspace_outlives_another_stream(call, monkeypatch):
    """A workspace that the call allocates is not given out again while the
    stream that the call was sent to may still use it."""
    torch = torch_cuda()
    M, N, K = 33, 96, 8192
    X = torch.from_numpy(synth.make_x(2, M, K)).cuda()
    blob = torch.from_numpy(sdq.pack(synth.make_w(2, 0, N, K), INT)).cuda()
    Xq, s_a = sdq.quantize_act(X, INT)
    nb = sdq.gemm_workspace_size(INT, M, N, K)
    want = sdq.gemm(Xq, s_a, blob, N, K, INT)
    out = torch.empty_like(want)
    q2, s2 = torch.empty_like(Xq), torch.empty_like(s_a)
    side, taken, empty = torch.cuda.Stream(), [], torch.empty
    torch.cuda.synchronize()

    def record(*a, **k):
        t = empty(*a, **k)
        taken.append((t.data_ptr(), t.nbytes))
        return t

    say("own workspace on a side stream", call)
    with torch.cuda.stream(side):
        torch.cuda._sleep(100_000_000)  # cycles; the call's kernels wait behind it
    monkeypatch.setattr(torch, "empty", record)
    if call == "linear":
        sdq.linear(X, blob, N, K, INT, out=out, xq=q2, scales=s2, stream=side)
    else:
        sdq.gemm(Xq, s_a, blob, N, K, INT, out=out, stream=side)
    monkeypatch.undo()
    (ptr, size), = taken
    assert size == nb and nb > 0
    other = torch.empty(nb, dtype=torch.uint8, device="cuda")
    assert not side.query(), "the side stream should still be asleep"
    assert other.data_ptr() != ptr
    torch.cuda.synchronize()
    assert torch.equal(out, want)


def test_a_used_config_copies_and_pickles():
    cfg = sdq.Config.int_family()
    assert sdq.pack_size(cfg, 64, 256) == sdq.pack_size(cfg, 64, 256)
    for other in (copy.deepcopy(cfg), pickle.loads(pickle.dumps(cfg))):
        assert other == cfg and hash(other) == hash(cfg) and sdq.pack_size(other, 64, 256) == sdq.pack_size(cfg, 64, 256)
    assert np.array_equal(sdq.pack(synth.make_w(2, 0, 64, 256), other), sdq.pack(synth.make_w(2, 0, 64, 256), cfg))
