"""mbq_linear_static (the entry point that allocates nothing: its workspace is a buffer inside the library image)
against mbq_linear on the same inputs, through the C ABI: two calls in a row, the second with a smaller input, and the
refusal of shapes whose workspace does not fit."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from helpers import assert_output_close, dev_bf16
from workloads import make_router, make_tokens, make_weight

pytestmark = pytest.mark.gpu


def _case(mbq, N, K, T, seed):
    W = make_weight(N, K, [seed], 4.0)
    Wr, br = make_router(K, [seed], mix=None)
    xb, _ = make_tokens(T, K, [seed, T], outlier_channel_frac=0.01)
    X = dev_bf16(xb)
    blob = mbq.mbq_encode(torch.from_numpy(W).cuda())
    prec, perm, offsets = mbq.mbq_route(X, torch.from_numpy(Wr).cuda(), torch.from_numpy(br).cuda())
    return W, xb, X, blob, prec, perm, offsets


@pytest.mark.parametrize("shapes", [((272, 4096, 16), (130, 1280, 5)),      # one-token-tile decode kernels
                                    ((96, 2048, 48), (40, 512, 33)),        # 17..64 tokens
                                    ((300, 1024, 200), (64, 512, 130)),     # the same kernel above 64 tokens
                                    ((2064, 4096, 150), (40, 512, 530))])   # tiled GEMM
def test_static_scratch_matches_workspace_call(mbq, shapes):
    for call, (N, K, T) in enumerate(shapes):          # the second call is the smaller one
        W, xb, X, blob, prec, perm, offsets = _case(mbq, N, K, T, 300 + call)
        assert mbq.load().mbq_linear_workspace_bytes(T, N, K) <= mbq.load().mbq_static_scratch_bytes()
        Y_ws = mbq.mbq_linear(X, blob, N, K, prec, perm, offsets)
        Y_st = torch.full((T, N), float("nan"), dtype=torch.float32, device="cuda")
        mbq.mbq_linear_static(X, blob, N, K, prec, perm, offsets, Y_st)
        torch.cuda.synchronize()
        codes, s0, z0 = O.encode(W)
        Yref = O.linear(xb, codes, s0, z0, prec.cpu().numpy())
        assert_output_close(Y_st.cpu().numpy(), Yref, f"static scratch, call {call}, N={N} K={K} T={T}")
        assert_output_close(Y_ws.cpu().numpy(), Yref, f"caller workspace, call {call}, N={N} K={K} T={T}")
        assert torch.equal(Y_st, Y_ws)  # the same kernels on the same inputs


def test_static_scratch_refuses_what_does_not_fit(mbq):
    lib = mbq.load()
    N, K, T = 256, 8192, 4096
    assert lib.mbq_linear_workspace_bytes(T, N, K) > lib.mbq_static_scratch_bytes()
    dummy = torch.zeros(256, dtype=torch.uint8, device="cuda")
    st = lib.mbq_linear_static(dummy.data_ptr(), T, dummy.data_ptr(), N, K, dummy.data_ptr(), dummy.data_ptr(),
                               dummy.data_ptr(), dummy.data_ptr(), 0, None)
    assert st == 3                                             # MBQ_ERR_WORKSPACE, nothing enqueued
    assert b"scratch" in lib.mbq_last_error()
    assert lib.mbq_linear_static(None, 0, None, 16, 128, None, None, None, None, 0, None) == 0   # T = 0: no-op
