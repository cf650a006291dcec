"""The skinny linear kernels over all their instantiations, against torch in 64 bits."""
import ctypes

import pytest
import torch

from test_gpu_parity import B, say, _capture_manager  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 128])
def test_linear_kernels_at_their_edges(B, M):
    """Every number of row tiles of x, at its first and last row, over cuts of every kind: few
    tiles and many per workgroup (a ragged last one), whole tiles and parts, one k-step and
    many, k ranges that leave wavefronts without work, columns that fill no k-step.  fp32 sums
    of K exact products: relative error of the 2-norm below 4 eps sqrt(K) (eps = 2^-24; chains
    of independent roundings), and no less than 2e-7."""
    say("linear edges", M)
    out = (ctypes.c_int * 5)()
    kinds = set()
    for N, K in [(5, 8), (64, 40), (300, 3416), (1280, 1280), (2600, 688), (5003, 4104), (9000, 264), (12300, 520),
                 (20000, 96), (33000, 64)]:
        g = torch.Generator(device="cuda").manual_seed(N + K + M)
        x = torch.randn((M, K + 8), generator=g, device="cuda").to(torch.float16)[:, :K]
        W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.float16)
        ws = B.workspace(B.lib().ghd_linear_workspace_bytes(M, N, K))
        ws.fill_(0xFF)                                  # NaN wherever something unwritten is read
        y = B.ghd_linear_skinny(x, B.ghd_pack_weight(W), N, ws=ws)
        assert B.ghd_step_status(ws) == 0
        ref = x.double() @ W.double().t()
        err = float((y.double() - ref).norm() / ref.norm())
        assert err < max(2e-7, 4 * 2.0 ** -24 * K ** 0.5), (N, K, err)
        B.lib().ghd_debug_cut(M, N, K, 256, 1, out)
        kinds.add((out[0], out[1], out[4]))
    assert len(kinds) >= 5, kinds
