"""Acceptance and commit at their edges, against plain torch on the host (exact)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import B, say, _capture_manager  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,V,shift", [(1, 1, 0), (2, 7, 1), (5, 8, 3), (64, 8191, 2), (128, 1003, 1), (3, 64001, 0)])
def test_row_argmax_from_any_4_byte_boundary(B, M, V, shift):
    """Rows that start and end at any 4 bytes, shorter and longer than the segments' 16-byte
    pieces, with ties (few distinct values), -inf and NaN (never chosen)."""
    say("argmax", M, V, shift)
    g = torch.Generator().manual_seed(M + V)
    lg = torch.randint(-3, 4, (M, V), generator=g).float()
    lg[:, ::5] = float("-inf")
    if V > 8:
        lg[:, 3] = float("nan")
    dev = torch.full((M * V + shift + 4,), 9.0, device="cuda")[shift:shift + M * V].view(M, V)
    dev.copy_(lg)
    want = np.nanargmax(lg.numpy(), axis=1)          # the first of equal ones
    parent = torch.tensor([-1] + [0] * (M - 1), dtype=torch.int32).cuda()
    tokens = torch.full((M,), -5, dtype=torch.int32).cuda()
    res, amax = B.ghd_accept_greedy(dev, tokens, parent)
    assert np.array_equal(amax.cpu().numpy(), want)
    assert res.cpu().tolist()[:3] == [1, int(want[0]), 0]


@pytest.mark.parametrize("M,step,bad", [(128, 1, None), (128, 1, 77), (128, 2, None), (100, 3, 50), (65, 64, None), (1, 1, None)])
def test_accepted_path_of_deep_trees(B, M, step, bad):
    """A path through every step-th node, valid down to node `bad` (none: all of it); the nodes
    between hang off the root with wrong tokens."""
    say("path", M, step, bad)
    path = list(range(0, M, step))
    parent, amax = [-1] + [0] * (M - 1), [1000 + i for i in range(M)]
    tokens = [-1] * M
    for a, b in zip(path, path[1:]):
        parent[b], tokens[b] = a, (-7 if b == bad else amax[a])
    n = path.index(bad) if bad in path else len(path)
    i32 = lambda v: torch.tensor(v, dtype=torch.int32).cuda()
    res = B.ghd_accept_path(i32(amax), i32(tokens), i32(parent)).cpu().tolist()
    assert res[0] == n and res[1] == amax[path[n - 1]] and res[2:2 + n] == path[:n]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("path", [[0], [0, 1, 2], [0, 2], [0, 1, 5, 9], list(range(0, 34, 2)), list(range(0, 36, 2)),
                                  [0, 1, 2] + list(range(5, 128, 2)), list(range(128))])
def test_commit_moves_exactly_the_path(B, d, path):
    """Paths that are in place, that move up to and past what fits the registers, and all 128."""
    from paper_2505_23219_amd.workloads import ModelShape
    say("commit", d, len(path))
    L, nh, M, kv, cap = 2, 3, 128, 37, 168
    k = torch.randn(L, nh, cap, d).half()
    v = torch.randn(L, nh, d, cap).half()
    want_k, want_v = k.clone(), v.clone()
    at = torch.tensor(path) + kv
    want_k[:, :, kv:kv + len(path)] = k[:, :, at]
    want_v[:, :, :, kv:kv + len(path)] = v[:, :, :, at]
    kd, vd = k.cuda(), v.cuda()
    g = torch.ones(8, dtype=torch.float16, device="cuda")
    none = {n: g for n in ("g_attn", "Wqkv", "Wo", "g_ffn", "Wgu", "Wdown")}
    shape = ModelShape("c", H=nh * d, nh=nh, d=d, F=8, V=16, L=L)
    stack = B.Stack(B.make_cfg(shape, cap), [none] * L, [(kd[l], vd[l]) for l in range(L)], {"g_final": g, "Wlm": g})
    res = torch.tensor([len(path), 4] + path + [0] * (M - len(path)), dtype=torch.int32).cuda()
    B.ghd_commit_path(stack, res, M, kv)
    assert torch.equal(kd.cpu(), want_k) and torch.equal(vd.cpu(), want_v)


@pytest.mark.parametrize("path", [[0], [0, 3, 4, 9]])
def test_commit_reads_no_more_of_the_result_than_the_path(B, path):
    """A result that ends with its path, in an allocation of just that size."""
    from paper_2505_23219_amd.workloads import ModelShape
    say("commit, short result", len(path))
    L, nh, d, M, kv, cap = 2, 2, 64, 128, 5, 136
    k, v = torch.randn(L, nh, cap, d).half(), torch.randn(L, nh, d, cap).half()
    want_k, want_v = k.clone(), v.clone()
    at = torch.tensor(path) + kv
    want_k[:, :, kv:kv + len(path)] = k[:, :, at]
    want_v[:, :, :, kv:kv + len(path)] = v[:, :, :, at]
    kd, vd = k.cuda(), v.cuda()
    g = torch.ones(8, dtype=torch.float16, device="cuda")
    none = {n: g for n in ("g_attn", "Wqkv", "Wo", "g_ffn", "Wgu", "Wdown")}
    shape = ModelShape("c", H=nh * d, nh=nh, d=d, F=8, V=16, L=L)
    stack = B.Stack(B.make_cfg(shape, cap), [none] * L, [(kd[l], vd[l]) for l in range(L)], {"g_final": g, "Wlm": g})
    res = torch.tensor([len(path), 4] + path, dtype=torch.int32).cuda()
    B.ghd_commit_path(stack, res, M, kv)
    assert torch.equal(kd.cpu(), want_k) and torch.equal(vd.cpu(), want_v)
