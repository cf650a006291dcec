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


@pytest.mark.parametrize("M", [33, 49, 65, 97, 128])
@pytest.mark.parametrize("out16", [False, True])
def test_shares_whose_fragments_are_finished_several_at_a_time(B, M, out16):
    """Shares of six, seven and eight tiles, whose fragments are odd and even in number for a wavefront of eight or
    of four.  fp32 results: as above; fp16: each rounded once, by 2^-11 of itself at most, as is
    then the 2-norm of the errors."""
    say("several fragments", M, out16)
    for N, K in [(24010, 96), (28001, 96), (32000, 96)]:
        g = torch.Generator(device="cuda").manual_seed(N + M)
        x = torch.randn((M, K), generator=g, device="cuda").to(torch.float16)
        W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.float16)
        ws = B.workspace(B.lib().ghd_linear_workspace_bytes(M, N, K))
        ws.fill_(0xFF)
        y = torch.full((M, N), float("nan"), dtype=torch.float16 if out16 else torch.float32, device="cuda")
        B.ghd_linear_skinny(x, B.ghd_pack_weight(W), N, ws=ws, y=y)
        ref = x.double() @ W.double().t()
        err = float((y.double() - ref).norm() / ref.norm())
        assert err < (2.0 ** -11 if out16 else max(2e-7, 4 * 2.0 ** -24 * K ** 0.5)), (N, K, err)


@pytest.mark.parametrize("M", [17, 32, 33, 49, 64, 65, 81, 128])
def test_row_groups_add_products_to_sets_of_sums(B, M):
    """Matrices of few tiles, which are dealt out in groups of rows: k ranges of no step, a step or two and of ragged
    lengths for a wavefront, whose products go to sets of sums in turn.  Tolerance as above."""
    say("row groups' sums", M)
    used, out = 0, (ctypes.c_int * 2)()
    for N, K in [(5, 8), (300, 40), (1280, 264), (100, 1000), (572, 2856), (1280, 1280), (2048, 2048), (80, 3960)]:
        B.lib().ghd_debug_groups(M, N, K, 256, 1, out)
        used += out[1] > 1
        g = torch.Generator(device="cuda").manual_seed(N + M)
        x = torch.randn((M, K), generator=g, device="cuda").to(torch.float16)
        W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.float16)
        ws = B.workspace(B.lib().ghd_linear_workspace_bytes(M, N, K))
        ws.fill_(0xFF)
        y = B.ghd_linear_skinny(x, B.ghd_pack_weight(W), N, ws=ws)
        assert B.ghd_step_status(ws) == 0
        ref = x.double() @ W.double().t()
        err = float((y.double() - ref).norm() / ref.norm())
        assert err < max(2e-7, 4 * 2.0 ** -24 * K ** 0.5), (N, K, err)
    assert used


def test_every_stream_gives_the_same_result(B):
    """The XCD that a dispatch begins with depends on the hardware queue it goes through.
    Several streams in turn (more than there are queues), each with a small launch of its own in
    between: the same layer, attention and split linear give the same bits and status 0 on all."""
    from paper_2505_23219_amd import model, workloads as wl
    say("streams")
    s = wl.ModelShape("streams", H=1024, nh=8, d=128, F=2752, V=500, L=1)
    M, kv = 40, 300
    w = model.upload_layer(wl.layer_weights(s, 3, 0), s.d)
    kc, vc = model.upload_cache(*wl.kv_cache(s, 384, kv, 3, 0))
    x0 = wl.activations(M, s.H, 3).float().cuda()
    parent = torch.from_numpy(wl.tree_random(M, 5, 3)).cuda()
    W = B.ghd_pack_weight(wl.activations(1000, 4096, 4, tag="w", std=0.02).cuda())
    xl = wl.activations(33, 4096, 5).cuda()
    cfg = B.make_cfg(s, 384)
    torch.cuda.synchronize()
    want = None
    for i in range(8):
        with torch.cuda.stream(torch.cuda.Stream() if i else torch.cuda.default_stream()):
            torch.zeros(64 * i + 1, device="cuda").add_(1)
            ws, lws = B.workspace(B.ghd_workspace_bytes(cfg, M, kv)), B.workspace(B.lib().ghd_linear_workspace_bytes(33, 1000, 4096))
            x = x0.clone()
            B.ghd_verify_layer(cfg, w, kc, vc, x, parent, kv, ws=ws)
            y = B.ghd_linear_skinny(xl, W, 1000, ws=lws)
            assert (B.ghd_step_status(ws), B.ghd_step_status(lws)) == (0, 0), i
            torch.cuda.synchronize()
            want = want or (x, y)
            assert torch.equal(x, want[0]) and torch.equal(y, want[1]), i


@pytest.mark.parametrize("M,N,K", [(16, 4096, 4096), (32, 1024, 1024), (64, 512, 512), (33, 200, 1000), (1, 64, 64)])
def test_linear_in_place(B, M, N, K):
    """y == x with an fp16 result: x counts as it was before the call.  fp16 rounding of an fp32
    sum: half an ulp (2^-11 of the value) plus the sum's own error, below 2e-6 of the row's scale."""
    say("linear in place", M, N, K)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.float16)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.float16)
    ref = x.double() @ W.double().t()
    y = x[:, :N]
    ws = B.workspace(B.lib().ghd_linear_workspace_bytes(M, N, K))
    B.ghd_linear_skinny(x, B.ghd_pack_weight(W), N, ws=ws, y=y)
    assert B.ghd_step_status(ws) == 0
    err = (y.double() - ref).abs()
    assert bool((err <= 2.0 ** -11 * ref.abs() + 2e-6 * ref.std() + 2.0 ** -25).all()), float(err.max())


@pytest.mark.parametrize("M", [16, 40])
def test_every_stream_gives_the_same_stack(B, M):
    """The same over three layers that share a QKV + attention launch each: every counter line is
    used again and again, the XCDs meet between the two halves of the launch, and a head's cached
    rows are split over several workgroups on both ways through the attention."""
    from paper_2505_23219_amd import model, workloads as wl
    say("streams, stack", M)
    s = wl.ModelShape("streams", H=4096, nh=32, d=128, F=1376, V=500, L=3)
    kv = 700
    layer = model.upload_layer(wl.layer_weights(s, 3, 0), s.d)
    caches = [model.upload_cache(*wl.kv_cache(s, 768, kv, 3, l)) for l in range(s.L)]
    stack = model.build_stack(s, 768, [layer] * s.L, caches, model.upload_head(wl.head_weights(s, 3)))
    x16 = wl.activations(M, s.H, 3).cuda()
    parent = torch.from_numpy(wl.tree_random(M, 5, 3)).cuda()
    torch.cuda.synchronize()
    want = None
    for i in range(8):
        with torch.cuda.stream(torch.cuda.Stream() if i else torch.cuda.default_stream()):
            torch.zeros(64 * i + 1, device="cuda").add_(1)
            ws = B.workspace(B.ghd_workspace_bytes(stack.cfg, M, kv))
            logits = B.ghd_verify_stack(stack, x16, parent, kv, ws=ws)
            assert B.ghd_step_status(ws) == 0, i
            torch.cuda.synchronize()
            want = logits if want is None else want
            assert torch.equal(logits, want) and bool(torch.isfinite(logits).all()), i


@pytest.mark.parametrize("M,N,K", [(1, 2048, 13824), (8, 2048, 5888), (16, 2048, 5888), (33, 9000, 5888), (64, 9000, 4096),
                                   (80, 22016, 11008), (96, 32000, 4096), (100, 9000, 11008), (128, 22016, 4096),
                                   (128, 27648, 2560), (128, 32000, 4096), (128, 5003, 13824)])
def test_linear_sums_are_not_left_in_long_chains(B, M, N, K):
    """The relative error (2-norm) of the fp32 sums, however a matrix is cut.  A chain of c MFMAs of 32
    columns leaves a squared error of about 5.5e-15 + 1.4e-15 c (measured over 1 to 60 of them, the
    sums over wavefronts and parts included); c is what an even deal of the matrix over 256 compute
    units of eight wavefronts makes it, of whole tiles for 640 tiles or more, else of the k-steps of
    four-tile blocks.  10% more for the spread between inputs and shapes."""
    say("linear sums", M, N, K)
    nks, tiles = (K + 31) // 32, (N + 15) // 16
    chain = nks / 8 if tiles >= 640 else nks / 8 * ((tiles + 3) // 4) / 256
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.float16)
    Wp, W64 = B.ghd_pack_weight(W), W.double().t()
    num = den = 0.0
    for _ in range(1 + 20000 // (M * N)):
        x = torch.randn((M, K), generator=g, device="cuda").to(torch.float16)
        ref = x.double() @ W64
        num += float(((B.ghd_linear_skinny(x, Wp, N).double() - ref) ** 2).sum())
        den += float((ref ** 2).sum())
    err = (num / den) ** 0.5
    assert err < 1.1 * (5.5e-15 + 1.4e-15 * chain) ** 0.5, err


@pytest.mark.parametrize("M", [1, 40, 64, 96, 128])
@pytest.mark.parametrize("steps", [1, 3, 7, 8, 9, 15, 16, 17, 31, 33, 50])
def test_wavefronts_take_the_k_steps_in_turn(B, M, steps):
    """k-steps of 32 columns that leave wavefronts with none, or with one more than others: in turns of eight and of
    four wavefronts, with and without the barrier that keeps them together, the last k-step whole and ragged.
    Bound as in test_linear_kernels_at_their_edges."""
    say("k-steps in turn", M, steps)
    for N, K in [(300, 32 * steps), (9000, 32 * steps - 24), (23000, 32 * steps - 8)]:
        g = torch.Generator(device="cuda").manual_seed(N + K + M)
        x = torch.randn((M, K), generator=g, device="cuda").to(torch.float16)
        W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.float16)
        ws = B.workspace(B.lib().ghd_linear_workspace_bytes(M, N, K))
        ws.fill_(0xFF)
        y = B.ghd_linear_skinny(x, B.ghd_pack_weight(W), N, ws=ws)
        assert B.ghd_step_status(ws) == 0
        ref = x.double() @ W.double().t()
        err = float((y.double() - ref).norm() / ref.norm())
        assert err < max(2e-7, 4 * 2.0 ** -24 * K ** 0.5), (N, K, err)


@pytest.mark.parametrize("M", [1, 9, 16, 17, 33, 40, 64])
@pytest.mark.parametrize("steps", [55, 56, 63, 64, 65, 71, 72, 73, 80, 81, 88, 89, 95, 96, 97, 127])
def test_four_k_steps_in_a_turn(B, M, steps):
    """Whole tiles of narrow matrices, around the line from which wavefronts take four k-steps in their turn: what whole
    rounds leave over is nothing, one run to eight of one, two, three and four, the last k-step whole and ragged; x read as it
    lies, and packed (y meets x).  Bounds as in test_linear_kernels_at_their_edges and test_linear_in_place."""
    say("four k-steps in a turn", M, steps)
    for K in (32 * steps, 32 * steps - 8):
        N = 200
        assert B.lib().ghd_debug_run(M, N, K, 256, 1) == (4 if steps >= 56 else 1)
        g = torch.Generator(device="cuda").manual_seed(K + M)
        x = torch.randn((M, K), generator=g, device="cuda").to(torch.float16)
        W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.float16)
        Wp, ref = B.ghd_pack_weight(W), x.double() @ W.double().t()
        ws = B.workspace(B.lib().ghd_linear_workspace_bytes(M, N, K))
        ws.fill_(0xFF)
        y = B.ghd_linear_skinny(x, Wp, N, ws=ws)
        assert B.ghd_step_status(ws) == 0
        err = float((y.double() - ref).norm() / ref.norm())
        assert err < max(2e-7, 4 * 2.0 ** -24 * K ** 0.5), (K, err)
        y = x[:, :N]
        B.ghd_linear_skinny(x, Wp, N, ws=ws, y=y)
        err = (y.double() - ref).abs()
        assert bool((err <= 2.0 ** -11 * ref.abs() + 2e-6 * ref.std() + 2.0 ** -25).all()), (K, float(err.max()))


@pytest.mark.parametrize("M,N,K,whole", [(1, 2560, 6904, 0), (16, 1536, 4096, 0), (5, 2048, 5504, 0), (24, 5120, 5120, 0),
                                         (16, 5120, 5120, 1), (32, 4608, 4608, 0), (1, 4096, 4096, 1), (16, 1536, 1536, 1)])
def test_narrow_matrices_inside_a_step(B, M, N, K, whole):
    """Narrow matrices as a step's launches cut them (a call whose result meets its input is cut so too): in
    parts or whole tiles on either side of the line.  Bound as in test_linear_in_place."""
    say("narrow, inside a step", M, N, K)
    out = (ctypes.c_int * 5)()
    B.lib().ghd_debug_cut(M, N, K, 256, 0, out)
    assert out[0] == whole
    g = torch.Generator(device="cuda").manual_seed(M + N)
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.float16)
    W = (torch.randn((N, K), generator=g, device="cuda") * 0.02).to(torch.float16)
    ref = x.double() @ W.double().t()
    y = x[:, :N]
    ws = B.workspace(B.lib().ghd_linear_workspace_bytes(M, N, K))
    B.ghd_linear_skinny(x, B.ghd_pack_weight(W), N, ws=ws, y=y)
    assert B.ghd_step_status(ws) == 0
    err = (y.double() - ref).abs()
    assert bool((err <= 2.0 ** -11 * ref.abs() + 2e-6 * ref.std() + 2.0 ** -25).all()), float(err.max())


@pytest.mark.parametrize("M", [1, 8, 70])
@pytest.mark.parametrize("shift", [0, 1])
def test_residual_stream_where_the_caller_wants_it(B, M, shift):
    """The final residual stream in a buffer of its own, in one whose storage is x_in's (at its start, or its middle), and not
    asked for: the same logits and the same x, bit for bit."""
    from paper_2505_23219_amd import model, workloads as wl
    say("x_out", M, shift)
    s = wl.ModelShape("x_out", H=256, nh=4, d=64, F=688, V=1000, L=2)
    kv = 100
    caches = [model.upload_cache(*wl.kv_cache(s, 192, kv, 5, l)) for l in range(s.L)]
    stack = model.build_stack(s, 192, [model.upload_layer(wl.layer_weights(s, 5, l), s.d) for l in range(s.L)], caches,
                              model.upload_head(wl.head_weights(s, 5)))
    x16 = wl.activations(M, s.H, 5).cuda()
    parent = torch.from_numpy(wl.tree_random(M, 5, 5)).cuda()
    ws = B.workspace(B.ghd_workspace_bytes(stack.cfg, M, kv))
    x_out = torch.full((M, s.H), float("nan"), dtype=torch.float32, device="cuda")
    logits = B.ghd_verify_stack(stack, x16, parent, kv, x_out=x_out, ws=ws)
    shared = torch.empty((M, s.H), dtype=torch.float32, device="cuda")
    x_in = shared.view(-1).view(torch.float16)[shift * M * s.H:][:M * s.H].view(M, s.H)
    x_in.copy_(x16)
    both = B.ghd_verify_stack(stack, x_in, parent, kv, x_out=shared, ws=ws)
    neither = B.ghd_verify_stack(stack, x16, parent, kv, ws=ws)
    assert bool(torch.isfinite(logits).all()) and torch.equal(both, logits) and torch.equal(neither, logits)
    assert torch.equal(shared, x_out)
    assert B.ghd_step_status(ws) == 0


@pytest.mark.parametrize("M", [1, 70, 128])
@pytest.mark.parametrize("where", ["parent", "parent_last", "workspace", "host", "pinned"])
def test_residual_stream_where_it_is_copied(B, M, where):
    """The final residual stream over parent[] (at its start, its last word), over the unused end of the workspace buffer,
    and in host memory: the same logits, x and argmaxes as in a buffer of its own, bit for bit."""
    from paper_2505_23219_amd import model, workloads as wl
    say("x_out copied", M, where)
    s = wl.ModelShape("x_out", H=256, nh=4, d=64, F=688, V=1000, L=2)
    kv = 100
    caches = [model.upload_cache(*wl.kv_cache(s, 256, kv, 5, l)) for l in range(s.L)]
    stack = model.build_stack(s, 256, [model.upload_layer(wl.layer_weights(s, 5, l), s.d) for l in range(s.L)], caches,
                              model.upload_head(wl.head_weights(s, 5)))
    x16 = wl.activations(M, s.H, 5).cuda()
    tree = torch.from_numpy(wl.tree_random(M, 5, 5)).cuda()
    need = B.ghd_workspace_bytes(stack.cfg, M, kv)
    ws = B.workspace(need)
    want = torch.full((M, s.H), float("nan"), dtype=torch.float32, device="cuda")
    logits = B.ghd_verify_stack(stack, x16, tree, kv, x_out=want, ws=ws)
    amax = B.ghd_verify_stack_argmax(stack, x16, tree, kv, ws=ws)
    for argmax in (False, True):
        parent, buf = tree, torch.full((M * s.H,), float("nan"), dtype=torch.float32, device="cuda")
        if where.startswith("parent"):
            parent = buf.view(torch.int32)[:M] if where == "parent" else buf.view(torch.int32)[M * s.H - M:]
            parent.copy_(tree)
        elif where == "workspace":
            at = (need + 255) // 256 * 256
            ws = B.workspace(at + 4 * M * s.H)
            buf = ws[at:at + 4 * M * s.H].view(torch.float32)
        else:
            buf = torch.full((M * s.H,), float("nan"), dtype=torch.float32, pin_memory=where == "pinned")
        x_out = buf.view(M, s.H)
        if argmax:
            assert torch.equal(B.ghd_verify_stack_argmax(stack, x16, parent, kv, x_out=x_out, ws=ws), amax)
        else:
            assert torch.equal(B.ghd_verify_stack(stack, x16, parent, kv, x_out=x_out, ws=ws), logits)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(want).all()) and torch.equal(x_out.cuda(), want)
        assert B.ghd_step_status(ws) == 0
