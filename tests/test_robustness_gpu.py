"""GPU tests of the failure handling and the batched row operator.

The row-cluster path waits for co-resident peer workgroups with a bounded
spin and reports a wait that gave up through a sticky error word in the
workspace.  The failure is forced from the host (the word is set before the
call), so every wait gives up at its first poll and every kernel exits
normally; the call must then be reported, and a clean call afterwards must
be correct.
"""
import numpy as np
import pytest

from oracle import comfuse_oracle as O
from paper_2608_03537_amd import inputs as I
from tests.helpers import assert_close_bf16, assert_close_f32, dev, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_03537_amd import comfuse as cf  # noqa: E402


def _postnorm_operands(inp):
    X, W, R = dev(inp.X), dev(I.lay_out_weight(inp.W, "nk")), dev(inp.R)
    b, g, be = dev(inp.bias, "f32"), dev(inp.gamma, "f32"), dev(inp.beta, "f32")
    return X, W, b, R, g, be


def test_peer_wait_failure_is_reported_then_cleared():
    inp = I.postnorm_inputs(512, 128, 768, "bf16", seed=41)
    X, W, b, R, g, be = _postnorm_operands(inp)
    Y = torch.empty((inp.M, inp.N), dtype=torch.bfloat16, device="cuda")
    need = cf.cf_gemm_postnorm_workspace(cf.postnorm_args(X, W, b, R, g, be, Y, path=cf.PATH_CLUSTER))
    assert need > 0
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    ws.view(torch.int32)[0] = 1            # as if an earlier wait had given up
    cf.gemm_postnorm(X, W, b, R, g, be, eps=inp.eps, path=cf.PATH_CLUSTER, out=Y, ws=ws, check=False)
    with pytest.raises(cf.CfError, match="PEER_TIMEOUT"):
        cf.check_workspace(ws)
    assert int(ws.view(torch.int32)[0].item()) == 0   # the check cleared the word
    cf.check_workspace(ws)                             # nothing new: no error
    # a clean call through the same workspace is checked and correct
    cf.gemm_postnorm(X, W, b, R, g, be, eps=inp.eps, path=cf.PATH_CLUSTER, out=Y, ws=ws)
    torch.cuda.synchronize()
    ref = O.postnorm(inp.X, inp.W, inp.bias, inp.R, inp.gamma, inp.beta, 1.0, inp.eps)
    assert_close_bf16(host(Y), ref, "cluster after a reported failure")


def test_helper_raises_on_failure():
    inp = I.postnorm_inputs(256, 128, 512, "bf16", seed=42, with_affine=False)
    X, W, b, R, _, _ = _postnorm_operands(inp)
    Z = torch.empty((inp.M, inp.N), dtype=torch.bfloat16, device="cuda")
    spec = [dict(kind=cf.CF_N_BIAS, v0=b), dict(kind=cf.CF_N_RESIDUAL, **{"in": R}, ld=inp.N, dtype=cf.CF_BF16),
            dict(kind=cf.CF_N_LAYERNORM, f0=inp.eps), dict(kind=cf.CF_N_STORE, out=Z, ld=inp.N, dtype=cf.CF_BF16)]
    need = cf.cf_gemm_subgraph_workspace(cf.subgraph_args(X, W, cf.make_nodes(spec), path=cf.PATH_CLUSTER))
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    ws.view(torch.int32)[0] = 1
    with pytest.raises(cf.CfError, match="PEER_TIMEOUT"):
        cf.gemm_subgraph(X, W, spec, path=cf.PATH_CLUSTER, ws=ws)   # check=True by default
    cf.gemm_subgraph(X, W, spec, path=cf.PATH_CLUSTER, ws=ws)
    torch.cuda.synchronize()
    ref = O.layernorm(O.bias_residual(O.matmul(inp.X, inp.W), inp.bias, inp.R), eps=inp.eps)
    assert_close_bf16(host(Z), ref, "subgraph after a reported failure")


def test_workspace_cache_is_per_stream():
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    a = cf.workspace(4096, "cuda", s1)
    b = cf.workspace(4096, "cuda", s2)
    assert a.data_ptr() != b.data_ptr()
    assert cf.workspace(4096, "cuda", s1).data_ptr() == a.data_ptr()


def test_rowop_batched_strided():
    # three 100 x 256 matrices inside a [3, 120, 256] buffer (batch stride
    # 120 rows): bias, LayerNorm, store of the 300 rows one after another
    rng = np.random.default_rng(43)
    full = rng.standard_normal((3, 120, 256)).astype(np.float32) * 2 + 0.5
    P = dev(full, "f32")[:, :100]
    b = rng.standard_normal(256).astype(np.float32) * 0.1
    Y = torch.empty((300, 256), dtype=torch.float32, device="cuda")
    cf.rowop(P, [dict(kind=cf.CF_N_BIAS, v0=dev(b, "f32")), dict(kind=cf.CF_N_LAYERNORM, f0=1e-5),
                 dict(kind=cf.CF_N_STORE, out=Y, ld=256, dtype=cf.CF_F32)])
    torch.cuda.synchronize()
    rows = full[:, :100].reshape(300, 256).astype(np.float64)
    assert_close_f32(host(Y), O.layernorm(O.bias_residual(rows, b), eps=1e-5), "batched rowop")


def test_rowop_batched_softmax_matches_flat():
    rng = np.random.default_rng(44)
    S = dev(rng.standard_normal((4, 64, 512)).astype(np.float32) * 3, "f32")
    A = torch.empty((256, 512), dtype=torch.float32, device="cuda")
    B = torch.empty((256, 512), dtype=torch.float32, device="cuda")
    cf.rowop(S, [dict(kind=cf.CF_N_SOFTMAX, out=A, ld=512, dtype=cf.CF_F32, f0=0.5)])
    cf.rowop(S.reshape(256, 512), [dict(kind=cf.CF_N_SOFTMAX, out=B, ld=512, dtype=cf.CF_F32, f0=0.5)])
    torch.cuda.synchronize()
    assert torch.equal(A, B)
    assert_close_f32(host(A), O.softmax_rows(0.5 * host(S).reshape(256, 512)), "batched softmax")


def test_cluster_calls_of_different_widths_share_a_workspace():
    # Row-cluster calls with 4, 8 and 16 peers per row block and one to three
    # rounds per peer group, all through one fresh workspace: each call's
    # exchange must only ever accept its own round's records, whatever earlier
    # calls of another width left in the header.
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")
    for M, N in [(2048, 1024), (4096, 2048), (1024, 4096), (6144, 1024), (2048, 2048), (3072, 1024)]:
        inp = I.postnorm_inputs(M, 64, N, "f32", seed=45 + N // 1024, with_residual=False)
        X, W = dev(inp.X, "f32"), dev(I.lay_out_weight(inp.W, "nk"), "f32")
        b, g, be = dev(inp.bias, "f32"), dev(inp.gamma, "f32"), dev(inp.beta, "f32")
        Y = torch.empty((M, N), dtype=torch.float32, device="cuda")
        spec = [dict(kind=cf.CF_N_BIAS, v0=b), dict(kind=cf.CF_N_LAYERNORM, v0=g, v1=be, f0=1e-5),
                dict(kind=cf.CF_N_STORE, out=Y, ld=N, dtype=cf.CF_F32)]
        cf.gemm_subgraph(X, W, spec, path=cf.PATH_CLUSTER, ws=ws)
        torch.cuda.synchronize()
        ref = O.postnorm(inp.X, inp.W, inp.bias, None, inp.gamma, inp.beta, 1.0, 1e-5)
        assert_close_f32(host(Y), ref, f"cluster {M}x{N} after other widths")


def _captured(fn, stream):
    """fn captured on `stream` (after two calls there that warm it up), and the graph's replay."""
    with torch.cuda.stream(stream):
        for _ in range(2):
            fn()
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        fn()
    return g


def _spoil_cached_workspaces():
    """Fills every workspace that the helpers keep and checks later that nothing else wrote to it."""
    torch.cuda.synchronize()
    kept = list(cf._ws_cache.values())
    cf._ws_cache.clear()
    for ws in kept:
        ws.fill_(0x5A)
    return kept


def test_captured_attention_keeps_no_cached_workspace():
    """Keys split over workgroups need a workspace, which eager calls take from the helper's cache.  A graph outlives
    what the cache holds (a larger call replaces it), so it must not refer to it: replays with the cached workspaces
    overwritten are right and leave them as they are; a workspace of the caller's own is used."""
    g = torch.Generator(device="cuda").manual_seed(8)
    Q, K, V = (torch.randn((2, 8, n, 128), generator=g, device="cuda").bfloat16() for n in (1, 3000, 3000))
    out = torch.empty_like(Q)
    ref = cf.b2b_attention(Q, K, V)
    stream = torch.cuda.Stream()
    graph = _captured(lambda: cf.b2b_attention(Q, K, V, out=out), stream)
    kept = _spoil_cached_workspaces()
    for _ in range(4):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert float((out.float() - ref.float()).norm() / ref.float().norm()) < 5e-3
        assert torch.equal(cf.b2b_attention(Q, K, V), ref)       # eager work between the replays
    assert kept and all(bool((ws == 0x5A).all()) for ws in kept)
    ws = torch.zeros(8 << 20, dtype=torch.uint8, device="cuda")
    own = _captured(lambda: cf.b2b_attention(Q, K, V, out=out, ws=ws), stream)
    for _ in range(3):
        out.zero_()
        own.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
    assert int(ws[:cf.CF_B2B_WS_HEADER_BYTES].sum()) == 0 and int(ws.count_nonzero()) > 0


def test_captured_narrow_row_call_keeps_no_cached_workspace():
    """The same for row calls whose workspace is optional (check=False lets eager calls take it)."""
    inp = I.postnorm_inputs(200, 400, 224, "bf16", seed=43)
    args = _postnorm_operands(inp)
    Y = torch.empty_like(args[3])
    call = lambda **kw: cf.gemm_postnorm(*args, eps=inp.eps, out=Y, check=False, **kw)
    ref = O.postnorm(inp.X, inp.W, inp.bias, inp.R, inp.gamma, inp.beta, 1.0, inp.eps)
    stream = torch.cuda.Stream()
    graph = _captured(call, stream)
    kept = _spoil_cached_workspaces()
    for _ in range(4):
        Y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert_close_bf16(host(Y), ref, "replay")
        call()
        cf.check_workspace(cf.workspace(cf.CF_WS_OPTIONAL_BYTES, "cuda"))
        assert_close_bf16(host(Y), ref, "eager between replays")
    assert kept and all(bool((ws == 0x5A).all()) for ws in kept)
    ws = torch.zeros(cf.CF_WS_OPTIONAL_BYTES, dtype=torch.uint8, device="cuda")
    own = _captured(lambda: call(ws=ws), stream)
    before = int(ws.count_nonzero())
    for _ in range(3):
        Y.zero_()
        own.replay()
        cf.check_workspace(ws)
        assert_close_bf16(host(Y), ref, "the caller's workspace")
    assert before > 0


def _check_replays(graph, call, Y, check, kept=()):
    """Replays of `graph` against the expected result, with eager work and fresh allocations between them."""
    for i in range(4):
        Y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        check(f"replay {i}")
        Y.zero_()
        call()
        torch.cuda.synchronize()
        check(f"eager call after replay {i}")
        torch.full((64 << 20,), 0x5A, dtype=torch.uint8, device="cuda")
    assert all(bool((ws == 0x5A).all()) for ws in kept)


@pytest.mark.parametrize("warm", [False, True])
def test_captured_cluster_calls_own_their_workspace(warm):
    """Row clusters captured into a graph without a workspace of the caller's own, with and without eager calls on
    the stream before (a cold capture must not leave eager calls a buffer that only the graph's replay would zero):
    replays are right with the helper's cached workspaces overwritten, eager calls before the first replay and between
    replays too, and so is a second graph that is replayed first."""
    inp = I.postnorm_inputs(300, 256, 768, "bf16", seed=44)
    args = _postnorm_operands(inp)
    Y = torch.empty_like(args[3])
    call = lambda: cf.gemm_postnorm(*args, eps=inp.eps, out=Y, check=False)
    ref = O.postnorm(inp.X, inp.W, inp.bias, inp.R, inp.gamma, inp.beta, 1.0, inp.eps)
    check = lambda what: assert_close_bf16(host(Y), ref, what)
    stream = torch.cuda.Stream()
    if warm:
        with torch.cuda.stream(stream):
            call()
        stream.synchronize()
    graphs = []
    for _ in range(2):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            call()
            call()
        graphs.append(g)
        # one buffer for both calls of the capture
        capture, ws = cf._ws_graph[str(Y.device), stream.cuda_stream, "rows"]
        assert capture is not None and ws.numel() == cf.CF_WS_HEADER_BYTES
    kept = _spoil_cached_workspaces()
    with torch.cuda.stream(stream):
        Y.zero_()
        call()
        cf.check_workspace(cf.workspace(cf.CF_WS_HEADER_BYTES, "cuda"))
    check("eager call before the first replay")
    _check_replays(graphs[1], call, Y, check)
    _check_replays(graphs[0], call, Y, check, kept)


def test_captured_split_mlp_owns_its_workspace():
    """The same for the split MLP, whose arrival counters must be zero."""
    inp = I.dlrm_mlp_inputs(M=4200, K=1088)
    X, W1, W2 = dev(inp.X), dev(np.ascontiguousarray(inp.W1.T)), dev(np.ascontiguousarray(inp.W2.T))
    b1, b2 = dev(inp.b1, "f32"), dev(inp.b2, "f32")
    Y = torch.empty((inp.M, 128), dtype=torch.bfloat16, device="cuda")
    call = lambda: cf.b2b_mlp(X, W1, b1, W2, b2, out=Y)
    ref = O.mlp_b2b(inp.X, inp.W1, inp.b1, inp.W2, inp.b2)
    graph = _captured(call, torch.cuda.Stream())
    kept = _spoil_cached_workspaces()
    assert kept
    _check_replays(graph, call, Y, lambda what: assert_close_bf16(host(Y), ref, what), kept)
