"""GPU parity of the small tiles (32 x 32, 32 x 64, 64 x 64, split K inside the
workgroup) that the automatic path takes for few rows, against the fp64 oracle:
row clusters of up to 16 peers, the plain product of the split path, and plain
products, at the edges of tiles, of K stages and of the row count."""
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

LAYOUT = {"nk": cf.CF_LAYOUT_NK, "kn": cf.CF_LAYOUT_KN}


def _chain(inp, layout, dtype, kind):
    """One subgraph call on the automatic path and the oracle's result."""
    X, W = dev(inp.X, dtype), dev(I.lay_out_weight(inp.W, layout), dtype)
    vec = lambda v: dev(v, "f32")
    out = torch.float32 if dtype == "f32" else torch.bfloat16
    Y = torch.empty((inp.M, inp.N), dtype=out, device="cuda")
    store = dict(kind=cf.CF_N_STORE, out=Y, ld=inp.N, dtype=cf._dt(Y))
    x = O.matmul(inp.X, inp.W)
    if kind == "ln":
        R = dev(inp.R, dtype)
        spec = [dict(kind=cf.CF_N_SCALE, f0=0.5), dict(kind=cf.CF_N_BIAS, v0=vec(inp.bias)),
                dict(kind=cf.CF_N_RESIDUAL, ld=inp.N, dtype=cf._dt(R), **{"in": R}),
                dict(kind=cf.CF_N_LAYERNORM, v0=vec(inp.gamma), v1=vec(inp.beta), f0=1e-5), store]
        ref = O.postnorm(inp.X, inp.W, inp.bias, inp.R, inp.gamma, inp.beta, 0.5, 1e-5)
    elif kind == "rms":
        spec = [dict(kind=cf.CF_N_BIAS, v0=vec(inp.bias)), dict(kind=cf.CF_N_RMSNORM, v0=vec(inp.gamma), f0=1e-5),
                store]
        ref = O.rmsnorm(O.bias_residual(x, inp.bias), inp.gamma, 1e-5)
    else:
        spec = [dict(kind=cf.CF_N_SCALE, f0=8.0), dict(kind=cf.CF_N_SOFTCAP, f0=10.0), dict(kind=cf.CF_N_SOFTMAX),
                store]
        ref = O.softmax_rows(10.0 * np.tanh(8.0 * x / 10.0))
    cf.gemm_subgraph(X, W, spec, w_layout=LAYOUT[layout])
    torch.cuda.synchronize()
    return host(Y), ref


@pytest.mark.parametrize("kind", ["ln", "rms", "msts"])
@pytest.mark.parametrize("layout,dtype", [("nk", "bf16"), ("kn", "bf16"), ("nk", "f32")])
@pytest.mark.parametrize("M,K,N", [
    (1, 512, 512),      # one row
    (33, 1040, 1024),   # one row past a tile, K a quarter stage past whole stages, 16 peers
    (65, 48, 768),      # less than one stage: three waves have no k
    (300, 272, 640),    # 32 x 64 tiles, an odd number of stages per wave
    (1000, 528, 768),   # 64 x 64 tiles (K past whole stages), ragged last row block
    (999, 1040, 1024),  # K past whole stages keeps the 64 x 64 tiles
    (2047, 256, 1024),  # 64 x 128 tiles, one row short of a row block
    (700, 1040, 512),   # 32 x 64 tiles of 8 peers: the deep ring
    (1500, 1040, 512),  # 64 x 64 tiles of 8 peers, the deep ring, ragged last row block
    (600, 784, 768),    # 64 x 64 tiles of 12 peers: the short ring, a quarter stage past whole stages
])
def test_row_clusters(M, K, N, layout, dtype, kind):
    inp = I.postnorm_inputs(M, K, N, dtype, seed=51, bias_std=0.5, gamma="uniform", beta_std=0.3)
    got, ref = _chain(inp, layout, dtype, kind)
    (assert_close_f32 if dtype == "f32" else assert_close_bf16)(got, ref, f"{kind} {M}x{K}x{N} {layout} {dtype}")


@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("M,N", [(40, 1024),    # cluster of 16 peers, two exchanges
                                 (129, 2048),   # cluster of 16 peers
                                 (70, 4128)])   # split path: plain product with a ragged last column tile
def test_quant_chain(M, N, layout):
    inp = I.postnorm_inputs(M, 1040, N, "bf16", seed=52, with_affine=False)
    X, W, R = dev(inp.X), dev(I.lay_out_weight(inp.W, layout)), dev(inp.R)
    Z, s, Q = cf.ln_gelu_amax(X, W, dev(inp.bias, "f32"), R, eps=inp.eps, z_dtype=torch.float32,
                              w_layout=LAYOUT[layout])
    torch.cuda.synchronize()
    z, _, _ = O.ln_gelu_amax(inp.X, inp.W, inp.bias, inp.R, eps=inp.eps)
    assert_close_f32(host(Z), z, f"Z {M}x{N}")
    s32, q32 = O.rowamax_quant_f32(host(Z).astype(np.float32))
    assert np.array_equal(s.cpu().numpy(), s32)
    assert np.array_equal(Q.cpu().numpy(), q32)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("batch,M,K,N", [(1, 17, 2064, 96), (1, 30, 784, 800), (3, 33, 1040, 160), (1, 1, 16, 32),
                                         (1, 515, 528, 1056)])
def test_plain_products(batch, M, K, N, layout, dtype):
    rng = np.random.default_rng(53)
    rnd = lambda *sh: (lambda v: I.round_to_bf16(v) if dtype == "bf16" else v)(rng.standard_normal(sh).astype(np.float32))
    A, B = rnd(batch, M, K), rnd(batch, K, N) / np.float32(np.sqrt(K) if dtype == "f32" else 2.0 ** 5)
    bias = rng.standard_normal(N).astype(np.float32)
    Bd = np.stack([I.lay_out_weight(b, layout) for b in B])
    C = cf.gemm(dev(A, dtype), dev(Bd, dtype), b_layout=LAYOUT[layout], bias=dev(bias, "f32"), alpha=0.5,
                out_dtype=torch.float32)
    torch.cuda.synchronize()
    for b in range(batch):
        assert_close_f32(host(C[b]), 0.5 * O.matmul(A[b], B[b]) + bias, f"{M}x{K}x{N} {layout} {dtype}")


def test_calls_of_all_tiles_share_a_workspace():
    """Row clusters of 32-, 64- and 128-row tiles through one workspace: their records lie differently in a slot's
    area, and each exchange must accept its own round's only."""
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")
    for M, N, path in [(300, 768, 0), (1024, 1024, 2), (1000, 1024, 0), (40, 1024, 0), (2048, 768, 2), (700, 512, 0),
                       (40, 2048, 0), (300, 768, 0)]:
        inp = I.postnorm_inputs(M, 256, N, "bf16", seed=M + N, with_affine=False)
        got = []
        for _ in range(2):
            Y = cf.gemm_postnorm(dev(inp.X), dev(I.lay_out_weight(inp.W, "nk")), dev(inp.bias, "f32"), dev(inp.R),
                                 eps=inp.eps, path=path, ws=ws)
            torch.cuda.synchronize()
            got.append(host(Y))
        assert np.array_equal(got[0], got[1])
        assert_close_bf16(got[0], O.postnorm(inp.X, inp.W, inp.bias, inp.R, None, None, 1.0, inp.eps), f"{M}x{N}")


def test_peer_wait_failure_is_reported():
    """With the sticky word set beforehand every wait gives up at its next poll, and the check reports it."""
    inp = I.postnorm_inputs(200, 256, 768, "bf16", seed=54)
    args = (dev(inp.X), dev(I.lay_out_weight(inp.W, "nk")), dev(inp.bias, "f32"), dev(inp.R), dev(inp.gamma, "f32"),
            dev(inp.beta, "f32"))
    ws = torch.zeros(cf.cf_gemm_postnorm_workspace(cf.postnorm_args(*args, Y=torch.empty_like(args[3]))),
                     dtype=torch.uint8, device="cuda")
    ws.view(torch.int32)[0] = 1
    cf.gemm_postnorm(*args, eps=inp.eps, ws=ws, check=False)
    with pytest.raises(cf.CfError, match="PEER_TIMEOUT"):
        cf.check_workspace(ws)
    Y = cf.gemm_postnorm(*args, eps=inp.eps, ws=ws)
    torch.cuda.synchronize()
    ref = O.postnorm(inp.X, inp.W, inp.bias, inp.R, inp.gamma, inp.beta, 1.0, inp.eps)
    assert_close_bf16(host(Y), ref, "after a reported failure")


@pytest.mark.parametrize("dtype,M,K,N", [("f32", 128, 256, 256), ("bf16", 200, 400, 224), ("f32", 70, 272, 320),
                                         ("bf16", 9000, 768, 768),
                                         ("bf16", 33, 272, 352), ("f32", 33, 272, 352)])   # 32 x 32 tiles, 11 peers
def test_optional_workspace(dtype, M, K, N):
    """Shapes whose workspace is optional: whole rows without one (or with one too small), row clusters with it; the
    helper leaves it out unless check=False."""
    inp = I.postnorm_inputs(M, K, N, dtype, seed=55, bias_std=0.5, gamma="uniform", beta_std=0.3)
    X, W, R = (dev(t, dtype) for t in (inp.X, I.lay_out_weight(inp.W, "nk"), inp.R))
    b, g, be = (dev(t, "f32") for t in (inp.bias, inp.gamma, inp.beta))
    check = assert_close_f32 if dtype == "f32" else assert_close_bf16
    ref = O.postnorm(inp.X, inp.W, inp.bias, inp.R, inp.gamma, inp.beta, 1.0, inp.eps)
    a = cf.postnorm_args(X, W, b, R, g, be, torch.empty_like(R), eps=inp.eps)
    assert cf.cf_gemm_postnorm_workspace(a) == cf.CF_WS_OPTIONAL_BYTES
    ws = torch.zeros(cf.CF_WS_OPTIONAL_BYTES, dtype=torch.uint8, device="cuda")
    for p, n in ((None, 0), (ws.data_ptr(), 4096), (ws.data_ptr() + 8, ws.numel() - 8)):
        Y = torch.empty_like(R)
        a.Y = Y.data_ptr()
        cf._check(cf.cf_gemm_postnorm(a, p, n, torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        assert int(ws.sum()) == 0                      # not touched
        check(host(Y), ref, "whole rows")
    whole = cf.gemm_postnorm(X, W, b, R, g, be, eps=inp.eps, ws=ws)
    assert int(ws.sum()) == 0 and torch.equal(whole, Y)
    for _ in range(2):
        Y = cf.gemm_postnorm(X, W, b, R, g, be, eps=inp.eps, ws=ws, check=False)
        cf.check_workspace(ws)
        check(host(Y), ref, "row clusters")
    assert int(ws.sum()) != 0


@pytest.mark.parametrize("dtype,M,K,N,rows", [
    ("bf16", 16, 1024, 1024, 32), ("bf16", 64, 2048, 2048, 64), ("bf16", 33, 1040, 1024, 32), ("f32", 32, 640, 640, 32),
    ("f32", 100, 512, 768, 32), ("bf16", 5, 272, 1280, 128)])
def test_groups_leave_room_for_another_call(dtype, M, K, N, rows):
    """An XCD has 32 CUs, and a waiting group holds one or, in pairs, half of one per peer: with at most 16 peers two
    (in pairs four) overlapping calls always complete.  The peers are counted by the records that a call on a fresh workspace leaves, `rows` from each."""
    inp = I.postnorm_inputs(M, K, N, dtype, seed=56, with_affine=False)
    ws = torch.zeros(64 << 20, dtype=torch.uint8, device="cuda")
    cf.gemm_postnorm(dev(inp.X, dtype), dev(I.lay_out_weight(inp.W, "nk"), dtype), dev(inp.bias, "f32"),
                     dev(inp.R, dtype), eps=inp.eps, ws=ws, check=False)
    cf.check_workspace(ws)
    words = ws[4096:cf.CF_WS_HEADER_BYTES].view(torch.int64)
    set_words, peer_words = 64 * 17 * 128 * 2, 128 * 2       # one parity of one stage; one peer of a slot
    first = words[set_words:set_words + 16 * peer_words]     # round 1 is odd: second set; without the leader's record
    peers = int(first.count_nonzero()) // 2 / rows
    assert 1 < peers <= 16 and peers == int(peers), peers


@pytest.mark.parametrize("M,K,N,groups", [(1200, 512, 768, 38), (2000, 512, 1024, 32)])
def test_pairs_on_a_cu(M, K, N, groups):
    """Row clusters of 12 and 16 peers whose workgroups fit a CU in pairs: the call runs all its row blocks' groups at
    once, where a CU per workgroup would leave room for 16.  Every group has left its round counter."""
    dtype = "f32"
    inp = I.postnorm_inputs(M, K, N, dtype, seed=58, with_affine=False)
    ws = torch.zeros(cf.CF_WS_HEADER_BYTES, dtype=torch.uint8, device="cuda")
    Y = cf.gemm_postnorm(dev(inp.X, dtype), dev(I.lay_out_weight(inp.W, "nk"), dtype), dev(inp.bias, "f32"),
                         dev(inp.R, dtype), eps=inp.eps, ws=ws)
    ref = O.postnorm(inp.X, inp.W, inp.bias, inp.R, None, None, 1.0, inp.eps)
    assert_close_f32(host(Y), ref, "pairs")
    assert int(ws[256:256 + 64 * 8].view(torch.int64).count_nonzero()) == groups


@pytest.mark.parametrize("count", [2, 4])
def test_streams_of_row_clusters(count):
    """Calls with the largest groups on `count` streams at once, each with a workspace of its own, all on one XCD: all
    of them complete and are right."""
    inp = I.postnorm_inputs(16, 512, 1024, "bf16", seed=57, with_affine=False)
    X, W, b, R = dev(inp.X), dev(I.lay_out_weight(inp.W, "nk")), dev(inp.bias, "f32"), dev(inp.R)
    ref = O.postnorm(inp.X, inp.W, inp.bias, inp.R, None, None, 1.0, inp.eps)
    streams = [torch.cuda.Stream() for _ in range(count)]
    outs = [[torch.empty_like(R) for _ in range(50)] for _ in streams]
    torch.cuda.synchronize()
    for i in range(50):
        for s, out in zip(streams, outs):
            with torch.cuda.stream(s):
                cf.gemm_postnorm(X, W, b, R, eps=inp.eps, out=out[i], check=False)
    torch.cuda.synchronize()
    for s, out in zip(streams, outs):
        cf.check_workspace(cf.workspace(cf.CF_WS_HEADER_BYTES, "cuda", s), s)
        for y in out:
            assert_close_bf16(host(y), ref, "overlapping calls")


@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("dtype,M,K,N", [
    ("bf16", 70, 272, 256),      # 32 x 32 tiles, K past whole stages
    ("bf16", 333, 512, 768),     # 32 x 64
    ("bf16", 999, 1040, 1024),   # 64 x 64
    ("bf16", 1000, 512, 1024),   # 64 x 128 on the ring
    ("bf16", 4097, 512, 2080),   # 256 x 256 tiles and a row pass, ragged
    ("f32", 100, 272, 512),
])
def test_row_clusters_with_pitches_and_special_values(dtype, M, K, N, layout):
    """Row pitches beyond the row for X, W, the residual, the stored rows and the codes; then an infinity or NaN in some
    rows of X: those rows become NaN (LayerNorm), every other keeps its bits."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    t = torch.float32 if dtype == "f32" else torch.bfloat16

    def apart(rows, cols, std=1.0, pad=16):
        store = torch.full((rows, cols + pad), float("nan"), device="cuda", dtype=t)
        store[:, :cols] = (torch.randn((rows, cols), generator=g, device="cuda") * std).to(t)
        return store[:, :cols]
    X, R = apart(M, K), apart(M, N)
    W = apart(*((N, K) if layout == "nk" else (K, N)), std=K ** -0.5)
    b = torch.randn(N, generator=g, device="cuda")
    Z = torch.full((M, N + 8), 7.0, device="cuda")
    s, Q = torch.zeros(M, device="cuda"), torch.full((M, N + 16), 7, device="cuda", dtype=torch.uint8)
    spec = [dict(kind=cf.CF_N_BIAS, v0=b), dict(kind=cf.CF_N_RESIDUAL, ld=N + 16, dtype=cf._dt(R), **{"in": R}),
            dict(kind=cf.CF_N_LAYERNORM, f0=1e-5), dict(kind=cf.CF_N_GELU),
            dict(kind=cf.CF_N_STORE, out=Z, ld=N + 8, dtype=cf.CF_F32),
            dict(kind=cf.CF_N_ROWAMAX_QUANT, out=s, out2=Q, ld=N + 16, f0=448.0)]
    ws = torch.zeros(128 << 20, dtype=torch.uint8, device="cuda")

    def run():
        cf.gemm_subgraph(X, W, spec, w_layout=LAYOUT[layout], ws=ws, check=False)
        cf.check_workspace(ws)
        assert bool((Z[:, N:] == 7.0).all()) and bool((Q[:, N:] == 7).all())
        return Z[:, :N].clone(), s.clone(), Q[:, :N].clone()
    z, sc, q = run()
    x = X.double() @ (W.double().t().contiguous() if layout == "nk" else W.double()) + b.double() + R.double()
    x = x - x.mean(1, keepdim=True)
    x = x / torch.sqrt(x.square().mean(1, keepdim=True) + 1e-5)
    ref = 0.5 * x * (1.0 + torch.erf(x / 2 ** 0.5))
    assert float((z.double() - ref).abs().max()) < 1e-4
    s32, q32 = O.rowamax_quant_f32(z.cpu().numpy())
    assert np.array_equal(sc.cpu().numpy(), s32) and np.array_equal(q.cpu().numpy(), q32)
    rows = [0, M // 2, M - 1]
    for m, k, v in zip(rows, (K - 1, 0, 5), (float("inf"), float("nan"), float("-inf"))):
        X[m, k] = v
    z2, sc2, q2 = run()
    keep = torch.ones(M, dtype=torch.bool, device="cuda")
    keep[rows] = False
    assert bool(torch.isnan(z2[~keep]).all())
    assert torch.equal(z2[keep], z[keep]) and torch.equal(sc2[keep], sc[keep]) and torch.equal(q2[keep], q[keep])
