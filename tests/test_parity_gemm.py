"""GPU parity of the unfused comparator pieces: cf_gemm (batched, both B
layouts, fp32/bf16) and cf_rowop softmax, against the fp64 oracle."""
import numpy as np
import pytest

from oracle import comfuse_oracle as O
from paper_2608_03537_amd import inputs as I
from tests.helpers import assert_close_bf16, assert_close_f32, dev, host, rel_rms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_03537_amd import comfuse as cf  # noqa: E402


def _rand(shape, seed, dtype, std=1.0):
    v = (np.random.default_rng(seed).standard_normal(shape) * std).astype(np.float32)
    return I.round_to_bf16(v) if dtype == "bf16" else v


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("M,K,N", [(100, 64, 96), (257, 160, 320), (64, 32, 512)])
def test_gemm(M, K, N, layout, dtype):
    A = _rand((M, K), 1, dtype)
    Bm = _rand((K, N), 2, dtype, 1 / np.sqrt(K))
    bias = _rand((N,), 3, "f32")
    Cg = cf.gemm(dev(A, dtype), dev(I.lay_out_weight(Bm, layout), dtype),
                 b_layout=cf.CF_LAYOUT_NK if layout == "nk" else cf.CF_LAYOUT_KN,
                 bias=dev(bias, "f32"), alpha=0.5, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = 0.5 * O.matmul(A, Bm) + bias
    got = host(Cg)
    assert_close_f32(got, ref, "gemm") if dtype == "f32" else None
    assert rel_rms(got, ref) < 1e-6


# bf16 B stored K x N with K a multiple of 64 (>= 192) takes the direct-to-LDS
# ring with transposing LDS reads: ragged M, N not a multiple of the tile
# width (clamped columns), batched operands.
@pytest.mark.parametrize("M,K,N,nb", [(300, 256, 224, 1), (129, 192, 288, 1), (64, 512, 1024, 2),
                                      (257, 256, 96, 1), (33, 2048, 128, 3)])
def test_gemm_kn_ring(M, K, N, nb):
    A = np.stack([_rand((M, K), 11 + i, "bf16") for i in range(nb)])
    Bm = np.stack([_rand((K, N), 21 + i, "bf16", 1 / np.sqrt(K)) for i in range(nb)])
    Cg = cf.gemm(dev(A), dev(Bm), b_layout=cf.CF_LAYOUT_KN, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = np.stack([O.matmul(A[i], Bm[i]) for i in range(nb)])
    got = host(Cg)
    assert got.shape == ref.shape
    assert rel_rms(got, ref) < 1e-6
    assert np.max(np.abs(got - ref)) < 1e-4 * np.max(np.abs(ref))


def test_gemm_kn_attention_pv_full_length():
    """P.V of two heads at the attention workload's length (2048 keys, d = 128):
    the unfused comparator's second product, B stored K x N."""
    nb, L, d = 2, 2048, 128
    rng = np.random.default_rng(31)
    Pb = I.round_to_bf16((rng.random((nb, L, L)) / L * 2).astype(np.float32))
    V = np.stack([_rand((L, d), 32 + i, "bf16") for i in range(nb)])
    O2 = cf.gemm(dev(Pb), dev(V), b_layout=cf.CF_LAYOUT_KN, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = np.stack([O.matmul(Pb[i], V[i]) for i in range(nb)])
    assert rel_rms(host(O2), ref) < 1e-6


def test_gemm_batched_attention_shapes():
    B, L, d = 3, 160, 64
    Q, K, V = (_rand((B, L, d), s, "bf16") for s in (4, 5, 6))
    S = cf.gemm(dev(Q), dev(K), b_layout=cf.CF_LAYOUT_NK, alpha=1 / 8, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = np.stack([O.matmul(Q[i], K[i].T) / 8 for i in range(B)])
    assert rel_rms(host(S), ref) < 1e-6
    Pm = (np.random.default_rng(7).random((B, L, L)) / L).astype(np.float32)
    Pb = I.round_to_bf16(Pm)
    O2 = cf.gemm(dev(Pb), dev(V), b_layout=cf.CF_LAYOUT_KN, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref2 = np.stack([O.matmul(Pb[i], V[i]) for i in range(B)])
    assert rel_rms(host(O2), ref2) < 1e-6


def test_rowop_softmax():
    S = _rand((50, 1024), 8, "f32", 3.0)
    Y = torch.empty((50, 1024), dtype=torch.float32, device="cuda")
    cf.rowop(dev(S, "f32"), [dict(kind=cf.CF_N_SOFTMAX, out=Y, ld=1024, dtype=cf.CF_F32, f0=0.25)])
    torch.cuda.synchronize()
    got = host(Y)
    ref = O.softmax_rows(0.25 * S.astype(np.float64))
    np.testing.assert_allclose(got.sum(axis=1), 1.0, atol=1e-5)
    assert np.max(np.abs(got - ref)) < 1e-6


@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("batch,M,N,K,out", [
    (1, 4096, 4096, 1024, "bf16"),    # whole tiles, an even number of k steps
    (1, 8165, 2080, 1088, "f32"),     # ragged last row block and column tile, an odd number of steps
    (3, 2049, 2048, 1152, "bf16"),    # one row in the last row block, batched
])
def test_gemm_large_tile(batch, M, N, K, out, layout):
    """Products large enough for the 256 x 256 tile, every element against an fp32 product.  Both sides sum K
    products of unit-variance terms in fp32 (error about 2^-24 sqrt(K) each, K <= 1152: 2e-6 of the rms; 1e-5
    allowed); bf16 stores round by at most 2^-8 of the value."""
    g = torch.Generator(device="cuda").manual_seed(M + N)
    A = torch.randn((batch, M, K), generator=g, device="cuda").bfloat16()
    B = (torch.randn((K, N) if layout == "kn" else (N, K), generator=g, device="cuda") / K ** 0.5).bfloat16()
    bias = torch.randn((N,), generator=g, device="cuda")
    C = cf.gemm(A, B, b_layout=cf.CF_LAYOUT_KN if layout == "kn" else cf.CF_LAYOUT_NK, bias=bias, alpha=0.5,
                out_dtype=torch.float32 if out == "f32" else torch.bfloat16)
    torch.cuda.synchronize()
    Bf = B.float() if layout == "kn" else B.float().t().contiguous()
    for b in range(batch):
        ref = 0.5 * (A[b].float() @ Bf) + bias
        err = (C[b].float() - ref).abs()
        assert float((err - (2.0 ** -8 * ref.abs() if out == "bf16" else 0.0)).max()) < 1e-5


def test_split_path_large_tile():
    """LayerNorm, GELU, row amax and codes over a product that takes the 256 x 256 tile: the row pass adds bias and
    residual and takes the statistics itself.  Sampled rows against fp64; the bounds are the chain's (bf16 Z)."""
    M, N, K = 4099, 4096, 1024
    g = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randn((M, K), generator=g, device="cuda").bfloat16()
    W = (torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).bfloat16()
    R = torch.randn((M, N), generator=g, device="cuda").bfloat16()
    b = torch.randn((N,), generator=g, device="cuda")
    Z, s, Q = cf.ln_gelu_amax(X, W, b, R)
    torch.cuda.synchronize()
    rows = list(range(0, M, 127)) + [M - 1]
    x = X[rows].double() @ W.double().t().contiguous() + b.double() + R[rows].double()
    x = x - x.mean(1, keepdim=True)
    x = x / torch.sqrt(x.square().mean(1, keepdim=True) + 1e-5)
    z = 0.5 * x * (1.0 + torch.erf(x / 2 ** 0.5))
    assert float((Z[rows].double() - z).abs().max()) < 2e-2
    assert torch.allclose(s[rows].double(), z.abs().amax(1) / 448.0, rtol=1e-3)
    assert bool((Q.view(torch.uint8) & 0x7F).amax(1).eq(0x7E).all())     # the row maximum is coded as +-448


def _apart(g, *shape, std=1.0, pad=8, gap=16, dtype=torch.bfloat16):
    """A tensor whose rows lie `pad` elements apart and whose matrices `gap` further; NaN in between."""
    *lead, rows, cols = shape
    n = int(np.prod(lead)) if lead else 1
    sb = rows * (cols + pad) + gap
    store = torch.full((n * sb,), float("nan"), device="cuda", dtype=dtype)
    t = store.as_strided((n, rows, cols), (sb, cols + pad, 1))
    t.copy_(torch.randn((n, rows, cols), generator=g, device="cuda") * std)
    return t if lead else t[0]


PITCHED = [
    (3, 33, 96, 272, "bf16"),       # 32 x 32 and 32 x 64 tiles, K past whole stages
    (2, 17, 160, 1040, "f32"),
    (1, 130, 4096, 1024, "bf16"),   # 64 x 64 tiles
    (1, 2049, 4128, 1088, "bf16"),  # 256 x 256 tiles, one row and 32 columns past
    (3, 2049, 2048, 1152, "bf16"),
    (1, 300, 768, 784, "f32"),
]


@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("batch,M,N,K,dtype", PITCHED)
def test_products_with_pitches_and_special_values(batch, M, N, K, dtype, layout):
    """Row pitches beyond the row and gaps between batch entries, fp32 outputs against an fp32 product (see
    test_gemm_large_tile for the bound; fp32 operands add their own rounding, 1e-4 as elsewhere); what lies between the
    rows stays.  Then an infinity or NaN in the first, a middle and the last row of A (in the last k) and in the last
    column of B: exactly their rows and columns are affected, as in the reference product."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    A = _apart(g, batch, M, K, dtype=t)
    B = _apart(g, batch, *((K, N) if layout == "kn" else (N, K)), std=K ** -0.5, dtype=t)
    bias = torch.randn((N,), generator=g, device="cuda")
    out = torch.full((batch, M, N + 8), 7.0, device="cuda")

    def run():
        cf.gemm(A, B, b_layout=cf.CF_LAYOUT_KN if layout == "kn" else cf.CF_LAYOUT_NK, bias=bias, alpha=0.5,
                out=out[..., :N])
        torch.cuda.synchronize()
        ref = [0.5 * (A[b].float() @ (B[b].float() if layout == "kn" else B[b].float().t().contiguous())) + bias
               for b in range(batch)]
        return out[..., :N], torch.stack(ref)
    got, ref = run()
    assert float((got - ref).abs().max()) < (1e-4 if dtype == "f32" else 1e-5)
    assert bool((out[..., N:] == 7.0).all())
    clean = got.clone()
    A[0, 0, K - 1], A[0, M // 2, 3], A[batch - 1, M - 1, K - 1] = float("inf"), float("nan"), float("-inf")
    if layout == "kn":
        B[0, K - 1, N - 1] = float("nan")
    else:
        B[0, N - 1, K - 1] = float("nan")
    got, ref = run()
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    inf = torch.isinf(ref)
    assert torch.equal(torch.isinf(got), inf) and torch.equal(got[inf], ref[inf])
    same = torch.isfinite(ref)
    assert torch.equal(got[same], clean[same])
