"""GPU parity of cf_b2bgemm (back-to-back GEMM with the intermediate in
registers) against the fp64 oracle.

FFN:  Y = LN(GELU(X W1 + b1) W2 + b2 + X), bf16, max-abs 2e-2 and rel-RMS
5e-3 (the on-chip intermediate S is rounded to bf16 as the second product's
operand; the oracle keeps it exact).  Full size M=65536, d=256, N1=512 is
compared over every element.
Attention: O = softmax(Q K^T / sqrt(d)) V per head, online softmax; rel-RMS
5e-3 is the binding check (|O| is small, so max-abs 2e-2 is loose), plus the
invariants V = 1 -> O = 1 and Q = 0 -> O = mean_j V_j.
"""
import ctypes as C

import numpy as np
import pytest

from oracle import comfuse_oracle as O
from paper_2608_03537_amd import inputs as I
from tests.helpers import assert_close_bf16, dev, host, max_abs, rel_rms

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_03537_amd import comfuse as cf  # noqa: E402


def run_ffn(inp, layernorm=True, residual=True):
    X = dev(inp.X)
    W1t = dev(I.lay_out_weight(inp.W1, "nk"))
    W2t = dev(I.lay_out_weight(inp.W2, "nk"))
    Y = cf.b2b_ffn(X, W1t, dev(inp.b1, "f32"), W2t, dev(inp.b2, "f32"), X if residual else None,
                   eps=inp.eps, layernorm=layernorm)
    torch.cuda.synchronize()
    return host(Y)


@pytest.mark.parametrize("M,d,N1", [(300, 64, 128), (129, 128, 256), (257, 256, 256), (200, 256, 512)])
def test_ffn_small(M, d, N1):
    inp = I.ffn_inputs(seed=2, M=M, d=d, N1=N1)
    ref = O.ffn_b2b(inp.X, inp.W1, inp.b1, inp.W2, inp.b2, eps=inp.eps)
    assert_close_bf16(run_ffn(inp), ref, f"FFN {M}x{d}x{N1}")


def test_ffn_without_layernorm():
    inp = I.ffn_inputs(seed=3, M=160, d=128, N1=256)
    got = run_ffn(inp, layernorm=False, residual=False)
    S = O.gelu_erf(O.bias_residual(O.matmul(inp.X, inp.W1), inp.b1))
    ref = O.bias_residual(O.matmul(S, inp.W2), inp.b2)
    assert rel_rms(got, ref) < 5e-3 and max_abs(got, ref) < 2e-2


@pytest.mark.parametrize("M,d,N1", [(190, 128, 256), (257, 256, 512)])
def test_ffn_other_residual_gamma_beta(M, d, N1):
    """Residual R != X (read from memory) and a LayerNorm with gamma/beta."""
    inp = I.ffn_inputs(seed=5, M=M, d=d, N1=N1)
    rng = np.random.default_rng(7)
    R = I.round_to_bf16(rng.standard_normal((M, d)).astype(np.float32))
    gamma = (1.0 + 0.1 * rng.standard_normal(d)).astype(np.float32)
    beta = (0.1 * rng.standard_normal(d)).astype(np.float32)
    X = dev(inp.X)
    Y = cf.b2b_ffn(X, dev(I.lay_out_weight(inp.W1, "nk")), dev(inp.b1, "f32"), dev(I.lay_out_weight(inp.W2, "nk")),
                   dev(inp.b2, "f32"), dev(R), dev(gamma, "f32"), dev(beta, "f32"), eps=inp.eps)
    torch.cuda.synchronize()
    S = O.gelu_erf(O.bias_residual(O.matmul(inp.X, inp.W1), inp.b1))
    ref = O.layernorm(O.bias_residual(O.matmul(S, inp.W2), inp.b2, R), gamma, beta, inp.eps)
    assert_close_bf16(host(Y), ref, f"FFN R != X {M}x{d}x{N1}")


def test_ffn_zero_second_weight_is_layernorm_of_input():
    inp = I.ffn_inputs(seed=4, M=256, d=256, N1=512)
    inp.W2[:] = 0.0
    inp.b2[:] = 0.0
    got = run_ffn(inp)
    assert_close_bf16(got, O.layernorm(inp.X), "W2 = 0")


def test_ffn_full_size():
    inp = I.ffn_inputs()
    ref = O.ffn_b2b(inp.X, inp.W1, inp.b1, inp.W2, inp.b2, eps=inp.eps)
    assert_close_bf16(run_ffn(inp), ref, "FFN 65536x256x512")


@pytest.mark.parametrize("residual", ["x", "other"])
def test_ffn_batched(residual):
    """batch = 3 entries of 257 rows, d = 256, N1 = 512: X, R, O [3, M, d];
    W1 shared (2-D), W2 per entry (3-D); b1, b2, gamma, beta shared.  R = X
    takes the kernel's residual-from-the-X-tile path, another R the load."""
    Bn, M, d, N1 = 3, 257, 256, 512
    ins = [I.ffn_inputs(seed=30 + b, M=M, d=d, N1=N1) for b in range(Bn)]
    X = dev(np.stack([t.X for t in ins]))
    Rh = np.stack([t.X for t in ins]) if residual == "x" else \
        I.round_to_bf16(np.random.default_rng(9).standard_normal((Bn, M, d)).astype(np.float32))
    R = X if residual == "x" else dev(Rh)
    W1t = dev(I.lay_out_weight(ins[0].W1, "nk"))
    W2t = dev(np.stack([I.lay_out_weight(t.W2, "nk") for t in ins]))
    Y = cf.b2b_ffn(X, W1t, dev(ins[0].b1, "f32"), W2t, dev(ins[0].b2, "f32"), R, eps=ins[0].eps)
    torch.cuda.synchronize()
    got = host(Y)
    for b in range(Bn):
        S = O.gelu_erf(O.bias_residual(O.matmul(ins[b].X, ins[0].W1), ins[0].b1))
        ref = O.layernorm(O.bias_residual(O.matmul(S, ins[b].W2), ins[0].b2, Rh[b]), eps=ins[0].eps)
        assert_close_bf16(got[b], ref, f"FFN batch entry {b} residual={residual}")


def run_attn(Q, K, V, scale=None):
    o = cf.b2b_attention(dev(Q), dev(K), dev(V), scale)
    torch.cuda.synchronize()
    return host(o)


@pytest.mark.parametrize("d,N1", [(64, 128), (128, 256), (256, 256), (256, 512)])
@pytest.mark.parametrize("batch,M,own", [(1, 1, True), (1, 33, False), (2, 1000, True), (1, 8192, False),
                                         (1, 8193, True), (3, 2753, False)])
def test_ffn_forms(batch, M, own, d, N1):
    """Both sides of the 32-row / 128-row choice (256 row blocks of 32), every compiled shape, with R = X and without
    gamma and beta (own) or with another R and an affine LayerNorm, against fp64 on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(M + N1 + d)
    rnd = lambda *sh, std=1.0: torch.randn(sh, generator=g, device="cuda") * std
    X = rnd(batch, M, d).bfloat16()
    W1, W2 = rnd(N1, d, std=d ** -0.5).bfloat16(), rnd(d, N1, std=N1 ** -0.5).bfloat16()
    b1, b2 = rnd(N1, std=0.5), rnd(d, std=0.5)
    R = X if own else rnd(batch, M, d).bfloat16()
    gamma, beta = (None, None) if own else (1.0 + rnd(d, std=0.1), rnd(d, std=0.1))
    Y = cf.b2b_ffn(X, W1, b1, W2, b2, R, gamma, beta)
    torch.cuda.synchronize()
    x = X.double().reshape(-1, d)
    h = x @ W1.double().t().contiguous() + b1.double()
    o = (0.5 * h * (1.0 + torch.erf(h / 2 ** 0.5))) @ W2.double().t().contiguous() + b2.double()
    o = o + R.double().reshape(-1, d)
    o = o - o.mean(1, keepdim=True)
    o = o / torch.sqrt(o.square().mean(1, keepdim=True) + 1e-5)
    if not own:
        o = o * gamma.double() + beta.double()
    err = Y.double().reshape(-1, d) - o
    # the suite's bf16 bounds, the largest error scaled with the largest value (an ulp at 4 is 2^-6)
    assert float(err.square().sum().sqrt() / o.square().sum().sqrt()) < 5e-3
    assert float((err.abs() / o.abs().clamp(min=1.0)).max()) < 2e-2


def attention_form(M, batch, Lk, d):
    """(query waves per workgroup, 0 for two workgroups per CU; workgroups that share a query block's keys): the
    library's own choice, by its C++ name."""
    f = cf.lib()._ZN2cf14attention_formEllli
    f.argtypes, f.restype = (C.c_int64, C.c_int64, C.c_int64, C.c_int), C.c_uint64
    r = f(M, batch, Lk, d)
    return r & 0xFFFFFFFF, r >> 32


@pytest.mark.parametrize("B,H,Lq,Lk,d", [(1, 2, 200, 300, 64), (2, 1, 129, 64, 128), (1, 3, 64, 1, 128),
                                         (1, 1, 256, 333, 128), (1, 2, 130, 289, 128), (1, 1, 100, 350, 64)])
def test_attention_small(B, H, Lq, Lk, d):
    a = I.attention_inputs(seed=5, B=B, H=H, Lq=Lq, Lk=Lk, d=d)
    got = run_attn(a.Q, a.K, a.V)
    ref = O.attention(a.Q, a.K, a.V)
    assert rel_rms(got, ref) < 5e-3, rel_rms(got, ref)
    assert max_abs(got, ref) < 2e-2


# Ragged Lk puts the partial last key block in either ring stage: with an odd
# block count (289 keys: five of 64) it is loaded from stage 1's step, with an
# even one (333: six) from stage 0's, for both head dimensions.
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Lk", [289, 333, 33, 70])
def test_attention_two_workgroups_per_cu(Lk, d):
    """The form of large calls (four query waves, one key group) with a partial last key block, some heads against the
    oracle."""
    B, H, Lq = 1, 257, 70
    assert attention_form(Lq, B * H, Lk, d) == (0, 1)
    a = I.attention_inputs(seed=9, B=B, H=H, Lq=Lq, Lk=Lk, d=d)
    got = run_attn(a.Q, a.K, a.V)
    heads = [0, 1, 100, 255, 256]
    ref = O.attention(a.Q[:, heads], a.K[:, heads], a.V[:, heads])
    assert rel_rms(got[:, heads], ref) < 5e-3 and max_abs(got[:, heads], ref) < 2e-2


@pytest.mark.parametrize("which", ["self", "target"])
def test_attention_table2_shapes(which):
    """Table 2 shapes (one batch, two heads), every element against the oracle:
    Self-Attention (512 x 512, d 128) and Target-Attention (4096 target rows,
    256 source rows, d 128)."""
    a = I.self_attention_table2(seed=3, B=1, H=2) if which == "self" else I.target_attention_table2(seed=3, B=1, H=2)
    got = run_attn(a.Q, a.K, a.V)
    ref = O.attention(a.Q, a.K, a.V)
    assert rel_rms(got, ref) < 5e-3 and max_abs(got, ref) < 2e-2, (rel_rms(got, ref), max_abs(got, ref))


def test_attention_invariants():
    a = I.attention_inputs(seed=6, B=1, H=2, Lq=128, Lk=200, d=128)
    # V = 1: the row sums l and the numerator add the same bf16 P (in fp32,
    # in different orders), so O / l is within a few fp32 ulps of 1 and every
    # bf16 output is exactly 1
    ones = run_attn(a.Q, a.K, np.ones_like(a.V))
    assert np.array_equal(ones, np.ones_like(ones)), np.max(np.abs(ones - 1.0))
    zq = run_attn(np.zeros_like(a.Q), a.K, a.V)
    mean_v = a.V.astype(np.float64).mean(axis=2, keepdims=True)
    assert max_abs(zq, np.broadcast_to(mean_v, zq.shape)) < 4e-3


def test_attention_full_size_sampled_rows():
    # one query row in every 128-query block of every (batch, head), at a
    # position that moves from block to block and head to head
    a = I.attention_inputs()
    got = run_attn(a.Q, a.K, a.V)
    nblk = (a.Lq + 127) // 128
    for b in range(a.B):
        for h in range(a.H):
            off = (np.arange(nblk) * 37 + 11 * (b * a.H + h)) % 128
            rows = np.minimum(np.arange(nblk) * 128 + off, a.Lq - 1)
            ref = O.attention(a.Q[b, h][rows], a.K[b, h], a.V[b, h])
            g = got[b, h][rows]
            assert rel_rms(g, ref) < 5e-3, (b, h, rel_rms(g, ref))
            assert max_abs(g, ref) < 2e-2, (b, h, max_abs(g, ref))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,H,Lq,Lk,qg", [
    (1, 3, 1, 1, 1),        # one query, one key: three of four key groups empty (d = 64: one key group)
    (2, 16, 5, 33, 1),      # two key blocks, the last of one key
    (1, 2, 31, 1000, 1),    # few queries, keys split over workgroups, ragged last block
    (2, 8, 16, 4097, 1),    # the same, one key past a block
    (1, 9, 33, 290, 1),     # two 32-query blocks
    (70, 4, 33, 129, 2),    # 32 < Lq <= 64: two query waves, four key groups
    (5, 13, 250, 200, 4),   # 130 128-query blocks: four query waves, two key groups
    (70, 4, 33, 128, 0),    # two query waves, with the most keys that keep one group
    (4, 16, 511, 192, 0),   # and for four query waves
    (4, 16, 511, 321, 4),   # 256 128-query blocks: an odd number of key blocks
    (1, 16, 600, 321, 2),   # 160 64-query blocks
])
def test_attention_key_groups(B, H, Lq, Lk, qg, d):
    """Shapes that take a form with several key groups per workgroup (and, with few queries, several workgroups per
    query block), with the workspace and without it, against the oracle on some heads."""
    form = attention_form(Lq, B * H, Lk, d)
    assert form[0] == (0 if d == 64 and Lk <= 64 else qg) and (form[1] > 1) == (Lk >= 1000)
    g = torch.Generator(device="cuda").manual_seed(Lq + Lk)
    Q, K, V = (torch.randn((B, H, n, d), generator=g, device="cuda").bfloat16() for n in (Lq, Lk, Lk))
    got = [cf.b2b_attention(Q, K, V), cf.b2b_attention(Q, K, V)]
    a = cf._b2b_args(batch=B * H, M=Lq, K=d, N1=Lk, N2=d, dtype=cf.CF_BF16, X=Q.data_ptr(), ldx=d, sx=Lq * d,
                     W1=K.data_ptr(), ldw1=d, sw1=Lk * d, w1_layout=cf.CF_LAYOUT_NK, mid=cf.CF_MID_SOFTMAX,
                     mid_scale=d ** -0.5, W2=V.data_ptr(), ldw2=d, sw2=Lk * d, w2_layout=cf.CF_LAYOUT_KN,
                     out=cf.CF_OUT_STORE, ldo=d, so=Lq * d)
    alone = torch.empty_like(Q)
    a.O = alone.data_ptr()
    cf._check(cf.cf_b2bgemm(a, None, 0, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert torch.equal(got[0], got[1])
    heads = [(0, 0), (B - 1, H - 1), (B // 2, H // 3)]
    for b, h in heads:
        q, k, v = (t[b:b + 1, h:h + 1].float().cpu().numpy() for t in (Q, K, V))
        ref = O.attention(q, k, v)[0, 0]
        for o in (got[0], alone):
            o = o[b, h].float().cpu().numpy().astype(np.float64)
            assert rel_rms(o, ref) < 5e-3 and max_abs(o, ref) < 2e-2
    ws = cf._ws_cache.get((str(Q.device), torch.cuda.current_stream().cuda_stream, "b2b"))
    if ws is not None:   # arrival counters are back at zero
        assert int(ws[:cf.CF_B2B_WS_HEADER_BYTES].view(torch.int32).abs().sum()) == 0


def test_attention_minus_infinity_scores_in_whole_key_groups():
    """Keys whose scores are -infinity have weight 0, also where they are all of a key group's or of a part's: for
    the even queries the products with every key from 20 on overflow to -infinity, the odd ones see all keys."""
    g = torch.Generator(device="cuda").manual_seed(3)
    Q, K, V = (torch.randn((1, 2, n, 128), generator=g, device="cuda").bfloat16() for n in (7, 1500, 1500))
    Q[:, :, ::2, 0], Q[:, :, 1::2, 0] = 4.0, 0.0
    K[:, :, :20, 0], K[:, :, 20:, 0] = 0.0, -3e38
    got = cf.b2b_attention(Q, K, V)
    torch.cuda.synchronize()
    for h in range(2):
        sc = Q[0, h].double() @ K[0, h].double().t().contiguous() * 128 ** -0.5
        sc[::2, 20:] = float("-inf")
        ref = torch.softmax(sc, 1) @ V[0, h].double()
        assert float((got[0, h].double() - ref).abs().max()) < 2e-2


def _wide(g, *shape, std=1.0, pad=8, gap=24):
    """A bf16 tensor whose rows lie `pad` elements apart and whose matrices `gap` further; NaN in between."""
    *lead, rows, cols = shape
    n = int(np.prod(lead)) if lead else 1
    sb = rows * (cols + pad) + gap
    store = torch.full((n * sb,), float("nan"), device="cuda", dtype=torch.bfloat16)
    t = store.as_strided((n, rows, cols), (sb, cols + pad, 1))
    t.copy_(torch.randn((n, rows, cols), generator=g, device="cuda") * std)
    return t, sb, cols + pad


@pytest.mark.parametrize("B,Lq,Lk,d", [(16, 1, 2111, 128), (8, 3, 1000, 64), (40, 40, 333, 64), (130, 40, 333, 128),
                                       (60, 400, 333, 64), (60, 400, 289, 128), (257, 70, 289, 64), (257, 70, 333, 128)])
def test_attention_row_pitches_and_batch_strides(B, Lq, Lk, d):
    """Every form with row pitches beyond d and gaps between the heads (the Python helper takes contiguous ones only),
    against an fp64 softmax; what lies between the rows is neither read into a result nor written."""
    g = torch.Generator(device="cuda").manual_seed(B + Lk)
    (Q, sq, lq), (K, sk, lk), (V, sv, lv) = (_wide(g, B, n, d) for n in (Lq, Lk, Lk))
    out = torch.full((B, Lq, d + 16), 7.0, device="cuda", dtype=torch.bfloat16)
    a = cf._b2b_args(batch=B, M=Lq, K=d, N1=Lk, N2=d, dtype=cf.CF_BF16, X=Q.data_ptr(), ldx=lq, sx=sq, W1=K.data_ptr(),
                     ldw1=lk, sw1=sk, w1_layout=cf.CF_LAYOUT_NK, mid=cf.CF_MID_SOFTMAX, mid_scale=d ** -0.5,
                     W2=V.data_ptr(), ldw2=lv, sw2=sv, w2_layout=cf.CF_LAYOUT_KN, out=cf.CF_OUT_STORE, O=out.data_ptr(),
                     ldo=d + 16, so=Lq * (d + 16))
    need = cf.cf_b2bgemm_workspace(a)
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda") if need else None
    for w in {None, ws}:
        out[..., :d] = 0.0
        cf._check(cf.cf_b2bgemm(a, cf._ptr(w), 0 if w is None else w.numel(), torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        for h in (0, B // 2, B - 1):
            ref = torch.softmax(Q[h].double() @ K[h].double().t().contiguous() * d ** -0.5, 1) @ V[h].double()
            err = out[h, :, :d].double() - ref
            assert float(err.norm() / ref.norm()) < 5e-3 and float(err.abs().max()) < 2e-2
        assert bool((out[..., d:] == 7.0).all()) and bool(torch.isfinite(out).all())


@pytest.mark.parametrize("M", [70, 3000])
@pytest.mark.parametrize("d,N1", [(64, 128), (256, 512)])
def test_ffn_row_pitches_and_special_values(d, N1, M):
    """Both FFN forms (32-row and, with 3 x 3000 rows, 128-row workgroups) with row pitches beyond the row and gaps
    between the batch entries; then rows of X that hold an infinity or NaN: they become NaN (LayerNorm) and no other
    row changes a bit."""
    g = torch.Generator(device="cuda").manual_seed(M + d)
    (X, sx, lx), (W1, sw1, l1), (W2, sw2, l2) = (_wide(g, 3, *s, std=f) for s, f in (
        ((M, d), 1.0), ((N1, d), d ** -0.5), ((d, N1), N1 ** -0.5)))
    R, _, _ = _wide(g, 3, M, d)
    b1, b2, gamma = (torch.randn(n, generator=g, device="cuda") * 0.5 for n in (N1, d, d))
    out = torch.full((3, M, d + 8), 7.0, device="cuda", dtype=torch.bfloat16)
    cf.b2b_ffn(X, W1, b1, W2, b2, R, gamma, out=out[..., :d])
    torch.cuda.synchronize()
    for i in range(3):
        h = X[i].double() @ W1[i].double().t().contiguous() + b1.double()
        o = (0.5 * h * (1.0 + torch.erf(h / 2 ** 0.5))) @ W2[i].double().t().contiguous() + b2.double() + R[i].double()
        o = o - o.mean(1, keepdim=True)
        o = o / torch.sqrt(o.square().mean(1, keepdim=True) + 1e-5) * gamma.double()
        err = out[i, :, :d].double() - o
        assert float(err.norm() / o.norm()) < 5e-3 and float((err.abs() / o.abs().clamp(min=1.0)).max()) < 2e-2
    assert bool((out[..., d:] == 7.0).all())
    before = out[..., :d].clone()
    spoiled = [(0, 3, 5, float("inf")), (1, 40, 0, float("nan")), (2, M - 1, d - 1, float("-inf"))]
    for b, m, k, v in spoiled:
        X[b, m, k] = v
    cf.b2b_ffn(X, W1, b1, W2, b2, R, gamma, out=out[..., :d])
    torch.cuda.synchronize()
    hit = torch.zeros((3, M), dtype=torch.bool, device="cuda")
    for b, m, _, _ in spoiled:
        hit[b, m] = True
    assert bool(torch.isnan(out[..., :d][hit]).all())
    assert torch.equal(out[..., :d][~hit], before[~hit])
