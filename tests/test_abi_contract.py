"""C-ABI contract tests that need no GPU: the library loads, exports every
symbol the header declares, and rejects invalid calls before any launch.
Fake (never dereferenced) device addresses are used: validation returns
before anything is enqueued, and M = 0 is a no-op."""
import ctypes as C
import os
import re

import pytest

from paper_2608_03537_amd import comfuse as cf

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "comfuse.h")
with open(HEADER) as _f:
    _TEXT = _f.read()
    HDR = int(re.search(r"#define CF_WS_HEADER_BYTES (\d+)", _TEXT).group(1))
    B2B_HDR = int(re.search(r"#define CF_B2B_WS_HEADER_BYTES (\d+)", _TEXT).group(1))

A = 0x7F0000000000          # 16-byte aligned fake device addresses
B = 0x7F0000100000
Y = 0x7F0000200000
R = 0x7F0000300000
V = 0x7F0000400000


def header_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(cf_[a-z0-9_]+)\s*\(", text)))


def test_exports_every_declared_symbol():
    lib = cf.lib()
    names = header_functions()
    assert len(names) >= 11
    for n in names:
        assert hasattr(lib, n), f"{n} declared in comfuse.h but not exported"


def test_version_and_status_strings():
    assert cf.cf_version() == 1
    for s in range(12):
        assert cf.cf_status_string(s).startswith(cf.STATUS[s])


def _pn(**kw):
    a = cf.PostnormArgs()
    a.struct_size = C.sizeof(cf.PostnormArgs)
    a.M, a.N, a.K = kw.get("M", 64), kw.get("N", 256), kw.get("K", 128)
    a.in_dtype, a.out_dtype = kw.get("in_dtype", cf.CF_BF16), kw.get("out_dtype", cf.CF_BF16)
    a.X, a.ldx = kw.get("X", A), kw.get("ldx", a.K)
    a.W, a.ldw, a.w_layout = kw.get("W", B), kw.get("ldw", a.K), kw.get("w_layout", cf.CF_LAYOUT_NK)
    a.bias, a.gamma, a.beta = kw.get("bias", V), kw.get("gamma", None), kw.get("beta", None)
    a.R, a.ldr = kw.get("R", R), kw.get("ldr", a.N)
    a.alpha, a.eps = 1.0, kw.get("eps", 1e-5)
    a.Y, a.ldy = kw.get("Y", Y), kw.get("ldy", a.N)
    a.path = kw.get("path", 0)
    return a


def _call(a, ws=None, nbytes=0):
    return cf.cf_gemm_postnorm(a, ws, nbytes, None)


def test_postnorm_m0_is_noop():
    assert _call(_pn(M=0)) == 0          # also proves the ctypes layout matches


@pytest.mark.parametrize("kw,status", [
    (dict(X=None), "CF_ERR_NULL"),
    (dict(Y=None), "CF_ERR_NULL"),
    (dict(W=None), "CF_ERR_NULL"),
    (dict(N=48), "CF_ERR_SHAPE"),
    (dict(K=40), "CF_ERR_SHAPE"),
    (dict(M=-1), "CF_ERR_SHAPE"),
    (dict(N=16384, ldy=16384, ldr=16384), "CF_ERR_SHAPE"),
    (dict(ldx=64), "CF_ERR_LD"),
    (dict(ldy=128), "CF_ERR_LD"),
    (dict(X=A + 2), "CF_ERR_ALIGN"),
    (dict(ldx=132), "CF_ERR_ALIGN"),
    (dict(bias=V + 4), "CF_ERR_ALIGN"),
    (dict(in_dtype=cf.CF_F32, out_dtype=cf.CF_BF16), "CF_ERR_DTYPE"),
    (dict(in_dtype=cf.CF_FP8_E4M3), "CF_ERR_DTYPE"),
    (dict(Y=A), "CF_ERR_ALIAS"),
    (dict(Y=R), "CF_ERR_ALIAS"),
    (dict(path=1, N=1024, ldy=1024, ldr=1024), "CF_ERR_UNSUPPORTED"),
    (dict(path=7), "CF_ERR_UNSUPPORTED"),
])
def test_postnorm_rejects(kw, status):
    s = _call(_pn(**kw))
    assert cf.STATUS[s] == status, cf.cf_last_error()
    assert cf.cf_last_error()


def test_struct_size_checked():
    a = _pn()
    a.struct_size = 8
    assert cf.STATUS[_call(a)] == "CF_ERR_STRUCT"


def test_split_workspace_required():
    a = _pn(path=3, N=1024, ldy=1024, ldr=1024)
    need = cf.cf_gemm_postnorm_workspace(a)
    # header + partials M x ceil(N/TN) float2 + fp32 x, each rounded to 256 B
    rnd = lambda v: (v + 255) // 256 * 256
    assert need in [HDR + rnd(64 * -(-1024 // tn) * 8) + 64 * 1024 * 4 for tn in (128, 192, 256)]
    assert cf.STATUS[_call(a)] == "CF_ERR_WORKSPACE"
    assert cf.STATUS[_call(a, A, need - 1)] == "CF_ERR_WORKSPACE"


def test_workspace_by_path():
    assert cf.cf_gemm_postnorm_workspace(_pn(N=768, ldy=768, ldr=768, path=1)) == 0
    # auto picks the row-cluster path here: the header holds its exchange records
    need = cf.cf_gemm_postnorm_workspace(_pn(N=768, ldy=768, ldr=768))
    assert need == HDR
    assert cf.STATUS[_call(_pn(N=768, ldy=768, ldr=768))] == "CF_ERR_WORKSPACE"


def _sg(nodes, **kw):
    arr = cf.make_nodes(nodes)
    a = cf.SubgraphArgs()
    a.struct_size = C.sizeof(cf.SubgraphArgs)
    a.M, a.N, a.K = kw.get("M", 64), 256, 128
    a.in_dtype = cf.CF_BF16
    a.X, a.ldx, a.W, a.ldw, a.w_layout = A, 128, B, 128, cf.CF_LAYOUT_NK
    a.nodes, a.n_nodes, a.path = arr, len(nodes), 0
    return a, arr


def test_subgraph_grammar():
    ok = [dict(kind=cf.CF_N_BIAS, v0=V), dict(kind=cf.CF_N_LAYERNORM, f0=1e-5), dict(kind=cf.CF_N_GELU),
          dict(kind=cf.CF_N_STORE, out=Y, ld=256, dtype=cf.CF_BF16),
          dict(kind=cf.CF_N_ROWAMAX_QUANT, out=R, out2=0x7F0000500000, ld=256, f0=448.0)]
    a, keep = _sg(ok, M=0)
    assert cf.cf_gemm_subgraph(a, None, 0, None) == 0
    bad_order = [ok[2], ok[1], ok[3]]
    a, keep = _sg(bad_order)
    assert cf.STATUS[cf.cf_gemm_subgraph(a, None, 0, None)] == "CF_ERR_UNSUPPORTED"
    no_out = ok[:3]
    a, keep = _sg(no_out)
    assert cf.STATUS[cf.cf_gemm_subgraph(a, None, 0, None)] == "CF_ERR_UNSUPPORTED"
    softmax = [dict(kind=cf.CF_N_SOFTMAX, out=Y, ld=256, dtype=cf.CF_BF16, f0=1.0)]
    a, keep = _sg(softmax)
    assert cf.STATUS[cf.cf_gemm_subgraph(a, None, 0, None)] == "CF_ERR_UNSUPPORTED"
    bad_q = ok[:4] + [dict(kind=cf.CF_N_ROWAMAX_QUANT, out=R, out2=0x7F0000500000, ld=250, f0=448.0)]
    a, keep = _sg(bad_q)
    assert cf.STATUS[cf.cf_gemm_subgraph(a, None, 0, None)] == "CF_ERR_ALIGN"


def test_subgraph_grammar_softcap_softmax():
    store = dict(kind=cf.CF_N_STORE, out=Y, ld=256, dtype=cf.CF_BF16)
    msts = [dict(kind=cf.CF_N_SCALE, f0=0.5), dict(kind=cf.CF_N_SOFTCAP, f0=30.0), dict(kind=cf.CF_N_SOFTMAX), store]
    a, keep = _sg(msts, M=0)
    assert cf.cf_gemm_subgraph(a, None, 0, None) == 0
    for cap in (0.0, -1.0, float("inf"), float("nan")):
        a, keep = _sg([dict(kind=cf.CF_N_SOFTCAP, f0=cap), store])
        assert cf.STATUS[cf.cf_gemm_subgraph(a, None, 0, None)] == "CF_ERR_SHAPE", cap
    for bad in ([dict(kind=cf.CF_N_LAYERNORM, f0=1e-5), dict(kind=cf.CF_N_SOFTMAX), store],
                [dict(kind=cf.CF_N_SOFTMAX), dict(kind=cf.CF_N_GELU), store],
                [dict(kind=cf.CF_N_SOFTCAP, f0=30.0), dict(kind=cf.CF_N_GELU), store]):
        a, keep = _sg(bad)
        assert cf.STATUS[cf.cf_gemm_subgraph(a, None, 0, None)] == "CF_ERR_UNSUPPORTED"


def test_gemm_and_rowop_validation():
    st = cf.STATUS
    assert cf.cf_gemm(1, 0, 256, 128, cf.CF_BF16, cf.CF_BF16, A, 128, 0, B, 128, 0, cf.CF_LAYOUT_NK,
                      None, 1.0, Y, 256, 0, None) == 0
    assert st[cf.cf_gemm(1, 64, 250, 128, cf.CF_BF16, cf.CF_BF16, A, 128, 0, B, 128, 0, cf.CF_LAYOUT_NK,
                         None, 1.0, Y, 256, 0, None)] == "CF_ERR_SHAPE"
    assert st[cf.cf_gemm(1, 64, 256, 128, cf.CF_BF16, cf.CF_BF16, A, 128, 0, B, 128, 0, cf.CF_LAYOUT_NK,
                         None, 1.0, A, 256, 0, None)] == "CF_ERR_ALIAS"
    nodes = cf.make_nodes([dict(kind=cf.CF_N_SOFTMAX, out=Y, ld=256, dtype=cf.CF_BF16, f0=1.0)])
    assert cf.cf_rowop(1, 0, 256, cf.CF_BF16, A, 256, 0, nodes, 1, None) == 0
    assert cf.cf_rowop(0, 64, 256, cf.CF_BF16, A, 256, 0, nodes, 1, None) == 0
    assert st[cf.cf_rowop(1, 4, 256, cf.CF_BF16, None, 256, 0, nodes, 1, None)] == "CF_ERR_NULL"
    nodes2 = cf.make_nodes([dict(kind=cf.CF_N_SOFTMAX, out=A, ld=256, dtype=cf.CF_BF16, f0=1.0)])
    assert st[cf.cf_rowop(1, 4, 256, cf.CF_BF16, A, 256, 0, nodes2, 1, None)] == "CF_ERR_ALIAS"
    # batch strides: multiples of 16 bytes, batch within [0, 65535]
    assert st[cf.cf_rowop(2, 4, 256, cf.CF_BF16, A, 256, 1028, nodes, 1, None)] == "CF_ERR_ALIGN"
    assert st[cf.cf_rowop(70000, 4, 256, cf.CF_BF16, A, 256, 1024, nodes, 1, None)] == "CF_ERR_SHAPE"


def test_workspace_check_without_workspace():
    # NULL workspace: nothing to check, no device call
    assert cf.cf_workspace_check(None, 0, None) == 0
    assert cf.STATUS[cf.cf_workspace_check(A + 8, 64, None)] == "CF_ERR_ALIGN"
    assert cf.STATUS[cf.cf_workspace_check(A, 2, None)] == "CF_ERR_WORKSPACE"


def test_noalloc_validation_before_any_device_call():
    store = dict(kind=cf.CF_N_STORE, out=Y, ld=256, dtype=cf.CF_BF16)
    ln = [dict(kind=cf.CF_N_LAYERNORM, f0=1e-5), store]
    a, keep = _sg(ln, M=0)
    assert cf.cf_gemm_subgraph_noalloc(a, None) == 0                 # M = 0: no-op
    a, keep = _sg(ln)
    a.path = cf.PATH_CLUSTER                                         # no cluster path here
    assert cf.STATUS[cf.cf_gemm_subgraph_noalloc(a, None)] == "CF_ERR_UNSUPPORTED"
    a, keep = _sg([dict(kind=cf.CF_N_GELU), store])
    a.struct_size = 8
    assert cf.STATUS[cf.cf_gemm_subgraph_noalloc(a, None)] == "CF_ERR_STRUCT"
    # split path larger than the 32 MiB scratch: 4096 x 4096 fp32 rows
    big_store = dict(kind=cf.CF_N_STORE, out=Y, ld=4096, dtype=cf.CF_BF16)
    arr = cf.make_nodes([dict(kind=cf.CF_N_LAYERNORM, f0=1e-5), big_store])
    b = cf.SubgraphArgs()
    b.struct_size = C.sizeof(cf.SubgraphArgs)
    b.M, b.N, b.K, b.in_dtype = 4096, 4096, 128, cf.CF_BF16
    b.X, b.ldx, b.W, b.ldw, b.w_layout = A, 128, B, 128, cf.CF_LAYOUT_NK
    b.nodes, b.n_nodes, b.path = arr, 2, 0
    assert cf.STATUS[cf.cf_gemm_subgraph_noalloc(b, None)] == "CF_ERR_WORKSPACE"
    assert "32" in cf.cf_last_error() or "scratch" in cf.cf_last_error()


def _mlp(**kw):
    a = cf.B2BArgs()
    a.struct_size = C.sizeof(cf.B2BArgs)
    a.batch, a.M, a.K, a.N1, a.N2 = (kw.get("batch", 1), kw.get("M", 300), kw.get("K", 1024), kw.get("N1", 512),
                                     kw.get("N2", 128))
    a.dtype, a.mid, a.out = cf.CF_BF16, cf.CF_MID_RELU_BIAS, kw.get("out", cf.CF_OUT_STORE)
    a.X, a.ldx, a.W1, a.ldw1, a.w1_layout = A, a.K, B, a.K, cf.CF_LAYOUT_NK
    a.W2, a.ldw2, a.w2_layout = R, a.N1, cf.CF_LAYOUT_NK
    a.b1, a.b2, a.O, a.ldo = V, V, Y, a.N2
    return a


def test_mlp_workspace_and_validation():
    # the fixed counter region, then 2 chunks x 300 rows x 128 fp32 partials (per batch entry)
    assert B2B_HDR == cf.CF_B2B_WS_HEADER_BYTES
    assert cf.cf_b2bgemm_workspace(_mlp()) == B2B_HDR + 2 * 300 * 128 * 4
    assert cf.cf_b2bgemm_workspace(_mlp(batch=3, M=1000, N1=1024)) == B2B_HDR + 3 * 4 * 1000 * 128 * 4
    # the split grid (batch x 128-row blocks x chunks) fits 256 workgroups;
    # beyond, one workgroup per row block runs every chunk: no workspace
    assert cf.cf_b2bgemm_workspace(_mlp(M=128 * 128)) == B2B_HDR + 2 * 128 * 128 * 128 * 4
    assert cf.cf_b2bgemm_workspace(_mlp(M=128 * 128 + 1)) == 0
    assert cf.cf_b2bgemm_workspace(_mlp(batch=2, M=128 * 64 + 1)) == 0
    assert cf.cf_b2bgemm_workspace(_mlp(batch=2, M=128 * 64)) == B2B_HDR + 2 * 2 * 128 * 64 * 128 * 4
    assert cf.cf_b2bgemm_workspace(_mlp(M=128 * 64, N1=1024)) == B2B_HDR + 4 * 128 * 64 * 128 * 4
    assert cf.cf_b2bgemm_workspace(_mlp(M=128 * 64 + 1, N1=1024)) == 0
    big = _mlp(batch=3, M=128 * 87382)
    big.sx, big.so = big.M * big.K, big.M * big.N2
    assert cf.cf_b2bgemm_workspace(big) == 0
    assert cf.STATUS[cf.cf_b2bgemm(_mlp(M=128 * 128), A, 1, None)] == "CF_ERR_WORKSPACE"
    assert cf.cf_b2bgemm_workspace(_mlp(N1=256)) == 0           # one chunk: nothing to sum
    assert cf.STATUS[cf.cf_b2bgemm(_mlp(), None, 0, None)] == "CF_ERR_WORKSPACE"
    assert cf.STATUS[cf.cf_b2bgemm(_mlp(N2=64), A, 1 << 30, None)] == "CF_ERR_UNSUPPORTED"
    assert cf.STATUS[cf.cf_b2bgemm(_mlp(N1=384), A, 1 << 30, None)] == "CF_ERR_UNSUPPORTED"
    assert cf.STATUS[cf.cf_b2bgemm(_mlp(K=96), A, 1 << 30, None)] == "CF_ERR_UNSUPPORTED"
    assert cf.STATUS[cf.cf_b2bgemm(_mlp(out=cf.CF_OUT_BIAS_RESIDUAL_LN), A, 1 << 30, None)] == "CF_ERR_UNSUPPORTED"
    assert cf.cf_b2bgemm(_mlp(M=0), None, 0, None) == 0


@pytest.mark.parametrize("M,N,K", [(200, 224, 400), (600, 256, 272), (9000, 768, 768)])
def test_optional_workspace_never_refuses(M, N, K):
    """A call whose workspace is optional runs on whole rows where the row cluster does not fit the device (here: no
    device at all, so the launch fails, as it does without the workspace)."""
    torch = pytest.importorskip("torch")
    if torch.cuda.is_available():
        pytest.skip("the addresses are fake: only without a device is nothing launched")
    kw = dict(M=M, N=N, K=K, ldy=N, ldr=N, ldw=K, ldx=K)
    need = cf.cf_gemm_postnorm_workspace(_pn(**kw))
    assert need == cf.CF_WS_OPTIONAL_BYTES
    assert cf.STATUS[_call(_pn(**kw))] == "CF_ERR_HIP"
    assert cf.STATUS[_call(_pn(**kw), 0x7F0000800000, need)] == "CF_ERR_HIP", cf.cf_last_error()
    # a path asked for by name is refused as before
    assert cf.STATUS[_call(_pn(**dict(kw, N=768, ldy=768, ldr=768, path=2)), 0x7F0000800000, need)] == "CF_ERR_UNSUPPORTED"
