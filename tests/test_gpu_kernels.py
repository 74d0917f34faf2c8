"""Single-kernel parity on the GPU through the C ABI (zl_inspect.h):
the GEMM in its operand layouts (with the LoRA segment and split K) and causal GQA attention, against
fp64 references computed on the CPU from the same (bf16-rounded) inputs."""
import numpy as np
import pytest

import oracle
from oracle import ops
from tests.gpu_cases import rel_err

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _zl():
    from paper_2608_07974_amd import zl
    return zl


def _dev():
    return torch.device("cuda")


def _stream():
    return torch.cuda.current_stream().cuda_stream


# bf16 operands with contiguous M need M % 8 == 0 (16-byte rows; the library
# rejects the rest, tested on the CPU); fp32 is a configuration of small shapes
# and not run at 4096 x 3848 (its two kernels by size: test_gemm_f32_tiles).
_LAYOUT_CASES = [(dt, lay, M, N, K)
                 for dt in ("bf16", "f32") for lay in ("nt", "nn", "tn")
                 for M, N, K in ((8, 8, 8), (1, 8, 8), (304, 520, 200), (129, 136, 1000),
                                 (4096, 3848, 264))
                 if not (dt == "bf16" and lay == "tn" and M % 8)
                 and not (dt == "f32" and M * N * K > 1e9)]


@pytest.mark.parametrize("dtype,layout,M,N,K", _LAYOUT_CASES)
def test_gemm_layouts(dtype, layout, M, N, K):
    """C = A B^T with A(m,k), B(n,k) stored K-major or MN-major (fwd: nt,
    dgrad: nn, wgrad: tn), ragged in every dimension."""
    zl = _zl()
    rng = np.random.default_rng(M + N + K)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    a_k = layout in ("nt", "nn")
    b_k = layout == "nt"
    A = rng.standard_normal((M, K) if a_k else (K, M)).astype(np.float32)
    B = rng.standard_normal((N, K) if b_k else (K, N)).astype(np.float32)
    At = torch.tensor(A, device=_dev()).to(tdt)
    Bt = torch.tensor(B, device=_dev()).to(tdt)
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device=_dev())
    torch.cuda.synchronize()
    zl.zl_kernel_gemm(M, N, K, At.data_ptr(), At.shape[1], a_k, Bt.data_ptr(), Bt.shape[1], b_k,
                      C.data_ptr(), N, zl.ZL_BF16 if dtype == "bf16" else zl.ZL_F32, _stream())
    torch.cuda.synchronize()
    a64 = At.double().cpu().numpy()
    b64 = Bt.double().cpu().numpy()
    ref = (a64 if a_k else a64.T) @ (b64 if b_k else b64.T).T
    got = C.cpu().double().numpy()
    assert np.all(np.isfinite(got))
    bound = 1e-5 * np.sqrt(K) * (np.abs(a64).max() * np.abs(b64).max()) + 1e-6
    assert np.max(np.abs(got - ref)) < bound * 8
    assert rel_err(got, ref) < 2e-6


def _gemm_operands(rng, layout, M, N, K, tdt):
    a_k = layout in ("nt", "nn")
    b_k = layout == "nt"
    A = rng.standard_normal((M, K) if a_k else (K, M)).astype(np.float32)
    B = rng.standard_normal((N, K) if b_k else (K, N)).astype(np.float32)
    return (torch.tensor(A, device=_dev()).to(tdt), torch.tensor(B, device=_dev()).to(tdt), a_k, b_k)


def _gemm_ref(At, Bt, a_k, b_k):
    a64 = At.double().cpu().numpy()
    b64 = Bt.double().cpu().numpy()
    return (a64 if a_k else a64.T) @ (b64 if b_k else b64.T).T


@pytest.mark.parametrize("dtype,layout,M,N,K,K2", [
    (dt, lay, M, N, K, K2) for dt in ("bf16", "f32") for lay in ("nt", "nn", "tn")
    for M, N, K, K2 in ((304, 520, 200, 8), (4096, 3848, 264, 48), (512, 768, 4096, 16),
                        (136, 64, 8, 200))
    if not (dt == "f32" and M * N * (K + K2) > 1e9)])
def test_gemm_second_segment(dtype, layout, M, N, K, K2):
    """C = A B^T + A2 B2^T with the second pair in the layouts of the first
    (the low-rank term of a LoRA projection), ragged in every dimension."""
    zl = _zl()
    rng = np.random.default_rng(M + N + K + K2)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    At, Bt, a_k, b_k = _gemm_operands(rng, layout, M, N, K, tdt)
    A2, B2, _, _ = _gemm_operands(rng, layout, M, N, K2, tdt)
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device=_dev())
    torch.cuda.synchronize()
    zl.zl_kernel_gemm(M, N, K, At.data_ptr(), At.shape[1], a_k, Bt.data_ptr(), Bt.shape[1], b_k,
                      C.data_ptr(), N, zl.ZL_BF16 if dtype == "bf16" else zl.ZL_F32, _stream(),
                      K2=K2, A2=A2.data_ptr(), lda2=A2.shape[1], B2=B2.data_ptr(), ldb2=B2.shape[1])
    torch.cuda.synchronize()
    ref = _gemm_ref(At, Bt, a_k, b_k) + _gemm_ref(A2, B2, a_k, b_k)
    got = C.cpu().double().numpy()
    assert np.all(np.isfinite(got))
    assert rel_err(got, ref) < 2e-6


@pytest.mark.parametrize("a_k,b_k", [(True, True), (True, False), (False, False), (False, True)])
@pytest.mark.parametrize("M,N,K,K2", [(16, 4104, 16384, 0), (4096, 16, 16384, 16), (200, 136, 3000, 24),
                                      (48, 1000, 1024, 0)])
def test_gemm_split_k(a_k, b_k, M, N, K, K2):
    """Outputs of too few tiles to fill the GPU (the LoRA factor GEMMs) split
    K into fp32 partials in the caller's workspace: same result as one pass
    within fp32 summation error, identical on a repeat (fixed summation
    order), and still correct when the workspace only holds two partials."""
    zl = _zl()
    rng = np.random.default_rng(M + N + K + K2 + 2 * a_k + b_k)

    def op(rows, k, kmaj):
        x = rng.standard_normal((rows, k) if kmaj else (k, rows)).astype(np.float32)
        return torch.tensor(x, device=_dev()).to(torch.bfloat16)
    At, Bt = op(M, K, a_k), op(N, K, b_k)
    A2, B2 = (op(M, K2, a_k), op(N, K2, b_k)) if K2 else (None, None)
    seg = dict(K2=K2, A2=A2.data_ptr(), lda2=A2.shape[1], B2=B2.data_ptr(), ldb2=B2.shape[1]) if K2 else {}

    def run(ws_elems):
        C = torch.full((M, N), float("nan"), dtype=torch.float32, device=_dev())
        ws = torch.full((max(ws_elems, 1),), float("nan"), dtype=torch.float32, device=_dev())
        torch.cuda.synchronize()
        zl.zl_kernel_gemm(M, N, K, At.data_ptr(), At.shape[1], a_k, Bt.data_ptr(), Bt.shape[1], b_k,
                          C.data_ptr(), N, zl.ZL_BF16, _stream(), workspace=ws.data_ptr() if ws_elems else None,
                          workspace_elems=ws_elems, **seg)
        torch.cuda.synchronize()
        return C.cpu().double().numpy()
    ref = _gemm_ref(At, Bt, a_k, b_k) + (_gemm_ref(A2, B2, a_k, b_k) if K2 else 0.0)
    one = run(0)
    split = run(64 * M * N)
    again = run(64 * M * N)
    two = run(2 * M * N)
    for got in (one, split, two):
        assert np.all(np.isfinite(got))
        assert rel_err(got, ref) < 2e-6
    assert np.array_equal(split, again)


@pytest.mark.parametrize("a_k,b_k", [(True, False), (True, True)])
def test_gemm_long_k_large_tiles_split(a_k, b_k):
    """A long reduction over few large tiles (the head's data gradient, K = V
    with rows x d small: here 2048 x 1024 x 65536, 32 tiles of 256 x 256)
    runs as large tiles split eight ways over K: sampled rows against fp64,
    the whole output against the unsplit launch, identical on a repeat."""
    zl = _zl()
    M, N, K = 2048, 1024, 65536
    gen = torch.Generator(device=_dev()).manual_seed(5)
    At = torch.randn((M, K) if a_k else (K, M), device=_dev(), generator=gen).to(torch.bfloat16)
    Bt = torch.randn((N, K) if b_k else (K, N), device=_dev(), generator=gen).to(torch.bfloat16)

    def run(ws_elems):
        C = torch.full((M, N), float("nan"), dtype=torch.float32, device=_dev())
        ws = torch.full((max(ws_elems, 1),), float("nan"), dtype=torch.float32, device=_dev())
        torch.cuda.synchronize()
        zl.zl_kernel_gemm(M, N, K, At.data_ptr(), At.shape[1], a_k, Bt.data_ptr(), Bt.shape[1], b_k,
                          C.data_ptr(), N, zl.ZL_BF16, _stream(),
                          workspace=ws.data_ptr() if ws_elems else None, workspace_elems=ws_elems)
        torch.cuda.synchronize()
        return C
    one = run(0)
    split = run(8 * M * N)
    again = run(8 * M * N)
    assert bool(torch.isfinite(split).all())
    assert torch.equal(split, again)
    assert rel_err(split.cpu().double().numpy(), one.cpu().double().numpy()) < 2e-6
    rows = np.random.default_rng(3).choice(M, size=48, replace=False)
    ridx = torch.tensor(rows, device=_dev())
    a = (At[ridx] if a_k else At[:, ridx].t()).double().cpu().numpy()
    b = (Bt if b_k else Bt.t()).double().cpu().numpy()
    ref = a @ b.T
    assert rel_err(split[ridx].cpu().double().numpy(), ref) < 2e-6


def test_gemm_register_staged_path_with_second_segment():
    """Both operands MN-major with A's row stride 16384 and K = 66000: A's
    tile offsets pass 2^31 bytes, so the direct-to-LDS kernel is not used and
    the register-staged MFMA kernel computes C = A B^T + A2 B2^T."""
    zl = _zl()
    M, N, K, K2, lda = 256, 256, 66000, 16, 16384
    rng = np.random.default_rng(5)
    A = torch.zeros((K, lda), dtype=torch.bfloat16, device=_dev())
    A[:, :M] = torch.tensor(rng.standard_normal((K, M)).astype(np.float32), device=_dev()).to(torch.bfloat16)
    Bt = torch.tensor(rng.standard_normal((K, N)).astype(np.float32), device=_dev()).to(torch.bfloat16)
    A2 = torch.tensor(rng.standard_normal((K2, M)).astype(np.float32), device=_dev()).to(torch.bfloat16)
    B2 = torch.tensor(rng.standard_normal((K2, N)).astype(np.float32), device=_dev()).to(torch.bfloat16)
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device=_dev())
    torch.cuda.synchronize()
    zl.zl_kernel_gemm(M, N, K, A.data_ptr(), lda, False, Bt.data_ptr(), N, False, C.data_ptr(), N,
                      zl.ZL_BF16, _stream(), K2=K2, A2=A2.data_ptr(), lda2=M, B2=B2.data_ptr(),
                      ldb2=N)
    torch.cuda.synchronize()
    ref = _gemm_ref(A[:, :M], Bt, False, False) + _gemm_ref(A2, B2, False, False)
    del A
    got = C.cpu().double().numpy()
    assert np.all(np.isfinite(got))
    assert rel_err(got, ref) < 2e-6


def _attn_inputs(B, S, Hq, Hkv, hd, lens, seed):
    rng = np.random.default_rng(seed)
    q = rng.standard_normal((B, S, Hq, hd)).astype(np.float32)
    k = rng.standard_normal((B, S, Hkv, hd)).astype(np.float32)
    v = rng.standard_normal((B, S, Hkv, hd)).astype(np.float32)
    do = rng.standard_normal((B, S, Hq, hd)).astype(np.float32)
    return q, k, v, do, np.array(lens, np.int32)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,S,Hq,Hkv,hd,lens", [
    (2, 37, 4, 2, 16, [37, 20]),
    (1, 130, 8, 2, 64, [130]),
    (2, 200, 4, 4, 128, [200, 77]),
    (1, 300, 4, 1, 128, [300]),
    (1, 5, 2, 1, 64, [0]),
    (3, 64, 2, 2, 32, [1, 64, 63]),
])
def test_attention_fwd_bwd(dtype, B, S, Hq, Hkv, hd, lens):
    zl = _zl()
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v, do, lens = _attn_inputs(B, S, Hq, Hkv, hd, lens, S + hd)
    ld = (Hq + 2 * Hkv) * hd
    qkv = np.concatenate([q.reshape(B * S, -1), k.reshape(B * S, -1), v.reshape(B * S, -1)], 1)
    QKV = torch.tensor(qkv, device=_dev()).to(tdt).contiguous()
    DO = torch.tensor(do.reshape(B * S, -1), device=_dev()).to(tdt)
    O = torch.zeros(B * S, Hq * hd, device=_dev(), dtype=tdt)
    LSE = torch.zeros(B, Hq, S, dtype=torch.float32, device=_dev())
    DQKV = torch.zeros_like(QKV)
    DEL = torch.zeros(B, Hq, S, dtype=torch.float32, device=_dev())
    SL = torch.tensor(lens, device=_dev())
    base = QKV.data_ptr()
    esz = QKV.element_size()
    torch.cuda.synchronize()
    args = (B, S, Hq, Hkv, hd, base, base + Hq * hd * esz, base + (Hq + Hkv) * hd * esz, ld,
            SL.data_ptr(), O.data_ptr(), LSE.data_ptr())
    dt = zl.ZL_BF16 if dtype == "bf16" else zl.ZL_F32
    zl.zl_kernel_attention(*args, 0, 0, 0, 0, 0, dt, 0, _stream())
    dbase = DQKV.data_ptr()
    zl.zl_kernel_attention(*args, DO.data_ptr(), dbase, dbase + Hq * hd * esz,
                           dbase + (Hq + Hkv) * hd * esz, DEL.data_ptr(), dt, 1, _stream())
    torch.cuda.synchronize()
    r = QKV.double().cpu().numpy()
    q64 = r[:, : Hq * hd].reshape(B, S, Hq, hd)
    k64 = r[:, Hq * hd: (Hq + Hkv) * hd].reshape(B, S, Hkv, hd)
    v64 = r[:, (Hq + Hkv) * hd:].reshape(B, S, Hkv, hd)
    do64 = DO.double().cpu().numpy().reshape(B, S, Hq, hd)
    o_ref, cache = ops.attention_fwd(q64, k64, v64, lens)
    dq_ref, dk_ref, dv_ref = ops.attention_bwd(do64, cache)
    tol = 1e-5 if dtype == "f32" else 1.2e-2
    o = O.double().cpu().numpy().reshape(B, S, Hq, hd)
    assert rel_err(o, o_ref) < tol
    d = DQKV.double().cpu().numpy()
    assert rel_err(d[:, : Hq * hd].reshape(dq_ref.shape), dq_ref) < tol
    assert rel_err(d[:, Hq * hd: (Hq + Hkv) * hd].reshape(dk_ref.shape), dk_ref) < tol
    assert rel_err(d[:, (Hq + Hkv) * hd:].reshape(dv_ref.shape), dv_ref) < tol
    # lse of rows with at least one visible key
    lse = LSE.cpu().double().numpy()
    scale = 1.0 / np.sqrt(hd)
    for b in range(B):
        for h in range(Hq):
            g = h // (Hq // Hkv)
            s = (q64[b, :, h] @ k64[b, :, g].T) * scale
            allowed = ops.attention_mask(B, S, lens)[b]
            for i in range(S):
                if allowed[i].any():
                    ref = np.log(np.sum(np.exp(s[i][allowed[i]] - s[i][allowed[i]].max()))) + s[i][allowed[i]].max()
                    assert abs(lse[b, h, i] - ref) < 1e-4 * max(1, abs(ref))
                else:
                    assert lse[b, h, i] == -np.inf


def _backward_profile(shp):
    import workload
    from tests.gpu_cases import make_inputs, device_chunk, to_dev
    zl = _zl()
    params, batch = make_inputs(shp, seed=3)
    ch = device_chunk(shp, params, batch)
    d = to_dev(batch, shp.dtype)
    ch.forward(d["h_in"], d["seq_lens"], d["pos_ids"])
    ch.objective(d["labels"])
    torch.cuda.synchronize()
    zl.zl_profile_begin(ch.handle, 4096)
    ch.backward(1.0, 0)
    torch.cuda.synchronize()
    prof = zl.zl_profile_end(ch.handle, 256)
    ch.close()
    return [e for e in prof if e["name"].endswith("_mn")]


def test_backward_pairs_weight_gradients():
    """The weight-gradient GEMMs of an 8B-shaped layer run as two launches,
    down with QKV and up with the output projection (their tiles fill whole
    waves together), each carrying the FLOPs of both; a 1B-shaped layer's
    QKV and output projections have too few tiles to pair and run alone."""
    import workload
    shp = workload.get_config("8b").with_(n_layers=1, batch=1, seq=256)
    T, d, ff = 256, shp.d_model, shp.d_ff
    nqkv = (shp.n_heads + 2 * shp.n_kv_heads) * shp.head_dim
    mn = _backward_profile(shp)
    assert [e["name"] for e in mn] == ["gemm_dma_256x256_mn"]
    assert mn[0]["launches"] == 2
    want = 2.0 * T * (d * ff + 2 * ff * d + d * shp.n_heads * shp.head_dim + nqkv * d)
    assert mn[0]["flops"] == pytest.approx(want, rel=1e-9)
    shp1 = workload.get_config("1b").with_(n_layers=1, batch=1, seq=512)
    launches = sum(e["launches"] for e in _backward_profile(shp1))
    assert launches == 4


@pytest.mark.parametrize("pad", [0, 24])
@pytest.mark.parametrize("b_k", [True, False])
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (16, 16, 128), (17, 24, 1032), (1000, 40, 2048), (300, 64, 136),
                                   (8200, 8, 520), (8200, 32, 264)])
def test_gemm_few_columns(b_k, M, N, K, pad):
    """At most 64 output columns over a K-major A (the LoRA products): rows
    past a block's 16 or 32, columns past 16 or 32, K past the waves' 128-wide
    slices, all against fp64 within fp32 summation error; dense rows, and rows
    of a wider matrix (as the chunk's, whose operands lie beside each other)
    whose other columns are neither read into the product nor written."""
    from tests.gemm_route import skinny
    assert skinny(M, N, K, b_k, 0)
    zl = _zl()
    gen = torch.Generator(device=_dev()).manual_seed(M + N + K)

    def op(rows, cols):
        x = torch.full((rows, cols + pad), float("nan"), device=_dev(), dtype=torch.bfloat16)
        x[:, :cols] = torch.randn(rows, cols, device=_dev(), generator=gen).to(torch.bfloat16)
        return x
    A, B = op(M, K), op(*((N, K) if b_k else (K, N)))
    C = torch.full((M + 1, N + pad), float("nan"), dtype=torch.float32, device=_dev())
    torch.cuda.synchronize()
    zl.zl_kernel_gemm(M, N, K, A.data_ptr(), K + pad, True, B.data_ptr(), B.shape[1], b_k, C.data_ptr(), N + pad,
                      zl.ZL_BF16, _stream())
    torch.cuda.synchronize()
    A, B = A[:, :K].double().cpu(), B[:, :K if b_k else N].double().cpu()
    ref = A @ (B.t() if b_k else B)
    assert bool(torch.isnan(C[M]).all())  # nothing written past the last row
    assert bool(torch.isnan(C[:, N:]).all())
    assert rel_err(C[:M, :N].cpu().double().numpy(), ref.numpy()) < 2e-6


@pytest.mark.parametrize("arch,rank,B,S", [("1b", 4, 1, 37), ("1b", 16, 3, 700), ("1b", 24, 2, 65), ("gpt2", 8, 5, 203)])
def test_lora_factor_gradients(arch, rank, B, S):
    """Factor gradients of one LoRA layer, dB = dy^T xa and dA = E^T x with
    xa = s x A^T and E = s dy B rounded to bf16 as stored, from the chunk's own
    operands in fp64: token counts that are no multiple of a slice, split rows
    (2100), three or two factors beside each other, and a rank whose stacked
    QKV factors are too wide for the low-rank kernel (3 x 24 > 64).  The
    recomputed operands may round differently where fp32 sums differ, half a
    bf16 unit (2^-9) on few entries."""
    import workload
    from paper_2608_07974_amd.chunk import TorchChunk, config_from_shape
    shp = workload.get_config(arch).with_(n_layers=1, batch=B, seq=S, lora_rank=rank)
    cfg = config_from_shape(shp, alpha=1.0, optimizer="sgd")
    ch = TorchChunk(cfg)
    gen = torch.Generator(device=_dev()).manual_seed(rank + S)
    ch.master.normal_(0.0, 0.02, generator=gen)
    ch.base_master.normal_(0.0, 0.02, generator=gen)
    ch.head_w.normal_(0.0, 0.02, generator=gen)
    zl = _zl()
    zl.zl_refresh_shadow(ch.handle, _stream())
    h = torch.randn(B, S, shp.d_model, device=_dev(), generator=gen).to(torch.bfloat16)
    lab = torch.randint(0, shp.vocab, (B, S), device=_dev(), generator=gen).to(torch.int32)
    ch.forward(h)
    ch.objective(lab)
    ch.backward(1.0, 0)
    s = cfg.lora_alpha / rank
    llama = arch != "gpt2"
    q, kv = shp.n_heads * shp.head_dim, shp.n_kv_heads * shp.head_dim
    groups = [("n2", "dup", ["wg", "wu"] if llama else ["wfc"], [shp.d_ff] * (2 if llama else 1)),
              ("act", "dxa", ["wd"] if llama else ["wproj"], [shp.d_model]),
              ("o", "dxb", ["wo"], [shp.d_model]),
              ("n1", "dqkv", ["wq", "wk", "wv"] if llama else ["wqkv"], [q, kv, kv] if llama else [q + 2 * kv])]
    for xn, dyn, names, widths in groups:
        x, dy = ch.inspect_device(xn).double(), ch.inspect_device(dyn).double()
        col = 0
        for name, w in zip(names, widths):
            a = ch.view(ch.shadow, f"L0.{name}_la").double()
            b = ch.view(ch.shadow, f"L0.{name}_lb").double()
            d = dy[:, col: col + w]
            xa = (s * (x @ a.t())).to(torch.bfloat16).double()
            e = (s * (d @ b)).to(torch.bfloat16).double()
            for key, ref in ((f"L0.{name}_lb", d.t() @ xa), (f"L0.{name}_la", e.t() @ x)):
                got = ch.view(ch.grad, key).double()
                assert bool(torch.isfinite(got).all()), key
                assert float((got - ref).norm() / ref.norm()) < 1e-3, key
            col += w
    ch.close()


@pytest.mark.parametrize("M,N,K,K2", [(2050, 1030, 24, 0), (1000, 3000, 5, 16), (1536, 4200, 40, 0), (777, 1100, 129, 0)])
@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
def test_gemm_f32_tiles(layout, M, N, K, K2):
    """fp32 products of many tiles: the 64 x 64 tiles (short K, a second
    segment, rows and columns past the last tile) and, the last shape, the
    32 x 32 ones with one k past a tile of 128."""
    from tests.gemm_route import f32_large
    zl = _zl()
    rng = np.random.default_rng(M + N + K)
    At, Bt, a_k, b_k = _gemm_operands(rng, layout, M, N, K, torch.float32)
    A2, B2, _, _ = _gemm_operands(rng, layout, M, N, K2, torch.float32)
    assert f32_large(M, N, K + K2, a_k, b_k) == (K < 100)
    C = torch.full((M + 1, N), float("nan"), device=_dev())
    torch.cuda.synchronize()
    seg = dict(K2=K2, A2=A2.data_ptr(), lda2=A2.shape[1], B2=B2.data_ptr(), ldb2=B2.shape[1]) if K2 else {}
    zl.zl_kernel_gemm(M, N, K, At.data_ptr(), At.shape[1], a_k, Bt.data_ptr(), Bt.shape[1], b_k, C.data_ptr(), N,
                      zl.ZL_F32, _stream(), **seg)
    torch.cuda.synchronize()
    ref = _gemm_ref(At, Bt, a_k, b_k) + (_gemm_ref(A2, B2, a_k, b_k) if K2 else 0.0)
    assert bool(torch.isnan(C[M]).all())
    assert rel_err(C[:M].cpu().double().numpy(), ref) < 2e-6


@pytest.mark.parametrize("arch", ["llama", "gpt2"])
@pytest.mark.parametrize("T", [4104, 8216, 16400, 40000])
def test_norm_and_bias_gradients_of_many_rows(arch, T):
    """Column sums over 512 partial rows (one stage of the reduction), 513 and
    1025 (two stages, the last group one row) and 2048 (blocks without rows
    among them): the norm gradients, and with a LayerNorm the bias
    gradients taken from the norm backward, against fp64 sums of the chunk's
    own operands.  Bound: each sum is at most 20 rows in a block, then trees,
    with a few roundings per term: under 64 units of fp32 of the absolute sum."""
    import workload
    from paper_2608_07974_amd.chunk import TorchChunk, config_from_shape
    zl = _zl()
    shp = workload.get_config("tiny").with_(arch=arch, d_ff=64, vocab=64, batch=T // 8, seq=8)
    ch = TorchChunk(config_from_shape(shp, alpha=1.0, optimizer="sgd"))
    gen = torch.Generator(device=_dev()).manual_seed(T)
    ch.master.normal_(0.0, 0.1, generator=gen)
    ch.head_w.normal_(0.0, 0.1, generator=gen)
    zl.zl_refresh_shadow(ch.handle, _stream())
    h = torch.randn(T // 8, 8, 64, device=_dev(), generator=gen)
    ch.forward(h)
    ch.objective(torch.randint(0, 64, (T // 8, 8), device=_dev(), generator=gen).to(torch.int32))
    ch.backward(1.0, 0)
    x, dn = ch.inspect_device("x", 0).double(), ch.inspect_device("dn").double()
    if arch == "gpt2":
        x = x - x.mean(1, keepdim=True)
    xhat = x * ch.inspect_device("rstd1", 0).double()
    want = {"L0.ln1_w": dn * xhat}
    if arch == "gpt2":
        want.update({"L0.ln1_b": dn, "L0.bo": ch.inspect_device("dxb").double(),
                     "L0.bproj": ch.inspect_device("dxa").double()})
    for key, terms in want.items():
        got = ch.view(ch.grad, key).double().reshape(-1)
        size = terms.abs().sum(0)
        assert bool((size > 0).all()), key
        assert bool(((got - terms.sum(0)).abs() <= 64 * 2.0 ** -24 * size).all()), key
    ch.close()


# Shape, sequences of 50 tokens, and what the projections take by their sizes:
# (columns of a wave tile, splits of K) of the QKV projection with RoPE and of the
# output projection's data gradient with delta.
_HEAD_CASES = [("1b", 4, "split", "split"), ("1b", 22, "64", "64"), ("8b", 4, "split", "split"),
               ("8b", 12, "128", "128"), ("8b", 60, "128", "large"), ("16", 22, "64", None), ("32", 22, "64", None)]


@pytest.mark.parametrize("name,B,qkv,delta", _HEAD_CASES)
def test_rotation_and_delta_epilogues_by_route(name, B, qkv, delta):
    """One layer's q|k|v after the rotation, dO, and through delta dq|dk|dv, from
    the chunk's own operands in fp64, on each kernel that can carry the
    epilogue: 128 x 128 tiles with 64- and 128-column wave tiles, their last rows
    partial (200, 600, 1100 and 3000 are no multiples of 32 or 128), the sum of
    split K, and 256 x 256 tiles.  q|k|v and dO: half a unit of bf16 of the value,
    plus fp32 sums of K terms (2^-18 of the sum of absolute products).  dq|dk|dv
    per head: the tolerance of the attention kernels; rows are short (50), so
    that delta is a large part of dq and dk."""
    import workload
    from paper_2608_07974_amd.chunk import TorchChunk, config_from_shape
    from tests.gemm_route import TILE_128, TILE_128_WIDE, TILE_256, route
    zl = _zl()
    base = dict(n_layers=1, batch=B, seq=50, vocab=512, d_ff=512)
    shp = workload.get_config(name).with_(**base) if name in ("1b", "8b") else workload.get_config("1b").with_(
        d_model=512, n_heads=512 // int(name), n_kv_heads=128 // int(name), head_dim=int(name), **base)
    T, d, hd, hq, hkv = 50 * B, shp.d_model, shp.head_dim, shp.n_heads, shp.n_kv_heads
    dq, nqkv = hq * hd, (hq + 2 * hkv) * hd
    for want, r in ((qkv, route(T, nqkv, d, 1, 1, heads=True, hd=hd)), (delta, route(T, dq, d, 1, 0, heads=True, hd=hd))):
        if want:
            got = "split" if r["nz"] > 1 else {TILE_128: "64", TILE_128_WIDE: "128", TILE_256: "large"}[r["tile"]]
            assert got == want, r
    ch = TorchChunk(config_from_shape(shp, alpha=1.0, optimizer="sgd"))
    gen = torch.Generator(device=_dev()).manual_seed(B + d)
    ch.master.normal_(0.0, 0.03, generator=gen)
    ch.head_w.normal_(0.0, 0.02, generator=gen)
    zl.zl_refresh_shadow(ch.handle, _stream())
    h = torch.randn(B, 50, d, device=_dev(), generator=gen).to(torch.bfloat16)
    ch.forward(h)
    ch.objective(torch.randint(0, 512, (B, 50), device=_dev(), generator=gen).to(torch.int32))
    ch.backward(1.0, 0)
    w = torch.cat([ch.view(ch.shadow, "L0." + n).double() for n in ("wq", "wk", "wv")])
    ang = torch.arange(50, device=_dev()).double()[:, None] * float(np.float32(shp.rope_theta)) ** (
        -torch.arange(hd // 2, device=_dev()).double() / (hd // 2))
    cs = torch.cat([ang.cos().float().double()] * 2, 1).repeat(B, 1)[:, None, :]  # [T, 1, hd]
    sn = torch.cat([-ang.sin().float().double(), ang.sin().float().double()], 1).repeat(B, 1)[:, None, :]

    def rotate(x, sign=1.0):  # the q and k heads of [T, nqkv]
        y = x.reshape(T, -1, hd).clone()
        r = y[:, : hq + hkv]
        y[:, : hq + hkv] = r * cs + sign * torch.roll(r, hd // 2, 2) * sn
        return y.reshape(T, -1)

    def close(got, ref, size):
        bad = (got - ref).abs() > 2.0 ** -8 * ref.abs() + 2.0 ** -18 * size
        assert not bool(bad.any()), (int(bad.sum()), bad.nonzero()[:4].tolist())
    n1 = ch.inspect_device("n1").double()
    size = (n1.abs() @ w.abs().t()).reshape(T, -1, hd)
    got = ch.inspect_device("qkv").double()
    close(got, rotate(n1 @ w.t()), (size + torch.roll(size, hd // 2, 2)).reshape(T, -1))
    dxb, wo = ch.inspect_device("dxb").double(), ch.view(ch.shadow, "L0.wo").double()
    do = ch.inspect_device("do").double()
    close(do, dxb @ wo, dxb.abs() @ wo.abs())
    q, k, v = (x.cpu().numpy().reshape(B, 50, -1, hd) for x in got.split([dq, hkv * hd, hkv * hd], 1))
    _, cache = ops.attention_fwd(q, k, v, np.full(B, 50, np.int32))
    ref = [torch.tensor(x.reshape(T, -1)).to(_dev()) for x in ops.attention_bwd(do.cpu().numpy().reshape(B, 50, hq, hd), cache)]
    ref = rotate(torch.cat(ref, 1), -1.0).reshape(T, -1, hd)
    err = ch.inspect_device("dqkv").double().reshape(T, -1, hd) - ref
    rel = err.pow(2).sum((0, 2)).sqrt() / ref.pow(2).sum((0, 2)).sqrt()
    assert float(rel.max()) < 1.2e-2, rel
    ch.close()
