"""Parity of the bf16 MFMA GEMM (layup_gemm_bf16) and the float32 GEMM with
float64 products of the same (bf16-valued) inputs: the dX = dY W and
dW = dY^T X products of the linear layers' backward (Algorithm 1, backward
pass at one layer), the forward product and the batched attention products.
Tolerance: rel 2e-2 for bf16-input GEMMs (float32 output is additionally held
to 1e-4 normwise)."""
import ctypes
import math

import numpy as np
import pytest

from paper_2410_05985_amd import synthetic as S
import oracle as O
from tests.parity import compare

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
from paper_2410_05985_amd import layup as LU  # noqa: E402

DEV = "cuda"


def bf16_tensor(shape, seed, std=1.0):
    x = torch.from_numpy(S.normal(shape, seed, std)).to(torch.bfloat16)
    return x


def as_f64(t):
    return t.float().cpu().numpy().astype(np.float64)


def run(layout, M, N, K, out_f32=True, bias=False, seed=0, ws=False):
    """layout: 'kk' (C = A B^T, forward), 'kn' (C = A B, dX), 'mn' (C = A^T B, dW)."""
    ak, bk = {"kk": (True, True), "kn": (True, False), "mn": (False, False)}[layout]
    A = bf16_tensor((M, K) if ak else (K, M), seed)
    B = bf16_tensor((N, K) if bk else (K, N), seed + 1)
    a64, b64 = as_f64(A), as_f64(B)
    ref = (a64 if ak else a64.T) @ (b64.T if bk else b64)
    bvec = None
    if bias:
        bvec = torch.from_numpy(S.normal((N,), seed + 2)).to(DEV)
        ref = ref + bvec.cpu().numpy().astype(np.float64)
    Ad, Bd = A.to(DEV), B.to(DEV)
    Cd = torch.empty((M, N), dtype=torch.float32 if out_f32 else torch.bfloat16, device=DEV)
    w = torch.empty(64 << 20, dtype=torch.uint8, device=DEV) if ws else None
    d = LU.gemm_desc(Ad, Bd, Cd, M, N, K, K if ak else M, K if bk else N, N, ak, bk, out_f32,
                     bias=bvec, workspace=w, workspace_bytes=(64 << 20) if ws else 0)
    LU.layup_gemm_bf16(d, torch.cuda.current_stream())
    torch.cuda.synchronize()
    return Cd.float().cpu().numpy().astype(np.float64), ref


@pytest.mark.parametrize("layout", ["kk", "kn", "mn"])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (128, 128, 128), (256, 384, 192),
                                   (200, 136, 72), (1000, 520, 264), (8, 8, 8), (40, 24, 8),
                                   (128, 64, 1000)])
def test_gemm_layouts_and_ragged_shapes(layout, M, N, K):
    got, ref = run(layout, M, N, K, out_f32=True, seed=M + N + K)
    compare(got, ref, 2e-2, f"{layout} {M}x{N}x{K}")
    assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)


@pytest.mark.parametrize("layout", ["kk", "kn", "mn"])
def test_gemm_bf16_output_and_bias(layout):
    got, ref = run(layout, 320, 192, 136, out_f32=False, bias=True, seed=5)
    compare(got, ref, 2e-2, "bf16 out")
    # a bf16 result is the float32 result rounded once: within half a bf16 ulp
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-3 * np.sqrt(np.mean(ref ** 2)))


@pytest.mark.parametrize("layout", ["mn", "kn"])
def test_gemm_split_k_deterministic(layout):
    """Few output tiles and a long K take the split-K path: float32 partials
    summed in a fixed order -- the result is reproducible bit for bit."""
    a, ref = run(layout, 256, 256, 8192, ws=True, seed=11)
    b, _ = run(layout, 256, 256, 8192, ws=True, seed=11)
    compare(a, ref, 2e-2, "split-K")
    assert np.linalg.norm(a - ref) <= 1e-4 * np.linalg.norm(ref)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("layout", ["kn", "kk"])
def test_gemm_long_k_split(layout):
    """K >= 16384 with a float32 output (as the tied head's dX over the
    vocabulary): a split of K, ragged M, N and K, reproducible bit for bit."""
    a, ref = run(layout, 520, 264, 16400, ws=True, seed=13)
    b, _ = run(layout, 520, 264, 16400, ws=True, seed=13)
    compare(a, ref, 2e-2, "long-K split")
    assert np.linalg.norm(a - ref) <= 1e-4 * np.linalg.norm(ref)
    assert np.array_equal(a, b)


def test_gemm_split_k_unaligned_columns():
    """Split-K whose output rows are not a multiple of four floats (N = 130,
    k-major B): the partial sums take the per-column path, with the bias;
    reproducible bit for bit."""
    a, ref = run("kk", 200, 130, 16400, bias=True, ws=True, seed=19)
    b, _ = run("kk", 200, 130, 16400, bias=True, ws=True, seed=19)
    compare(a, ref, 2e-2, "split-K N=130")
    assert np.linalg.norm(a - ref) <= 1e-4 * np.linalg.norm(ref)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("layout", ["kk", "kn", "mn"])
def test_gemm_degenerate_sizes(layout):
    """K = 0: C = bias (float32 and bf16 outputs, and the float32 GEMM), the
    row sums of A are 0, and the operands, never read, may be NULL.  M = 0 or
    N = 0: nothing is written."""
    ak, bk = {"kk": (True, True), "kn": (True, False), "mn": (False, False)}[layout]
    M, N = 72, 40
    bvec = torch.from_numpy(S.normal((N,), 3)).to(DEV)
    lda, ldb = (0 if ak else M), (0 if bk else N)
    s = torch.cuda.current_stream()
    for f32 in (True, False):
        C = torch.full((M, N), float("nan"), dtype=torch.float32 if f32 else torch.bfloat16, device=DEV)
        rs = torch.full((M,), float("nan"), dtype=torch.float32, device=DEV) if not ak else None
        d = LU.gemm_desc(None, None, C, M, N, 0, lda, ldb, N, ak, bk, f32, bias=bvec, a_rowsum=rs)
        LU.layup_gemm_bf16(d, s)
        torch.cuda.synchronize()
        want = bvec if f32 else bvec.to(torch.bfloat16)
        assert torch.equal(C, want.expand(M, N)), f32
        if rs is not None:
            assert torch.equal(rs, torch.zeros_like(rs))
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device=DEV)
    LU.layup_gemm_f32(LU.gemm_desc(None, None, C, M, N, 0, lda, ldb, N, ak, bk, True, bias=bvec), s)
    torch.cuda.synchronize()
    assert torch.equal(C, bvec.expand(M, N))
    # M = 0 or N = 0: a sentinel output is left as it is
    A = bf16_tensor((M, 64) if ak else (64, M), 5).to(DEV)
    B = bf16_tensor((N, 64) if bk else (64, N), 6).to(DEV)
    sentinel = torch.full((M, N), 7.0, dtype=torch.float32, device=DEV)
    for m_, n_ in ((0, N), (M, 0)):
        d = LU.gemm_desc(A, B, sentinel, m_, n_, 64, 64 if ak else max(m_, 8), 64 if bk else max(n_, 8),
                         max(n_, 8), ak, bk, True)
        LU.layup_gemm_bf16(d, s)
    torch.cuda.synchronize()
    assert torch.equal(sentinel, torch.full_like(sentinel, 7.0))


def test_gemm_dw_many_tiles():
    """dW = dY^T X with more output tiles than CUs (as the head's dW); ragged N
    and K."""
    got, ref = run("mn", 4096, 2200, 200, seed=17)
    compare(got, ref, 2e-2, "dW many tiles")
    assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)


@pytest.mark.parametrize("M,N,K,ws", [(256, 384, 192, False), (200, 136, 72, False),
                                      (256, 256, 8192, True), (520, 264, 3000, True),
                                      (2304, 768, 8192, True)])
def test_gemm_dw_bias_row_sums(M, N, K, ws):
    """dW = dY^T X with the bias gradient db = column sums of dY accumulated
    by the same kernel (a_rowsum), with and without split-K (ragged shapes):
    both against the oracle's linear-layer backward of the same bf16 values,
    db at 1e-4 (float32 sums of K terms)."""
    A = bf16_tensor((K, M), 41 + M, 0.5)   # dY, tokens x out
    B = bf16_tensor((K, N), 42 + N, 0.5)   # X, tokens x in
    dy, x = as_f64(A), as_f64(B)
    dw_ref, db_ref, _ = O.linear_bwd(dy, x, None, need_dx=False)
    Cd = torch.empty((M, N), dtype=torch.float32, device=DEV)
    db = torch.full((M,), float("nan"), dtype=torch.float32, device=DEV)
    w = torch.empty(64 << 20, dtype=torch.uint8, device=DEV) if ws else None
    d = LU.gemm_desc(A.to(DEV), B.to(DEV), Cd, M, N, K, M, N, N, False, False, True,
                     workspace=w, workspace_bytes=(64 << 20) if ws else 0, a_rowsum=db)
    LU.layup_gemm_bf16(d, torch.cuda.current_stream())
    torch.cuda.synchronize()
    compare(Cd.cpu().numpy(), dw_ref, 2e-2, f"dW {M}x{N}x{K}")
    compare(db.cpu().numpy(), db_ref, 1e-4, f"db {M}x{N}x{K}")


def test_gemm_row_sums_need_m_major_a():
    A = bf16_tensor((64, 64), 1).to(DEV)
    Cd = torch.empty((64, 64), dtype=torch.float32, device=DEV)
    db = torch.empty(64, dtype=torch.float32, device=DEV)
    d = LU.gemm_desc(A, A, Cd, 64, 64, 64, 64, 64, 64, True, False, True, a_rowsum=db)
    with pytest.raises(RuntimeError):
        LU.layup_gemm_bf16(d, torch.cuda.current_stream())


def test_gemm_batched_attention_strides():
    """Batched products over z = b*H + h with two-level operand offsets, as the
    attention core uses them: S_z = Q_h K_h^T from a packed qkv matrix."""
    B, T, H, dh = 2, 96, 3, 32
    d = H * dh
    qkv = bf16_tensor((B * T, 3 * d), 21)
    q64 = as_f64(qkv).reshape(B, T, 3, H, dh)
    ref = np.einsum("bihk,bjhk->bhij", q64[:, :, 0], q64[:, :, 1])
    dq = qkv.to(DEV)
    Sd = torch.empty((B, H, T, T), dtype=torch.float32, device=DEV)
    ptr = dq.data_ptr()
    d_ = LU.gemm_desc(ptr, ptr + 2 * d, Sd, T, T, dh, 3 * d, 3 * d, T, True, True, True,
                      batch=B * H, inner=H, a_strides=(T * 3 * d, dh), b_strides=(T * 3 * d, dh),
                      c_strides=(H * T * T, T * T))
    LU.layup_gemm_bf16(d_, torch.cuda.current_stream())
    torch.cuda.synchronize()
    compare(Sd.cpu().numpy(), ref, 2e-2, "batched scores")


@pytest.mark.parametrize("M,N,K,layout", [
    (8192, 768, 2304, "kn"),    # qkv dX, GPT-2-small
    (2304, 768, 8192, "mn"),    # qkv dW
    (8192, 3072, 768, "kn"),    # mlp-proj dX
    (768, 3072, 8192, "mn"),    # mlp-proj dW
    (768, 768, 8192, "mn"),     # attn-proj dW
    (8192, 2304, 768, "kk"),    # qkv forward
    (1024, 768, 50304, "kn"),   # head dX over the vocabulary (1024 of the 8192 rows)
    (50304, 768, 1024, "mn"),   # head dW (K = 1024 of the 8192 tokens)
    (8192, 1024, 4096, "kn"),   # GPT-2-medium fc dX
    (4096, 1024, 8192, "mn"),   # GPT-2-medium fc dW (split K)
    (8192, 8192, 2048, "kn"),   # 1.3B mlp-proj dX (256x256 tiles)
    (2048, 8192, 8192, "mn"),   # 1.3B mlp-proj dW (256x256 tiles, long K)
    (8192, 6144, 2048, "kk"),   # 1.3B qkv forward
])
def test_gemm_full_size_sampled(M, N, K, layout):
    """Full backward shapes of the GPT-2-small, GPT-2-medium and 1.3B blocks
    (8192 tokens), checked on 4096 sampled outputs, each an independent
    float64 dot product."""
    ak, bk = {"kk": (True, True), "kn": (True, False), "mn": (False, False)}[layout]
    A = bf16_tensor((M, K) if ak else (K, M), 31, 0.5)
    B = bf16_tensor((N, K) if bk else (K, N), 32, 0.5)
    Cd = torch.empty((M, N), dtype=torch.float32, device=DEV)
    w = torch.empty(64 << 20, dtype=torch.uint8, device=DEV)
    d = LU.gemm_desc(A.to(DEV), B.to(DEV), Cd, M, N, K, K if ak else M, K if bk else N, N, ak, bk,
                     True, workspace=w, workspace_bytes=64 << 20)
    LU.layup_gemm_bf16(d, torch.cuda.current_stream())
    torch.cuda.synchronize()
    rng = np.random.default_rng(M + N)
    mi, ni = rng.integers(0, M, 4096), rng.integers(0, N, 4096)
    a64, b64 = as_f64(A), as_f64(B)
    arows = a64[mi] if ak else a64[:, mi].T
    bcols = b64[ni] if bk else b64[:, ni].T
    ref = np.sum(arows * bcols, axis=1)
    got = Cd.cpu().numpy()[mi, ni].astype(np.float64)
    compare(got, ref, 2e-2, f"{M}x{N}x{K}")
    assert np.linalg.norm(got - ref) <= 1e-4 * np.linalg.norm(ref)


@pytest.mark.parametrize("layout", ["kk", "kn", "mn"])
def test_gemm_f32(layout):
    ak, bk = {"kk": (True, True), "kn": (True, False), "mn": (False, False)}[layout]
    M, N, K = 32, 10, 256
    A = S.normal((M, K) if ak else (K, M), 41)
    B = S.normal((N, K) if bk else (K, N), 42)
    ref = (A.astype(np.float64) if ak else A.T.astype(np.float64)) @ \
        (B.T.astype(np.float64) if bk else B.astype(np.float64))
    Cd = torch.empty((M, N), dtype=torch.float32, device=DEV)
    d = LU.gemm_desc(torch.from_numpy(A).to(DEV), torch.from_numpy(B).to(DEV), Cd, M, N, K,
                     K if ak else M, K if bk else N, N, ak, bk, True)
    LU.layup_gemm_f32(d, torch.cuda.current_stream())
    torch.cuda.synchronize()
    compare(Cd.cpu().numpy(), ref, 1e-5, "f32 gemm")


@pytest.mark.parametrize("ak,bk", [(True, True), (True, False), (False, False), (False, True)])
@pytest.mark.parametrize("M,N,K,ld", [(1, 1, 1, 0), (16, 16, 64, 0), (17, 33, 65, 0), (31, 15, 513, 3), (64, 48, 515, 4),
                                      (1040, 1000, 20, 1), (1100, 1010, 70, 0)])
def test_gemm_f32_tiles_and_remainders(ak, bk, M, N, K, ld):
    """Edges of the 16 x 16 and 32 x 32 tiles, of the K chunks of each wave
    and of the vector loads (leading dimensions off a multiple of four).
    Bound: a float32 sum of K products in any order is within (K + 1) 2^-24
    (first order; 1.01 for the rest) of the exact one, times the sum of
    their absolute values."""
    g = torch.Generator().manual_seed(M + 7 * N + 13 * K)
    A = torch.randn((M, K + ld) if ak else (K, M + ld), generator=g)
    B = torch.randn((N, K + ld) if bk else (K, N + ld), generator=g)
    a = (A[:, :K] if ak else A[:, :M].t()).double()
    b = (B[:, :K].t() if bk else B[:, :N]).double()
    Ad, Bd = A.to(DEV), B.to(DEV)
    C = torch.full((M, N), float("nan"), device=DEV)
    LU.layup_gemm_f32(LU.gemm_desc(Ad, Bd, C, M, N, K, A.shape[1], B.shape[1], N, ak, bk, True),
                      torch.cuda.current_stream())
    torch.cuda.synchronize()
    bound = 1.01 * (K + 1) * 2.0 ** -24 * (a.abs() @ b.abs())
    assert torch.all((C.cpu().double() - a @ b).abs() <= bound)


@pytest.mark.parametrize("ak,bk", [(True, True), (True, False), (False, False), (False, True)])
@pytest.mark.parametrize("M,N,K,ld", [(2048, 2048, 256, 0), (2052, 2044, 260, 4), (2049, 2051, 275, 1),
                                      (2044, 2050, 300, 2), (70000, 68, 257, 0), (64, 65600, 256, 0)])
def test_gemm_f32_large_tiles(ak, bk, M, N, K, ld):
    """The 64 x 64 tiles of large products (at least 1024 of them, K >= 256):
    whole and ragged, with and without the vector loads of rows and stores of
    columns.  Bound as above."""
    g = torch.Generator(device=DEV).manual_seed(M + 7 * N + 13 * K)
    A = torch.randn((M, K + ld) if ak else (K, M + ld), device=DEV, generator=g)
    B = torch.randn((N, K + ld) if bk else (K, N + ld), device=DEV, generator=g)
    bias = torch.randn(N, device=DEV, generator=g)
    a = (A[:, :K] if ak else A[:, :M].t()).double()
    b = (B[:, :K].t() if bk else B[:, :N]).double()
    C = torch.full((M + 1, N + ld), float("nan"), device=DEV)
    LU.layup_gemm_f32(LU.gemm_desc(A, B, C, M, N, K, A.shape[1], B.shape[1], N + ld, ak, bk, True, bias=bias),
                      torch.cuda.current_stream())
    torch.cuda.synchronize()
    bound = 1.01 * (K + 2) * 2.0 ** -24 * (a.abs() @ b.abs() + bias.double().abs())
    assert torch.all((C[:M, :N].double() - a @ b - bias.double()).abs() <= bound)
    assert torch.all(torch.isnan(C[M])) and torch.all(torch.isnan(C[:, N:]))


@pytest.mark.parametrize("layout", ["kk", "kn", "mn"])
@pytest.mark.parametrize("M,N", [(8192, 768), (8192, 3072), (4104, 4096), (2048, 8192), (1368, 3304), (520, 264), (72, 40)])
@pytest.mark.parametrize("K", [8, 64, 72, 128, 200, 264])
def test_gemm_tiles_and_short_k(layout, M, N, K):
    """The tiles the library chooses for large and small outputs with a short K
    (test_gemm_every_tile names them all) at the edges of their pipelines:
    fewer K steps than stages, exactly as many, one more, and partial last
    steps.  Bound per element: a float32 sum of K exact products
    in any order, 2 (K + 8) 2^-24 of the sum of absolute values (the factor
    two covers adders that truncate)."""
    ak, bk = {"kk": (True, True), "kn": (True, False), "mn": (False, False)}[layout]
    g = torch.Generator(device=DEV).manual_seed(M + 3 * N + 5 * K)
    A = torch.randn((M, K) if ak else (K, M), device=DEV, generator=g).to(torch.bfloat16)
    B = torch.randn((N, K) if bk else (K, N), device=DEV, generator=g).to(torch.bfloat16)
    C = torch.full((M, N), float("nan"), device=DEV)
    rs = None if ak else torch.full((M,), float("nan"), device=DEV)
    LU.layup_gemm_bf16(LU.gemm_desc(A, B, C, M, N, K, K if ak else M, K if bk else N, N, ak, bk, True, a_rowsum=rs),
                       torch.cuda.current_stream())
    torch.cuda.synchronize()
    a = (A if ak else A.t().contiguous()).double()
    b = (B.t().contiguous() if bk else B).double()
    assert torch.all((C.double() - a @ b).abs() <= 2 * (K + 8) * 2.0 ** -24 * (a.abs() @ b.abs()))
    if rs is not None:
        assert torch.all((rs.double() - a.sum(1)).abs() <= 2 * (K + 8) * 2.0 ** -24 * a.abs().sum(1))


def _gelu64(x):
    """GELU (tanh form) of float64 x: value, derivative, and s, 2u, x s' of them."""
    c = math.sqrt(2.0 / math.pi)
    u2 = 2.0 * c * (x + 0.044715 * x ** 3)
    e = torch.exp(-u2)
    s = 1.0 / (1.0 + e)
    t = x * s * (e * s) * 2.0 * c * (1.0 + 3.0 * 0.044715 * x * x)
    return x * s, s + t, s, u2, t


def _gelu_epilogue(x, y, dy):
    f = LU.lib().layup_test_gelu
    f.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int64, ctypes.c_void_p]
    assert f(x.data_ptr(), y.data_ptr(), dy.data_ptr(), x.numel(), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()


@pytest.mark.parametrize("lo,hi", [(-9.9, -5.0), (-5.0, -1.0), (-1.0, 1.0), (1.0, 10.0)])
def test_gelu_epilogue_arithmetic(lo, hi):
    """The GELU of the epilogues in float32, before the bfloat16 store, at four
    million points a range.  With eps = 2^-24: the exponent t = -2u log2(e)
    carries at most 2 eps (half an ulp each of x^2, weighted by its share, and
    of K1 + K2 x^2, and their constants), which costs e at most 2 |2u| eps, of
    which 1 - s reaches s; the exponential, reciprocal (an ulp each), sums and
    products add at most 6 eps.  The derivative s + t (t = x s' has s (1 - s))
    adds the same once more to each term."""
    x = torch.linspace(lo, hi, 4_000_001, dtype=torch.float32, device=DEV)
    y, dy = torch.empty_like(x), torch.empty_like(x)
    _gelu_epilogue(x, y, dy)
    ref, dref, s, u2, t = _gelu64(x.double())
    eps = 2.0 ** -24
    rel_s = 2 * u2.abs() * (1 - s) + 6
    assert torch.all((y.double() - ref).abs() <= eps * rel_s * ref.abs())
    rel_t = 2 * u2.abs() * (1 - 2 * s).abs() + 12
    assert torch.all((dy.double() - dref).abs() <= eps * (rel_s * s + rel_t * t.abs()))


def test_gelu_epilogue_extremes():
    """Far from zero: GELU is x (and its derivative 1) to the right; to the
    left s <= 2^-125, so it is below 2e-37 |x| in magnitude and its derivative
    below 2e-37 |x| (1 + x^2); NaN stays NaN."""
    x = torch.tensor([12.9, 13.0, 100.0, 1e12, -10.0, -13.0, -1e4, 0.0, float("nan")], device=DEV)
    y, dy = torch.empty_like(x), torch.empty_like(x)
    _gelu_epilogue(x, y, dy)
    assert torch.equal(y[:4], x[:4]) and torch.equal(dy[:4], torch.ones_like(x[:4]))
    assert torch.all(y[4:7].abs() <= 2e-37 * x[4:7].abs()) and torch.all(dy[4:7].abs() <= 2e-37 * x[4:7].abs() * (1 + x[4:7] ** 2))
    assert y[7] == 0 and dy[7] == 0.5 and torch.isnan(y[8]) and torch.isnan(dy[8])


def _tile(descs, group=0, cfg=-1, splits=1, run=1 << 62, upd=None, hp=None, alpha=0.5):
    """Products through the test entry: tile configuration and split given, or (cfg < 0) chosen by the library."""
    f = LU.lib().layup_test_gemm_tile
    f.argtypes = [ctypes.c_void_p] + [ctypes.c_int32] * 4 + [ctypes.c_int64] + \
        [ctypes.c_void_p] * 2 + [ctypes.c_float, ctypes.c_void_p]
    arr = (LU.layup_gemm_desc * len(descs))(*descs)
    ups = (LU.layup_tensor * len(descs))(*upd) if upd else None
    st = f(ctypes.addressof(arr), len(descs), group, cfg, splits, run,
           ctypes.addressof(ups) if upd else None, ctypes.addressof(hp) if hp else None, alpha,
           torch.cuda.current_stream().cuda_stream)
    assert st == 0, LU.lib().layup_global_error()
    torch.cuda.synchronize()


class _Prod:
    """Operands (bf16 of unit normals), outputs and float64 reference of one product."""

    def __init__(self, layout, M, N, K, ws=None, seed=0):
        ak, bk = {"kk": (True, True), "kn": (True, False), "mn": (False, False)}[layout]
        g = torch.Generator(device=DEV).manual_seed(seed + M + 3 * N + 5 * K)
        A = torch.randn((M, K) if ak else (K, M), device=DEV, generator=g).to(torch.bfloat16)
        B = torch.randn((N, K) if bk else (K, N), device=DEV, generator=g).to(torch.bfloat16)
        self.A, self.B, self.C = A, B, torch.full((M, N), float("nan"), device=DEV)
        self.rs = None if ak else torch.full((M,), float("nan"), device=DEV)
        self.desc = LU.gemm_desc(A, B, self.C, M, N, K, K if ak else M, K if bk else N, N, ak, bk, True,
                                 workspace=ws, workspace_bytes=ws.numel() if ws is not None else 0, a_rowsum=self.rs)
        self.a, self.b = (A if ak else A.t().contiguous()), (B.t().contiguous() if bk else B)

    def ref(self):
        return self.a.double() @ self.b.double()

    def rel(self):
        ref = self.ref()
        return float((self.C.double() - ref).norm() / ref.norm())


# the error of a float32 sum of K products in one run of the matrix instruction: 16 of them take two roundings, each
# off by 0.41 x 2^-24 of the partial sum (rms over a binade), whose square grows linearly: sqrt(run / 16) in all; a
# fifth more for the instruction's own additions and the sum of the runs
def _run_error(run):
    return 1.2 * 0.41 * (run / 16) ** 0.5 * 2.0 ** -24


@pytest.mark.parametrize("d,ff,tokens,runs", [
    (768, 3072, 8192, (2048, 1024, 2752, 2752)),     # splits of 4, 8, 3 and 3
    (1024, 4096, 8192, (4096, 1024, 4096, 4096)),    # 2, 8, 2 and 2
    (2048, 8192, 8192, (8192, 4096, 8192, 8192)),    # enough tiles for whole sums but for the attention projection
    (1248, 3744, 2880, (2880, 576, 2880, 2880)),     # the same, ragged
])
def test_block_weight_gradients_are_summed_in_short_runs(d, ff, tokens, runs):
    """The four dW products of a block as one group: none is summed in longer
    runs than where K is split to fill the chip with 128 x 128 tiles."""
    ws = torch.empty(128 << 20, dtype=torch.uint8, device=DEV)
    ps = [_Prod("mn", m, n, tokens, ws) for m, n in ((3 * d, d), (d, d), (ff, d), (d, ff))]
    for beside in (False, True):
        _tile([p.desc for p in ps], group=2 if beside else 1)
        for p, run in zip(ps, runs):
            assert p.rel() <= _run_error(run), (p.C.shape, p.rel())


@pytest.mark.parametrize("layout,M,N,K,run", [("kn", 8192, 768, 50304, 6304), ("kn", 8192, 1024, 50304, 6304),
                                              ("kn", 1368, 832, 3304, 576), ("kn", 2048, 2048, 8192, 4096),
                                              ("mn", 768, 768, 8192, 1024)])
def test_long_products_are_summed_in_short_runs(layout, M, N, K, run):
    """The same for single products, through the public call."""
    ws = torch.empty(256 << 20, dtype=torch.uint8, device=DEV)
    p = _Prod(layout, M, N, K, ws)
    LU.layup_gemm_bf16(p.desc, torch.cuda.current_stream())
    torch.cuda.synchronize()
    assert p.rel() <= _run_error(run), p.rel()


def _within(p, tail=8):
    """C and the row sums within a float32 sum of K exact products in any
    order: 2 (K + 8) 2^-24 of the sum of absolute values (the factor two
    covers adders that truncate)."""
    K = p.a.shape[1]
    a, b = p.a.double(), p.b.double()
    eps = 2 * (K + tail) * 2.0 ** -24
    assert torch.all((p.C.double() - a @ b).abs() <= eps * (a.abs() @ b.abs()))
    if p.rs is not None:
        assert torch.all((p.rs.double() - a.sum(1)).abs() <= eps * a.abs().sum(1))


# (K, split, longest run): no whole K step, one, as many as stages and one more, partial last steps; splits whose
# length is an odd multiple of 32 (1000 / 2 -> 512, 1056 / 3 -> 352, 4576 / 5 -> 928, with the last one short); runs of
# one K step, of some, longer than the split
EDGES = [(8, 1, None), (64, 1, None), (72, 1, None), (192, 1, None), (264, 1, 64), (328, 1, 128), (1000, 2, None),
         (1056, 3, None), (1056, 3, 64), (4576, 5, 512), (4576, 1, 512), (2056, 1, 1984)]


@pytest.mark.parametrize("cfg", range(7))
@pytest.mark.parametrize("layout", ["kk", "kn", "mn"])
def test_gemm_every_tile(layout, cfg):
    """Every tile configuration in every layout, two tiles and a ragged rest in
    both dimensions, at the edges of the K loop, of the split of K and of the
    runs that the accumulators take (tiles that have the short-run form)."""
    ws = torch.empty(64 << 20, dtype=torch.uint8, device=DEV)
    flushes = cfg >= 2 and not (cfg == 4 and layout != "mn")
    for K, splits, run in EDGES:
        if run is not None and not flushes:
            continue
        p = _Prod(layout, 544, 536, K, ws, seed=cfg)
        _tile([p.desc], cfg=cfg, splits=splits, run=run or 1 << 62)
        _within(p)


@pytest.mark.parametrize("cfg", [0, 2, 4])
@pytest.mark.parametrize("K,splits", [(8, 1), (200, 1), (1000, 2), (4576, 5), (2056, 1), (1600, 0), (2624, 0)])
def test_gemm_group_every_tile(cfg, K, splits):
    """Four products of a group, small and ragged, on each of its tiles: without
    a split, split alike, and each as far as its limit asks (splits = 0: from
    K = 1536 on)."""
    ws = torch.empty(64 << 20, dtype=torch.uint8, device=DEV)
    ps = [_Prod("mn", m, n, K, ws, seed=cfg) for m, n in ((264, 136), (72, 72), (520, 264), (2048, 2304))]
    _tile([p.desc for p in ps], group=1, cfg=cfg, splits=splits)
    for p in ps:
        _within(p)


@pytest.mark.parametrize("K", [1600, 2112, 2624, 2632, 3136, 4672])
def test_gemm_group_tiles_agree_bit_for_bit(K):
    """The tile does not change the order of the sums: 256 x 128 and 128 x 128,
    with rings of three and of two stages, give the same bits, also where a run
    ends within the last steps of K (2624 is 41 steps in runs of 8)."""
    ws = torch.empty(64 << 20, dtype=torch.uint8, device=DEV)
    ps = [_Prod("mn", m, n, K, ws) for m, n in ((264, 136), (72, 72), (520, 264))]
    out = []
    for cfg in (2, 4):
        _tile([p.desc for p in ps], group=1, cfg=cfg)
        out.append([t.clone() for p in ps for t in (p.C, p.rs)])
    for x, y in zip(*out):
        assert torch.equal(x, y)


@pytest.mark.parametrize("cfg", [0, 2, 4])
@pytest.mark.parametrize("K,splits", [(72, 1), (1000, 2), (2056, 1), (1600, 0)])
@pytest.mark.parametrize("optim", ["adamw", "sgd"])
def test_gemm_group_update_epilogue(cfg, K, splits, optim):
    """The same with the weight update in the epilogue or in the split's sum: equal to the gradients of the float32 epilogue
    put through the update + mix kernel, bit for bit but for the last rounding
    of the update (2 2^-24 of the step's terms)."""
    ws = torch.empty(64 << 20, dtype=torch.uint8, device=DEV)
    hp = LU.hparams("adamw", 1e-2, 0.0, 0.1, 0.9, 0.95, 1e-8, 3) if optim == "adamw" else LU.hparams("sgd", 1e-2, 0.9, 5e-5)
    ps = [_Prod("mn", m, n, K, ws, seed=cfg) for m, n in ((264, 136), (72, 72), (520, 264))]
    _tile([p.desc for p in ps], group=1, cfg=cfg, splits=splits)
    g = torch.Generator(device=DEV).manual_seed(K)
    fused, plain, ups = [], [], []
    for p in ps:
        n = p.C.numel()
        st = {k: torch.randn(n, device=DEV, generator=g) for k in ("param", "state0", "peer")}
        st["state1"] = torch.rand(n, device=DEV, generator=g)
        pair = [{k: v.clone() for k, v in st.items()} for _ in range(2)]
        for d in pair:
            d["param_bf16"] = torch.zeros(n, dtype=torch.int16, device=DEV)
        ts = []
        for d in pair:
            t = LU.layup_tensor()
            t.param, t.state0, t.peer = (d[k].data_ptr() for k in ("param", "state0", "peer"))
            t.state1 = d["state1"].data_ptr() if optim == "adamw" else None
            t.param_bf16, t.numel, t.decay, t.grad = d["param_bf16"].data_ptr(), n, 1, p.C.data_ptr()
            ts.append(t)
        fused.append(pair[0])
        plain.append(pair[1])
        ups.append(ts[0])
        LU.layup_layer_update_mix_static([ts[1]], hp, 0.25, None, torch.cuda.current_stream())
    keep = [p.rs.clone() for p in ps]
    _tile([p.desc for p in ps], group=1, cfg=cfg, splits=splits, upd=ups, hp=hp, alpha=0.25)
    for p, rs, a, b in zip(ps, keep, fused, plain):
        assert torch.equal(p.rs, rs)
        for k in ("param", "state0", "state1"):
            assert torch.all((a[k] - b[k]).abs() <= 2.0 ** -22 * (1 + b[k].abs())), k
        assert torch.equal(a["peer"], b["peer"])
        assert torch.equal(a["param_bf16"].view(torch.bfloat16), a["param"].to(torch.bfloat16))
