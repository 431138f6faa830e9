"""Each HIP kernel against the oracle's op, through the C ABI, element by
element on seeded inputs: sizes span several tiles and a ragged tail."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from oracle import stack_oracle as O  # noqa: E402
from paper_2410_08791_amd import binding as sp  # noqa: E402
from tests.gpu_util import (DEV, bf16_vals, dev_f32, dev_u16, host_u16, ptr, rand_bf16,  # noqa: E402
                            stream_ptr)

BF16_EPS = 2.0 ** -8     # half an ulp of bf16, relative


def sync():
    torch.cuda.synchronize()


@pytest.mark.parametrize("T,d", [(37, 256), (5, 4096), (3, 8192), (7, 1280), (1, 64)])
@pytest.mark.parametrize("ln", [False, True])
def test_norm(T, d, ln):
    rng = np.random.default_rng(T * 7 + d + ln)
    h = (rng.standard_normal((T, d)) * 2 + (0.5 if ln else 0)).astype(np.float32)
    gb, g = rand_bf16(rng, d, 0.3)
    g = g + 1.0
    gb = __import__("paper_2410_08791_amd.synth", fromlist=["x"]).f32_to_bf16_bits(g.astype(np.float32))
    g = bf16_vals(gb)
    bb, b = rand_bf16(rng, d, 0.3)
    out = torch.zeros((T, d), dtype=torch.int16, device=DEV)
    hd, gd, bd = dev_f32(h), dev_u16(gb), dev_u16(bb)      # keep the device buffers alive
    rc = sp.spk_norm(stream_ptr(), ptr(hd), ptr(gd), ptr(bd) if ln else None, ptr(out), T, d, 1e-5)
    assert rc == sp.SP_OK
    sync()
    got = bf16_vals(host_u16(out))
    h64 = h.astype(np.float64)
    ref = O.layernorm(h64, g, b, 1e-5) if ln else O.rmsnorm(h64, g, 1e-5)
    assert np.all(np.abs(got - ref) <= BF16_EPS * np.abs(ref) + 1e-5)


def gemm_ref(A, W, epi, R=None, bias=None, N=None):
    acc = A @ W.T
    if bias is not None:
        acc = acc + bias
    if epi == sp.EPI_RESID_F32:
        return R + acc
    if epi == sp.EPI_GELU_BF16:
        return O.gelu(acc)
    if epi == sp.EPI_SWIGLU_BF16:
        return O.silu(acc[:, :N]) * acc[:, N:]
    return acc


@pytest.mark.parametrize("tile", [1, 2, 3, 4, 5, 6, 7, 8, 10, 0])
@pytest.mark.parametrize("M,N,K", [(200, 328, 128), (257, 296, 64), (300, 520, 256), (64, 128, 1024)])
@pytest.mark.parametrize("epi", [sp.EPI_BF16, sp.EPI_RESID_F32, sp.EPI_GELU_BF16, sp.EPI_SWIGLU_BF16, sp.EPI_F32])
def test_gemm_kmajor(epi, M, N, K, tile):
    if tile in (8, 10) and epi == sp.EPI_SWIGLU_BF16:
        pytest.skip("the 256x192 and 256x320 tiles do not take the SwiGLU epilogue")
    rng = np.random.default_rng(M + N * 3 + K * 5 + epi)
    Ab, A = rand_bf16(rng, (M, K))
    nw = 2 * N if epi == sp.EPI_SWIGLU_BF16 else N
    Wb, W = rand_bf16(rng, (nw, K), 0.1)
    bias_b, bias = (rand_bf16(rng, N, 0.5) if epi in (sp.EPI_GELU_BF16, sp.EPI_BF16, sp.EPI_RESID_F32) else (None, None))
    R = rng.standard_normal((M, N)).astype(np.float32)
    f32out = epi in (sp.EPI_RESID_F32, sp.EPI_F32)
    Cd = dev_f32(R) if epi == sp.EPI_RESID_F32 else torch.zeros((M, N), dtype=torch.float32 if f32out else torch.int16, device=DEV)
    Ad, Wd = dev_u16(Ab), dev_u16(Wb)
    bd = dev_u16(bias_b) if bias_b is not None else None
    rc = sp.spk_gemm(stream_ptr(), epi, ptr(Ad), K, 0, ptr(Wd), K, 0, ptr(Cd), N,
                     ptr(Cd) if epi == sp.EPI_RESID_F32 else None, N, ptr(bd), M, N, K, tile)
    assert rc == sp.SP_OK
    sync()
    ref = gemm_ref(A, W, epi, R.astype(np.float64), bias, N)
    got = Cd.cpu().numpy().astype(np.float64) if f32out else bf16_vals(host_u16(Cd))
    scale = np.max(np.abs(ref))
    tol = 2e-6 * np.sqrt(K) * scale + (0 if f32out else BF16_EPS * np.abs(ref))
    assert np.all(np.abs(got - ref) <= tol + 1e-6), float(np.max(np.abs(got - ref)))


@pytest.mark.parametrize("tile", [9, 0, 11, 12, 13])
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (8, 328, 4096), (16, 24, 320), (5, 1288, 1088), (13, 4096, 192),
                                   (17, 40, 448), (32, 328, 1280), (33, 72, 64), (64, 5128, 1280)])
@pytest.mark.parametrize("epi", [sp.EPI_BF16, sp.EPI_RESID_F32, sp.EPI_GELU_BF16, sp.EPI_SWIGLU_BF16, sp.EPI_F32])
def test_gemm_few_rows_streams_the_weights(epi, M, N, K, tile):
    """At most 64 activation rows (a decode step, the ragged last rows of a long launch): the
    small-tile kernel with its few-row tiles, forced (tile 9; 11-13 with 16, 32, 64 rows per work-group, the rest of
    the rows in further work-groups) and as the heuristic's choice; N not a multiple of the
    16 columns of a work-group nor of the 8 column blocks of a dispatch group, K / 32 not a multiple of the eight waves that share the
    contraction, M at and next to the limits of its one, two and four 16-row tiles."""
    rng = np.random.default_rng(M + N * 3 + K * 5 + epi)
    Ab, A = rand_bf16(rng, (M, K))
    nw = 2 * N if epi == sp.EPI_SWIGLU_BF16 else N
    Wb, W = rand_bf16(rng, (nw, K), 0.1)
    bias_b, bias = (rand_bf16(rng, N, 0.5) if epi in (sp.EPI_GELU_BF16, sp.EPI_BF16, sp.EPI_RESID_F32) else (None, None))
    R = rng.standard_normal((M, N)).astype(np.float32)
    f32out = epi in (sp.EPI_RESID_F32, sp.EPI_F32)
    # one guard row behind C: the kernel must not write past row M - 1
    Cd = torch.full((M + 1, N), 7.0 if f32out else 7, dtype=torch.float32 if f32out else torch.int16, device=DEV)
    if epi == sp.EPI_RESID_F32:
        Cd[:M] = dev_f32(R)
    Ad, Wd = dev_u16(Ab), dev_u16(Wb)
    bd = dev_u16(bias_b) if bias_b is not None else None
    rc = sp.spk_gemm(stream_ptr(), epi, ptr(Ad), K, 0, ptr(Wd), K, 0, ptr(Cd), N,
                     ptr(Cd) if epi == sp.EPI_RESID_F32 else None, N, ptr(bd), M, N, K, tile)
    assert rc == sp.SP_OK
    sync()
    ref = gemm_ref(A, W, epi, R.astype(np.float64), bias, N)
    out = Cd.cpu()
    assert bool((out[M] == 7).all())
    got = out[:M].numpy().astype(np.float64) if f32out else bf16_vals(host_u16(out[:M].contiguous()))
    scale = np.max(np.abs(ref))
    tol = 2e-6 * np.sqrt(K) * scale + (0 if f32out else BF16_EPS * np.abs(ref))
    assert np.all(np.abs(got - ref) <= tol + 1e-6), float(np.max(np.abs(got - ref)))


@pytest.mark.parametrize("tile", [14, 15, 16, 17, 18, 19, 20])
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (16, 16, 512), (97, 136, 64), (65, 264, 832), (257, 72, 1280)])
@pytest.mark.parametrize("epi", [sp.EPI_BF16, sp.EPI_RESID_F32, sp.EPI_GELU_BF16, sp.EPI_SWIGLU_BF16, sp.EPI_F32])
def test_gemm_small_tiles(epi, M, N, K, tile):
    """Every tile of the small-tile kernel: one row and one column group, whole tiles, ragged rows and
    columns; fewer k-tiles than contraction groups, a count no group count divides, many."""
    rng = np.random.default_rng(M + N * 3 + K * 5 + epi)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (2 * N if epi == sp.EPI_SWIGLU_BF16 else N, K), 0.1)
    bias_b, bias = (rand_bf16(rng, N, 0.5) if epi in (sp.EPI_GELU_BF16, sp.EPI_BF16, sp.EPI_RESID_F32) else (None, None))
    R = rng.standard_normal((M, N)).astype(np.float32)
    f32out = epi in (sp.EPI_RESID_F32, sp.EPI_F32)
    Cd = torch.full((M + 1, N), 7.0 if f32out else 7, dtype=torch.float32 if f32out else torch.int16, device=DEV)
    if epi == sp.EPI_RESID_F32:
        Cd[:M] = dev_f32(R)
    Ad, Wd = dev_u16(Ab), dev_u16(Wb)
    bd = dev_u16(bias_b) if bias_b is not None else None
    assert sp.spk_gemm(stream_ptr(), epi, ptr(Ad), K, 0, ptr(Wd), K, 0, ptr(Cd), N,
                       ptr(Cd) if epi == sp.EPI_RESID_F32 else None, N, ptr(bd), M, N, K, tile) == sp.SP_OK
    sync()
    ref = gemm_ref(A, W, epi, R.astype(np.float64), bias, N)
    out = Cd.cpu()
    assert bool((out[M] == 7).all())                      # the row behind C
    got = out[:M].numpy().astype(np.float64) if f32out else bf16_vals(host_u16(out[:M].contiguous()))
    tol = 2e-6 * np.sqrt(K) * np.max(np.abs(ref)) + (0 if f32out else BF16_EPS * np.abs(ref))   # as in test_gemm_kmajor
    assert np.all(np.abs(got - ref) <= tol + 1e-6), float(np.max(np.abs(got - ref)))


@pytest.mark.parametrize("tile", [16, 18])
@pytest.mark.parametrize("M,N,K", [(8, 8, 64), (72, 136, 320), (264, 520, 1088)])
def test_gemm_small_tiles_transposed_operands(M, N, K, tile):
    """The backward forms on the small-tile kernel: W, and both operands, with the row index contiguous."""
    rng = np.random.default_rng(M * 3 + N + K + tile)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (N, K), 0.1)
    Ad, ATd, WTd = dev_u16(Ab), dev_u16(Ab.T), dev_u16(Wb.T)
    C1 = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    C2 = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    assert sp.spk_gemm(stream_ptr(), sp.EPI_F32, ptr(Ad), K, 0, ptr(WTd), N, 1, ptr(C1), N, None, 0, None, M, N, K, tile) == sp.SP_OK
    assert sp.spk_gemm(stream_ptr(), sp.EPI_F32, ptr(ATd), M, 1, ptr(WTd), N, 1, ptr(C2), N, None, 0, None, M, N, K, tile) == sp.SP_OK
    sync()
    ref = A @ W.T
    tol = 2e-6 * np.sqrt(K) * np.max(np.abs(ref))
    for C_ in (C1, C2):
        assert np.all(np.abs(C_.cpu().numpy() - ref) <= tol)


@pytest.mark.parametrize("M", [1, 16, 17, 33, 64])
@pytest.mark.parametrize("N,K", [(8192, 8192), (1280, 5120)])
def test_gemm_few_rows_fp32_sums_are_short(M, N, K):
    """The fp32 result of at most 64 rows against float64: eight partial sums per element.  With sums of K products the
    error of such a product of independent normals is about c sqrt(K / parts) 2^-24 of it; c = 0.089 was measured for
    eight parts (1.68e-7 at K = 8192); four parts exceed the bound below by a tenth or more."""
    rng = np.random.default_rng(M + N)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (N, K), 0.02)
    Ad, Wd = dev_u16(Ab), dev_u16(Wb)
    R = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    assert sp.spk_gemm(stream_ptr(), sp.EPI_RESID_F32, ptr(Ad), K, 0, ptr(Wd), K, 0, ptr(R), N, ptr(R), N, None, M, N, K, 0) == sp.SP_OK
    sync()
    ref = torch.from_numpy(A).to(DEV) @ torch.from_numpy(W).to(DEV).t().contiguous()
    err = float((R.double() - ref).norm() / ref.norm())
    assert err <= 1.2 * 0.089 * np.sqrt(K / 8) * 2.0 ** -24, err


def test_gemm_few_rows_kernel_refuses_what_it_cannot_take():
    z = torch.zeros(1 << 16, dtype=torch.int16, device=DEV)
    f = torch.zeros(1 << 14, dtype=torch.float32, device=DEV)
    # 65 rows; an operand with the row index contiguous
    assert sp.spk_gemm(stream_ptr(), sp.EPI_BF16, ptr(z), 64, 0, ptr(z), 64, 0, ptr(z), 64, None, 0, None, 65, 64, 64, 9) == sp.SP_ERR_INVALID_ARG
    assert sp.spk_gemm(stream_ptr(), sp.EPI_F32, ptr(z), 64, 0, ptr(z), 64, 1, ptr(f), 64, None, 0, None, 8, 64, 64, 9) == sp.SP_ERR_INVALID_ARG
    sync()


def test_gemm_output_rows_not_16_byte_aligned():
    """A bf16 output whose row stride is a multiple of 4 but not of 8 elements: the kernel that
    writes 16-byte pieces of a row cannot take it, the library must fall back by itself (also
    when one of that kernel's tiles is forced) and leave the padding columns alone."""
    M, N, K, ldc = 300, 264, 128, 268
    rng = np.random.default_rng(5)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (N, K), 0.1)
    Ad, Wd = dev_u16(Ab), dev_u16(Wb)
    ref = A @ W.T
    for tile in (0, 5, 7):
        Cd = torch.full((M, ldc), 0x7fc0, dtype=torch.int16, device=DEV)
        rc = sp.spk_gemm(stream_ptr(), sp.EPI_BF16, ptr(Ad), K, 0, ptr(Wd), K, 0, ptr(Cd), ldc,
                         None, 0, None, M, N, K, tile)
        assert rc == sp.SP_OK
        sync()
        raw = host_u16(Cd)
        got = bf16_vals(raw[:, :N])
        assert np.all(np.abs(got - ref) <= BF16_EPS * np.abs(ref) + 2e-6 * np.sqrt(K) * np.max(np.abs(ref)))
        assert np.all(raw[:, N:] == 0x7fc0)


@pytest.mark.parametrize("epi", [sp.EPI_GELU_BF16, sp.EPI_RESID_F32])
def test_gemm_ragged_rows_cut_off(epi):
    """A shape whose last, ragged row of 256-row tiles would cost a whole extra round: the
    library's own choice computes rows 1024.. in a second launch.  Every row must come out."""
    M, N, K = 1088, 13312, 64
    rng = np.random.default_rng(11 + epi)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (N, K), 0.1)
    bias_b, bias = rand_bf16(rng, N, 0.5)
    R = rng.standard_normal((M, N)).astype(np.float32)
    f32out = epi == sp.EPI_RESID_F32
    Cd = dev_f32(R) if f32out else torch.zeros((M, N), dtype=torch.int16, device=DEV)
    Ad, Wd, bd = dev_u16(Ab), dev_u16(Wb), dev_u16(bias_b)
    rc = sp.spk_gemm(stream_ptr(), epi, ptr(Ad), K, 0, ptr(Wd), K, 0, ptr(Cd), N,
                     ptr(Cd) if f32out else None, N, ptr(bd), M, N, K, 0)
    assert rc == sp.SP_OK
    sync()
    ref = gemm_ref(A, W, epi, R.astype(np.float64), bias, N)
    got = Cd.cpu().numpy().astype(np.float64) if f32out else bf16_vals(host_u16(Cd))
    tol = 2e-6 * np.sqrt(K) * np.max(np.abs(ref)) + (0 if f32out else BF16_EPS * np.abs(ref))
    assert np.all(np.abs(got - ref) <= tol + 1e-6), float(np.max(np.abs(got - ref)))


@pytest.mark.parametrize("tile", [1, 2, 3, 4, 6, 0])
@pytest.mark.parametrize("M,N,K", [(200, 328, 128), (264, 520, 192)])
def test_gemm_transposed_operands(M, N, K, tile):
    """The backward forms: dX = dY W (weight read with its row index contiguous) and
    dW = dY^T X (both operands transposed on the way in)."""
    rng = np.random.default_rng(M * 3 + N + K + tile)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (N, K), 0.1)
    # (0,1): W given as [K, N]
    WbT = np.ascontiguousarray(Wb.T)
    C1 = torch.zeros((M, N), dtype=torch.int16, device=DEV)
    Ad, WTd = dev_u16(Ab), dev_u16(WbT)
    rc = sp.spk_gemm(stream_ptr(), sp.EPI_BF16, ptr(Ad), K, 0, ptr(WTd), N, 1, ptr(C1), N,
                     None, 0, None, M, N, K, tile)
    assert rc == sp.SP_OK
    # (1,1): both given transposed, fp32 output
    AbT = np.ascontiguousarray(Ab.T)
    C2 = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    ATd = dev_u16(AbT)
    rc = sp.spk_gemm(stream_ptr(), sp.EPI_F32, ptr(ATd), M, 1, ptr(WTd), N, 1, ptr(C2), N,
                     None, 0, None, M, N, K, tile)
    assert rc == sp.SP_OK
    sync()
    ref = A @ W.T
    scale = np.max(np.abs(ref))
    assert np.all(np.abs(bf16_vals(host_u16(C1)) - ref) <= BF16_EPS * np.abs(ref) + 2e-6 * np.sqrt(K) * scale)
    assert np.all(np.abs(C2.cpu().numpy() - ref) <= 2e-6 * np.sqrt(K) * scale)


@pytest.mark.parametrize("tile", [5, 6, 7, 8, 10, 0])
@pytest.mark.parametrize("M,N,K", [(8, 8, 64), (264, 328, 192), (520, 648, 128), (256, 320, 64), (1032, 3592, 64)])
def test_gemm_transposed_operands_lds_dma(M, N, K, tile):
    """The backward forms on the LDS-DMA kernel: one row group, whole tiles, ragged rows and columns of
    every tile width, one k-tile, a shape whose ragged rows the library cuts off.  One guard row behind C."""
    rng = np.random.default_rng(M * 3 + N + K + tile)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (N, K), 0.1)
    R = rng.standard_normal((M, N)).astype(np.float32)
    Ad, ATd, WTd = dev_u16(Ab), dev_u16(Ab.T), dev_u16(Wb.T)
    ref = A @ W.T
    tol = 2e-6 * np.sqrt(K) * np.max(np.abs(ref))                          # as in test_gemm_transposed_operands
    for epi, a_form in ((sp.EPI_BF16, 0), (sp.EPI_F32, 0), (sp.EPI_RESID_F32, 0), (sp.EPI_F32, 1)):
        f32out = epi != sp.EPI_BF16
        Cd = torch.full((M + 1, N), 7.0 if f32out else 7, dtype=torch.float32 if f32out else torch.int16, device=DEV)
        if epi == sp.EPI_RESID_F32:
            Cd[:M] = dev_f32(R)
        assert sp.spk_gemm(stream_ptr(), epi, ptr(ATd if a_form else Ad), M if a_form else K, a_form, ptr(WTd), N, 1, ptr(Cd), N,
                           ptr(Cd) if epi == sp.EPI_RESID_F32 else None, N, None, M, N, K, tile) == sp.SP_OK
        sync()
        out = Cd.cpu()
        assert bool((out[M] == 7).all())
        got = out[:M].numpy() if f32out else bf16_vals(host_u16(out[:M].contiguous()))
        want = ref + R if epi == sp.EPI_RESID_F32 else ref
        assert np.all(np.abs(got - want) <= tol + (2.0 ** -23 * np.abs(want) if f32out else BF16_EPS * np.abs(want))), (epi, a_form)


@pytest.mark.parametrize("tile", [5, 6, 7, 8, 10])
@pytest.mark.parametrize("K", [64, 128, 192, 320, 384, 704])
def test_gemm_lds_dma_k_tiles(K, tile):
    """One to eleven k-tiles through the rings of three to five stages and slots (fewer than the ring holds, its
    length, once and twice round), several tiles of every width in both directions so that both orders of fetching
    the operands occur, ragged rows and columns; every operand form against the same float64 product."""
    M, N = 536, 712
    rng = np.random.default_rng(K + tile)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (N, K), 0.1)
    d = [dev_u16(x) for x in (Ab, Wb, Ab.T, Wb.T)]
    ref = A @ W.T
    for epi, a_form, w_form in ((sp.EPI_F32, 0, 0), (sp.EPI_F32, 0, 1), (sp.EPI_F32, 1, 1), (sp.EPI_BF16, 0, 0)):
        f32out = epi == sp.EPI_F32
        Cd = torch.full((M + 1, N), 7.0 if f32out else 7, dtype=torch.float32 if f32out else torch.int16, device=DEV)
        assert sp.spk_gemm(stream_ptr(), epi, ptr(d[2 * a_form]), M if a_form else K, a_form, ptr(d[1 + 2 * w_form]), N if w_form else K, w_form,
                           ptr(Cd), N, None, 0, None, M, N, K, tile) == sp.SP_OK
        sync()
        out = Cd.cpu()
        assert bool((out[M] == 7).all())
        got = out[:M].numpy() if f32out else bf16_vals(host_u16(out[:M].contiguous()))
        tol = 2e-6 * np.sqrt(K) * np.max(np.abs(ref))                      # as in test_gemm_transposed_operands
        assert np.all(np.abs(got - ref) <= tol + (0 if f32out else BF16_EPS * np.abs(ref))), (epi, a_form, w_form)


@pytest.mark.parametrize("a_form,w_form,far,ld", [
    (0, 0, "a", 8_421_512), (0, 0, "w", 8_421_512), (0, 1, "w", 34_087_048), (1, 1, "a", 34_087_048),   # 255 or 63 rows just past 4 GiB
    (0, 0, "a", 8_421_448), (1, 1, "w", 34_086_968),                                                    # ... and just below
    (0, 0, "a", -128), (0, 0, "w", -136), (0, 1, "w", -328), (1, 1, "a", -264),                         # rows in reverse order
])
@pytest.mark.parametrize("tile", [0, 5, 6, 8, 10])
def test_gemm_rows_far_apart_or_in_reverse(tile, a_form, w_form, far, ld):
    """Operands whose rows lie so far apart that an offset inside a tile passes 32 bits, and views with a negative stride:
    every element of the product, whichever tile is asked for."""
    M, N, K = 256, 320, 128
    rng = np.random.default_rng(abs(ld) + tile)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (N, K), 0.1)
    def place(bits, form, lead):                       # -> (buffer, address of element (0, 0), leading dimension)
        rows = np.ascontiguousarray(bits.T if form else bits)
        n, width = rows.shape
        if not lead:
            t = dev_u16(rows)
            return t, t.data_ptr(), width
        buf = torch.zeros((n - 1) * abs(lead) + width, dtype=torch.int16, device=DEV)
        view = buf.as_strided((n, width), (abs(lead), 1))
        view.copy_(dev_u16(rows if lead > 0 else rows[::-1].copy()))
        return buf, buf.data_ptr() + (0 if lead > 0 else 2 * (n - 1) * -lead), lead
    abuf, ap, lda = place(Ab, a_form, ld if far == "a" else 0)
    wbuf, wp, ldw = place(Wb, w_form, ld if far == "w" else 0)
    Cd = torch.full((M + 1, N), 7.0, dtype=torch.float32, device=DEV)
    assert sp.spk_gemm(stream_ptr(), sp.EPI_F32, ap, lda, a_form, wp, ldw, w_form, ptr(Cd), N, None, 0, None, M, N, K, tile) == sp.SP_OK
    sync()
    ref = A @ W.T
    assert bool((Cd[M] == 7).all())
    assert np.max(np.abs(Cd[:M].cpu().numpy() - ref)) <= 2e-6 * np.sqrt(K) * np.max(np.abs(ref))      # as in test_gemm_transposed_operands


@pytest.mark.parametrize("M,N,K", [(1024, 4096, 64), (2560, 640, 320), (640, 640, 512), (512, 2048, 64), (2072, 1032, 256), (264, 40, 1088),
                                   (1032, 2560, 128)])
def test_gemm_transposed_operands_own_choice(M, N, K):
    """The backward forms with the library's own tile: few tokens (short contractions), narrow and wide outputs, ragged
    rows and columns.  One guard row behind C."""
    rng = np.random.default_rng(M + N + K)
    Ab, A = rand_bf16(rng, (M, K))
    Wb, W = rand_bf16(rng, (N, K), 0.1)
    Ad, ATd, WTd = dev_u16(Ab), dev_u16(Ab.T), dev_u16(Wb.T)
    ref = A @ W.T
    tol = 2e-6 * np.sqrt(K) * np.max(np.abs(ref))                          # as in test_gemm_transposed_operands
    for epi, a_form in ((sp.EPI_BF16, 0), (sp.EPI_F32, 0), (sp.EPI_F32, 1)):
        f32out = epi != sp.EPI_BF16
        Cd = torch.full((M + 1, N), 7.0 if f32out else 7, dtype=torch.float32 if f32out else torch.int16, device=DEV)
        assert sp.spk_gemm(stream_ptr(), epi, ptr(ATd if a_form else Ad), M if a_form else K, a_form, ptr(WTd), N, 1, ptr(Cd), N,
                           None, N, None, M, N, K, 0) == sp.SP_OK
        sync()
        out = Cd.cpu()
        assert bool((out[M] == 7).all())
        got = out[:M].numpy() if f32out else bf16_vals(host_u16(out[:M].contiguous()))
        assert np.all(np.abs(got - ref) <= tol + (0 if f32out else BF16_EPS * np.abs(ref))), (epi, a_form)


def test_gemm_rejects_shapes_it_cannot_take():
    z = torch.zeros(1 << 16, dtype=torch.int16, device=DEV)
    args = lambda M, N, K, lda=64, ldw=64, ldc=64: sp.spk_gemm(  # noqa: E731
        stream_ptr(), sp.EPI_BF16, ptr(z), lda, 0, ptr(z), ldw, 0, ptr(z), ldc, None, 0, None, M, N, K, 0)
    assert args(8, 8, 63) == sp.SP_ERR_INVALID_ARG        # K not a multiple of 64
    assert args(8, 7, 64) == sp.SP_ERR_INVALID_ARG        # N not a multiple of 8
    assert args(8, 8, 64, lda=60) == sp.SP_ERR_INVALID_ARG
    assert args(0, 8, 64) == sp.SP_OK                     # empty problem: nothing to do
    assert sp.spk_gemm(stream_ptr(), 9, ptr(z), 64, 0, ptr(z), 64, 0, ptr(z), 64, None, 0, None, 8, 8, 64, 0) == sp.SP_ERR_INVALID_ARG
    sync()


@pytest.mark.parametrize("T,f", [(33, 1024), (7, 11008), (1, 8)])
def test_swiglu(T, f):
    rng = np.random.default_rng(T + f)
    gb, g = rand_bf16(rng, (T, 2 * f), 2.0)
    z = torch.zeros((T, f), dtype=torch.int16, device=DEV)
    gd = dev_u16(gb)
    assert sp.spk_swiglu(stream_ptr(), ptr(gd), ptr(z), T, f) == sp.SP_OK
    sync()
    ref = O.silu(g[:, :f]) * g[:, f:]
    assert np.all(np.abs(bf16_vals(host_u16(z)) - ref) <= BF16_EPS * np.abs(ref) + 1e-6)


@pytest.mark.parametrize("B,S,Hq,Hkv,hd,causal", [
    (2, 128, 4, 4, 64, 1),      # the tiny workload's shape
    (3, 257, 4, 4, 80, 0),      # ViT-like: ragged S, head_dim 80, bidirectional
    (1, 300, 8, 2, 128, 1),     # grouped-query heads, ragged S
    (2, 64, 2, 1, 128, 0),
    (1, 1, 2, 2, 64, 1),        # a single token attends to itself
    (1, 129, 2, 2, 64, 1),      # one query past a block boundary
    (2, 33, 2, 2, 80, 1),       # head_dim 80 (padded 192-byte LDS rows), causal, less than one key tile
    (1, 1, 2, 1, 128, 0),
    (11, 520, 16, 4, 128, 1),   # enough work-groups for the paired causal blocks; ragged last key tile
    # head_dim 80 around the query-block (32 / 128) and key-tile (64) boundaries, a last key tile of 1, 32, 33, 63 and
    # 64 keys (few work-groups: from 105 tokens on 32 queries each)
    (2, 127, 2, 2, 80, 0), (1, 128, 2, 2, 80, 0), (2, 129, 2, 2, 80, 0), (1, 160, 2, 2, 80, 0), (1, 161, 2, 2, 80, 0),
    (2, 256, 2, 2, 80, 0), (2, 257, 16, 16, 80, 0), (1, 258, 2, 2, 80, 0), (1, 289, 4, 2, 80, 1), (1, 257, 2, 1, 80, 1),
    (1, 96, 2, 2, 80, 1), (1, 97, 2, 2, 80, 0),
    # ragged blocks at the other head dims
    (2, 77, 2, 2, 128, 1), (1, 520, 4, 2, 64, 1), (2, 33, 2, 2, 64, 0), (1, 289, 2, 2, 64, 0),
])
def test_attention(B, S, Hq, Hkv, hd, causal):
    rng = np.random.default_rng(B + S + Hq + hd + causal)
    nqkv = (Hq + 2 * Hkv) * hd
    qb, qkv = rand_bf16(rng, (B * S, nqkv))
    sh = O.StackShape(O.DECODER, 1, Hq * hd, Hq, Hkv, hd, 64, bool(causal))
    nq, nk = Hq * hd, Hkv * hd
    q, k, v = qkv[:, :nq], qkv[:, nq:nq + nk], qkv[:, nq + nk:]
    ref = O.attention(q, k, v, B, S, sh)
    o = torch.zeros((B * S, nq), dtype=torch.int16, device=DEV)
    lse = torch.zeros((B, Hq, S), dtype=torch.float32, device=DEV)
    qd = dev_u16(qb)
    rc = sp.spk_attention(stream_ptr(), ptr(qd), ptr(o), ptr(lse), B, S, Hq, Hkv, hd, causal)
    assert rc == sp.SP_OK
    sync()
    got = bf16_vals(host_u16(o))
    # probabilities and the output are each rounded to bf16 once
    assert np.max(np.abs(got - ref)) <= 3 * BF16_EPS * np.max(np.abs(ref))
    # log-sum-exp of the scaled, masked scores
    want = np.empty((B, Hq, S))
    for b in range(B):
        qb_ = q[b * S:(b + 1) * S].reshape(S, Hq, hd)
        kb_ = np.repeat(k[b * S:(b + 1) * S].reshape(S, Hkv, hd), Hq // Hkv, axis=1)
        s = np.einsum("ihd,jhd->hij", qb_, kb_) / np.sqrt(hd)
        if causal:
            s = np.where(np.arange(S)[None, :] <= np.arange(S)[:, None], s, -np.inf)
        m = s.max(-1)
        want[b] = m + np.log(np.exp(s - m[..., None]).sum(-1))
    # head_dim 80: the kernel takes the softmax denominator from the matrix pipe as the sum of the
    # bf16-ROUNDED probabilities (positive terms, each within 2^-9 of its value), so log(sum) is
    # within 2^-9 of the exact one; the other head dims add the fp32 probabilities
    atol = 2e-4 + (2.0 ** -9 if hd == 80 else 0.0)
    np.testing.assert_allclose(lse.cpu().numpy(), want, rtol=0, atol=atol * max(1.0, np.abs(want).max()))


@pytest.mark.parametrize("B,S,Hq,Hkv,hd", [
    (9, 296, 12, 3, 128),       # 324 work-groups, three blocks per head: heads straddle the batches of ids
    (3, 777, 16, 4, 64),        # 336, seven blocks per head
    (2, 1100, 17, 17, 80),      # 306, nine blocks per head, an odd number of heads
])
def test_attention_causal_writes_every_query_block(B, S, Hq, Hkv, hd):
    """More causal work-groups than one round of the chip, too few to be paired, and heads whose blocks do
    not divide the batches in which the walking direction alternates: every block once."""
    rng = np.random.default_rng(S)
    nq, nk = Hq * hd, Hkv * hd
    qb, qkv = rand_bf16(rng, (B * S, nq + 2 * nk))
    sh = O.StackShape(O.DECODER, 1, nq, Hq, Hkv, hd, 64, True)
    ref = O.attention(qkv[:, :nq], qkv[:, nq:nq + nk], qkv[:, nq + nk:], B, S, sh)
    o = torch.full((B * S, nq), 0x7FC1, dtype=torch.int16, device=DEV)      # bf16 NaN where nothing is written
    qd = dev_u16(qb)
    assert sp.spk_attention(stream_ptr(), ptr(qd), ptr(o), None, B, S, Hq, Hkv, hd, 1) == sp.SP_OK
    sync()
    got = bf16_vals(host_u16(o))
    assert np.max(np.abs(got - ref)) <= 3 * BF16_EPS * np.max(np.abs(ref))   # as in test_attention


@pytest.mark.parametrize("hd,Hq,Hkv,causal", [(64, 4, 2, 1), (64, 2, 2, 0), (80, 2, 2, 0), (80, 4, 2, 1), (128, 4, 1, 1), (128, 2, 2, 0)])
@pytest.mark.parametrize("S", [65, 95, 97, 193, 257, 319, 512, 513])
def test_attention_key_tiles_shared_by_waves(S, hd, Hq, Hkv, causal):
    """Few work-groups: waves with no key tile, one or several, ragged last tiles of 1, 32, 33 and 63 keys, queries that
    see none of a wave's keys; scores spread over tens of units, so that the waves' maxima differ widely, with the
    largest keys first or last."""
    rng = np.random.default_rng(S + hd + causal)
    nq, nk = Hq * hd, Hkv * hd
    _, qkv = rand_bf16(rng, (2 * S, nq + 2 * nk))
    grow = np.tile(np.linspace(0.1, 6.0, S), 2) if S % 2 else np.tile(np.linspace(6.0, 0.1, S), 2)
    qkv[:, nq:nq + nk] *= grow[:, None]
    t = torch.from_numpy(qkv).to(torch.bfloat16)
    qkv = t.to(torch.float64).numpy()
    sh = O.StackShape(O.DECODER, 1, nq, Hq, Hkv, hd, 64, bool(causal))
    ref = O.attention(qkv[:, :nq], qkv[:, nq:nq + nk], qkv[:, nq + nk:], 2, S, sh)
    o = torch.full((2 * S, nq), 0x7FC1, dtype=torch.int16, device=DEV)      # bf16 NaN where nothing is written
    qd = t.to(DEV)
    assert sp.spk_attention(stream_ptr(), ptr(qd), ptr(o), None, 2, S, Hq, Hkv, hd, causal) == sp.SP_OK
    sync()
    got = bf16_vals(host_u16(o))
    assert np.max(np.abs(got - ref)) <= 3 * BF16_EPS * np.max(np.abs(ref))   # as in test_attention


def attention_both(qkv, B, S, Hq, Hkv, hd, causal):
    """Kernel output and log-sum-exp over qkv (float64 of bf16 values, [B * S, ...]), and the same in float64."""
    nq, nk = Hq * hd, Hkv * hd
    o = torch.full((B * S, nq), 0x7FC1, dtype=torch.int16, device=DEV)      # bf16 NaN where nothing is written
    lse = torch.full((B, Hq, S), np.nan, dtype=torch.float32, device=DEV)
    qd = torch.from_numpy(qkv).to(torch.bfloat16).to(DEV)
    assert sp.spk_attention(stream_ptr(), ptr(qd), ptr(o), ptr(lse), B, S, Hq, Hkv, hd, causal) == sp.SP_OK
    sync()
    heads = lambda x, n: x.reshape(B, S, n, hd).transpose(0, 2, 1, 3)  # noqa: E731
    q, k, v = heads(qkv[:, :nq], Hq), heads(qkv[:, nq:nq + nk], Hkv), heads(qkv[:, nq + nk:], Hkv)
    k, v = np.repeat(k, Hq // Hkv, axis=1), np.repeat(v, Hq // Hkv, axis=1)
    s = q @ k.transpose(0, 1, 3, 2) / np.sqrt(hd)
    if causal:
        s = np.where(np.arange(S)[None, :] <= np.arange(S)[:, None], s, -np.inf)
    m = s.max(-1, keepdims=True)
    e = np.exp(s - m)
    ref = (e / e.sum(-1, keepdims=True)) @ v
    return (bf16_vals(host_u16(o)), lse.cpu().numpy().astype(np.float64), ref.transpose(0, 2, 1, 3).reshape(B * S, nq),
            (m + np.log(e.sum(-1, keepdims=True)))[..., 0])


def check_attention(qkv, B, S, Hq, Hkv, hd, causal):
    got, lse, ref, want = attention_both(qkv, B, S, Hq, Hkv, hd, causal)
    assert np.max(np.abs(got - ref)) <= 3 * BF16_EPS * np.max(np.abs(ref))                    # as in test_attention
    atol = 2e-4 + (2.0 ** -9 if hd == 80 else 0.0)
    np.testing.assert_allclose(lse, want, rtol=0, atol=atol * max(1.0, np.abs(want).max()))


def bf16_qkv(rng, B, S, Hq, Hkv, hd, grow=False):
    """Random activations; grow: keys that grow over the sequence (shrink for even S), scores spread over tens of units."""
    _, qkv = rand_bf16(rng, (B * S, (Hq + 2 * Hkv) * hd))
    if grow:
        f = np.linspace(0.1, 6.0, S)
        qkv[:, Hq * hd:(Hq + Hkv) * hd] *= np.tile(f if S % 2 else f[::-1], B)[:, None]
        qkv = torch.from_numpy(qkv).to(torch.bfloat16).to(torch.float64).numpy()
    return qkv


@pytest.mark.parametrize("hd,group,causal", [(64, 1, 0), (64, 2, 1), (80, 1, 0), (80, 2, 1), (128, 1, 0), (128, 4, 1)])
@pytest.mark.parametrize("S", [65, 95, 96, 97, 127, 129, 160, 161, 257, 289, 319])
def test_attention_many_work_groups(S, hd, group, causal):
    """Too many work-groups of 32 queries for the chip: 128 queries each, all waves over the same key tiles.  Last tiles of
    1, 31, 32, 33 and 63 keys (half a tile is worked where no more is left), query blocks with idle waves, the reference
    maximum moving late or never."""
    blocks = (S + 31) // 32
    heads = (512 // blocks // 2 + 1) * group // group + group
    Hq = (heads + group - 1) // group * group
    assert blocks * Hq * 2 > 512
    check_attention(bf16_qkv(np.random.default_rng(S + hd), 2, S, Hq, Hq // group, hd, grow=True), 2, S, Hq, Hq // group, hd, causal)


@pytest.mark.parametrize("B,S,Hq,hd,causal", [
    (2, 256, 16, 80, 0), (1, 256, 33, 80, 0), (1, 256, 32, 80, 1), (3, 256, 11, 80, 1),      # 256 and 264 work-groups of 32 queries
    (1, 104, 3, 80, 0), (1, 105, 3, 80, 0), (1, 104, 2, 80, 1), (1, 105, 2, 80, 1),          # the second tile's length
    (1, 64, 3, 64, 0), (1, 65, 3, 64, 0), (1, 64, 3, 128, 1), (1, 65, 3, 128, 1),            # one tile, two
    (2, 128, 64, 64, 0), (1, 128, 129, 64, 0), (4, 128, 32, 64, 1), (3, 128, 43, 64, 1),     # 512 and 516
    (1, 256, 32, 128, 0), (1, 256, 33, 128, 0), (1, 511, 16, 128, 1), (1, 511, 17, 128, 1),  # 256, 264 and 272
    (2, 512, 12, 128, 1), (1, 512, 25, 128, 1), (1, 1023, 12, 128, 1), (1, 1023, 13, 128, 1),  # 384, 400 and 416
    (1, 1024, 16, 128, 1), (1, 1024, 17, 128, 1),                                             # 512 and 544
])
def test_attention_both_sides_of_the_limits(B, S, Hq, hd, causal):
    check_attention(bf16_qkv(np.random.default_rng(S + Hq), B, S, Hq, Hq, hd), B, S, Hq, Hq, hd, causal)


@pytest.mark.parametrize("hd", [64, 80, 128])
@pytest.mark.parametrize("causal", [0, 1])
def test_attention_infinite_and_nan_scores(hd, causal):
    """Key tiles shared by waves: a key with a score of -inf takes no part, also where a wave sees no other; a NaN key reaches
    the queries that see it and no other."""
    B, S, H = 1, 321, 2
    qkv = bf16_qkv(np.random.default_rng(hd), B, S, H, H, hd)
    nq = H * hd
    qkv[:, 0] = np.abs(qkv[:, 0]) + 0.5                      # first head's queries: a positive element for the infinite keys
    off = np.r_[1:64, 128:192, 300]                          # (key 0 stays: a query that sees no finite score has no result)
    qkv[off, nq] = -np.inf
    qkv = torch.from_numpy(qkv).to(torch.bfloat16).to(torch.float64).numpy()     # + 0.5 left bf16
    with np.errstate(invalid="ignore"):
        got, lse, ref, want = attention_both(qkv, B, S, H, H, hd, causal)
    assert np.all(np.isfinite(got)) and np.all(np.isfinite(lse))
    assert np.max(np.abs(got - ref)) <= 3 * BF16_EPS * np.max(np.abs(ref))                    # as in test_attention
    atol = 2e-4 + (2.0 ** -9 if hd == 80 else 0.0)
    np.testing.assert_allclose(lse, want, rtol=0, atol=atol * max(1.0, np.abs(want).max()))
    clean = got
    qkv[200, nq + 1] = np.nan
    with np.errstate(invalid="ignore"):
        got, lse, ref, want = attention_both(qkv, B, S, H, H, hd, causal)
    hit = np.isnan(ref)
    assert hit.any() and np.array_equal(np.isnan(got), hit) and np.array_equal(np.isnan(lse), np.isnan(want))
    assert np.array_equal(got[~hit], clean[~hit])


def test_attention_rejects_unsupported_head_dim():
    z = torch.zeros(1 << 16, dtype=torch.int16, device=DEV)
    assert sp.spk_attention(stream_ptr(), ptr(z), ptr(z), None, 1, 8, 2, 2, 48, 1) == sp.SP_ERR_INVALID_ARG
    assert sp.spk_attention(stream_ptr(), ptr(z), ptr(z), None, 1, 8, 3, 2, 64, 1) == sp.SP_ERR_INVALID_ARG
    sync()


# ------------------------------------------------------------------ backward kernels
def test_mse_loss_and_gradient():
    rng = np.random.default_rng(3)
    n = 3 * 77 * 256
    y = rng.standard_normal(n).astype(np.float32)
    t = rng.standard_normal(n).astype(np.float32)
    yd, td = dev_f32(y), dev_f32(t)
    dy = torch.zeros(n, dtype=torch.float32, device=DEV)
    dyb = torch.zeros(n, dtype=torch.int16, device=DEV)
    scratch = torch.zeros(1024, dtype=torch.float32, device=DEV)
    loss = torch.zeros(1, dtype=torch.float32, device=DEV)
    assert sp.spk_mse(stream_ptr(), ptr(yd), ptr(td), ptr(dy), ptr(dyb), ptr(scratch), ptr(loss), n) == sp.SP_OK
    sync()
    ref = O.mse_loss(y.astype(np.float64), t.astype(np.float64))
    assert abs(float(loss.item()) - ref) <= 1e-5 * ref
    dref = 2.0 * (y.astype(np.float64) - t) / n
    np.testing.assert_allclose(dy.cpu().numpy(), dref, rtol=1e-5, atol=1e-12)
    assert np.all(np.abs(bf16_vals(host_u16(dyb)) - dref) <= BF16_EPS * np.abs(dref) + 1e-12)


@pytest.mark.parametrize("T,f", [(33, 1024), (5, 5504)])
def test_swiglu_backward(T, f):
    rng = np.random.default_rng(T + f)
    gb, gu = rand_bf16(rng, (T, 2 * f), 2.0)
    db, dz = rand_bf16(rng, (T, f))
    gud, dzd = dev_u16(gb), dev_u16(db)
    assert sp.spk_swiglu_bwd(stream_ptr(), ptr(dzd), ptr(gud), T, f) == sp.SP_OK
    sync()
    dg, du = O._swiglu_bwd(dz, gu[:, :f], gu[:, f:])
    got = bf16_vals(host_u16(gud))
    ref = np.concatenate([dg, du], axis=1)
    assert np.all(np.abs(got - ref) <= BF16_EPS * np.abs(ref) + 1e-6)


@pytest.mark.parametrize("T,d", [(300, 256), (37, 2048), (5, 8192), (700, 512),
                                 # 1024 rows and more of at most 2048 elements: one wave per row
                                 (1501, 2048), (1100, 320), (1024, 64), (2050, 1280)])
def test_rmsnorm_backward(T, d):
    rng = np.random.default_rng(T * 3 + d)
    da = rng.standard_normal((T, d)).astype(np.float32)
    h = (rng.standard_normal((T, d)) * 1.5).astype(np.float32)
    dh0 = rng.standard_normal((T, d)).astype(np.float32)
    gb, g = rand_bf16(rng, d, 0.3)
    dad, hd, gd, dhd = dev_f32(da), dev_f32(h), dev_u16(gb), dev_f32(dh0)
    dhb = torch.zeros((T, d), dtype=torch.int16, device=DEV)
    scratch = torch.zeros(256 * d, dtype=torch.float32, device=DEV)
    dgain = torch.zeros(d, dtype=torch.float32, device=DEV)
    rc = sp.spk_rmsnorm_bwd(stream_ptr(), ptr(dad), ptr(hd), ptr(gd), ptr(dhd), ptr(dhb), ptr(scratch), ptr(dgain),
                            T, d, 1e-5)
    assert rc == sp.SP_OK
    sync()
    dh_ref, dg_ref = O._rmsnorm_bwd(da.astype(np.float64), h.astype(np.float64), g, 1e-5)
    dh_ref = dh_ref + dh0
    got = dhd.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - dh_ref)) <= 1e-5 * np.max(np.abs(dh_ref))
    assert np.max(np.abs(dgain.cpu().numpy() - dg_ref)) <= 1e-5 * np.max(np.abs(dg_ref)) * np.sqrt(T)
    assert np.all(np.abs(bf16_vals(host_u16(dhb)) - got) <= BF16_EPS * np.abs(got) + 1e-12)


@pytest.mark.parametrize("B,S,Hq,Hkv,hd,causal", [
    (2, 128, 4, 4, 64, 1),
    (1, 300, 8, 2, 128, 1),     # grouped-query heads, ragged S
    (2, 77, 2, 2, 128, 0),
    (2, 257, 2, 2, 80, 0),
    (1, 33, 4, 1, 64, 1),
])
def test_attention_backward(B, S, Hq, Hkv, hd, causal):
    rng = np.random.default_rng(B * 5 + S + Hq + hd + causal)
    nq, nk = Hq * hd, Hkv * hd
    nqkv = nq + 2 * nk
    qb, qkv = rand_bf16(rng, (B * S, nqkv))
    dob, dO = rand_bf16(rng, (B * S, nq))
    sh = O.StackShape(O.DECODER, 1, nq, Hq, Hkv, hd, 64, bool(causal))
    q, k, v = qkv[:, :nq], qkv[:, nq:nq + nk], qkv[:, nq + nk:]
    dq, dk, dv = O._attention_bwd(dO, np.ascontiguousarray(q), np.ascontiguousarray(k), np.ascontiguousarray(v), B, S, sh)
    qd, dod = dev_u16(qb), dev_u16(dob)
    o = torch.zeros((B * S, nq), dtype=torch.int16, device=DEV)
    lse = torch.zeros((B, Hq, S), dtype=torch.float32, device=DEV)
    assert sp.spk_attention(stream_ptr(), ptr(qd), ptr(o), ptr(lse), B, S, Hq, Hkv, hd, causal) == sp.SP_OK
    scratch = torch.zeros(sp.spk_attention_bwd_scratch_bytes(B, S, Hq, Hkv, hd), dtype=torch.uint8, device=DEV)
    dqkv = torch.zeros((B * S, nqkv), dtype=torch.int16, device=DEV)
    rc = sp.spk_attention_bwd(stream_ptr(), ptr(qd), ptr(o), ptr(dod), ptr(lse), ptr(scratch), ptr(dqkv),
                              B, S, Hq, Hkv, hd, causal)
    assert rc == sp.SP_OK
    sync()
    got = bf16_vals(host_u16(dqkv))
    for name, g, r in (("dq", got[:, :nq], dq), ("dk", got[:, nq:nq + nk], dk), ("dv", got[:, nq + nk:], dv)):
        err = np.max(np.abs(g - r)) / np.max(np.abs(r))
        assert err <= 1.5e-2, (name, err)


@pytest.mark.parametrize("B,S,Hq,Hkv,hd,causal", [
    (1, 2, 2, 1, 128, 1), (1, 31, 2, 2, 128, 0), (1, 64, 2, 2, 128, 1), (1, 65, 2, 1, 128, 0), (2, 129, 2, 2, 128, 1),
    (1, 257, 4, 2, 128, 1), (1, 191, 2, 2, 128, 0),
    (1, 2, 2, 2, 80, 0), (1, 129, 2, 2, 80, 1), (1, 64, 2, 2, 80, 0), (2, 161, 2, 1, 80, 0),
    (1, 2, 2, 2, 64, 1), (1, 193, 4, 2, 64, 1), (1, 160, 2, 2, 64, 0), (1, 384, 2, 2, 64, 1),
])
def test_attention_backward_tile_edges(B, S, Hq, Hkv, hd, causal):
    """Around the 32-row halves, 64-row tiles and 128-row blocks: a last tile of 1, 31, 32, 33, 63, 64 rows, key
    blocks with idle key groups, fewer rows than a tile (the second half of the keys clamped), several heads per
    key head."""
    test_attention_backward(B, S, Hq, Hkv, hd, causal)


@pytest.mark.parametrize("T,d", [(300, 256), (37, 1280), (5, 8192), (700, 320)])
def test_layernorm_backward(T, d):
    rng = np.random.default_rng(T * 5 + d)
    da = rng.standard_normal((T, d)).astype(np.float32)
    h = (rng.standard_normal((T, d)) * 1.5 + 0.7).astype(np.float32)
    dh0 = rng.standard_normal((T, d)).astype(np.float32)
    gb, g = rand_bf16(rng, d, 0.3)
    dad, hd, gd, dhd = dev_f32(da), dev_f32(h), dev_u16(gb), dev_f32(dh0)
    dhb = torch.zeros((T, d), dtype=torch.int16, device=DEV)
    scratch = torch.zeros(256 * 2 * d, dtype=torch.float32, device=DEV)
    dgain = torch.zeros(d, dtype=torch.float32, device=DEV)
    dbias = torch.zeros(d, dtype=torch.float32, device=DEV)
    rc = sp.spk_layernorm_bwd(stream_ptr(), ptr(dad), ptr(hd), ptr(gd), ptr(dhd), ptr(dhb), ptr(scratch), ptr(dgain),
                              ptr(dbias), T, d, 1e-5)
    assert rc == sp.SP_OK
    sync()
    dh_ref, dg_ref, db_ref = O._layernorm_bwd(da.astype(np.float64), h.astype(np.float64), g, 1e-5)
    dh_ref = dh_ref + dh0
    got = dhd.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - dh_ref)) <= 1e-5 * np.max(np.abs(dh_ref))
    assert np.max(np.abs(dgain.cpu().numpy() - dg_ref)) <= 1e-5 * np.max(np.abs(dg_ref)) * np.sqrt(T)
    assert np.max(np.abs(dbias.cpu().numpy() - db_ref)) <= 1e-5 * np.max(np.abs(db_ref)) * np.sqrt(T)
    assert np.all(np.abs(bf16_vals(host_u16(dhb)) - got) <= BF16_EPS * np.abs(got) + 1e-12)


@pytest.mark.parametrize("T,d", [(1024, 64), (1024, 512), (1027, 516), (1501, 2048), (1100, 2052), (1030, 4096), (2050, 4100), (1025, 8192)])
def test_norm_backward_many_rows(T, d):
    """1024 rows and more: a row held by one, two or four waves (RMSNorm; LayerNorm up to 4096 elements), at
    and past each limit, row counts that leave the last work-groups short."""
    test_rmsnorm_backward(T, d)
    test_layernorm_backward(T, d)


@pytest.mark.parametrize("T,d", [(1024, 256), (2048, 1280), (1100, 4096)])
def test_layernorm_backward_many_rows_error(T, d):
    """The residual gradient of the many-rows form against float64, all operands N(0, 1): 4.6e-8 relative, as the
    row-per-work-group form has it.  One more rounding per element (the products with the gain taken from the row sums
    instead of being fused) gives 4.9e-8, the formula multiplied out 5.05e-8."""
    gen = torch.Generator(device=DEV).manual_seed(T + d)
    da, h, dh = (torch.randn(T, d, device=DEV, generator=gen) for _ in range(3))
    gain = (1 + 0.02 * torch.randn(d, device=DEV, generator=gen)).bfloat16()
    H = h.double().requires_grad_()
    torch.nn.functional.layer_norm(H, (d,), gain.double(), None, 1e-5).backward(da.double())
    ref = dh.double() + H.grad
    dhb, scratch = torch.zeros(T, d, dtype=torch.bfloat16, device=DEV), torch.zeros(256 * 2 * d + 4096, device=DEV)
    dg, db = torch.zeros(d, device=DEV), torch.zeros(d, device=DEV)
    assert sp.spk_layernorm_bwd(stream_ptr(), ptr(da), ptr(h), ptr(gain), ptr(dh), ptr(dhb), ptr(scratch), ptr(dg), ptr(db), T, d, 1e-5) == sp.SP_OK
    sync()
    err = float((dh.double() - ref).norm() / ref.norm())
    assert err <= 4.78e-8, err


@pytest.mark.parametrize("n", [8, 4096 * 33, 5120 * 7])
def test_gelu_and_its_backward(n):
    rng = np.random.default_rng(n)
    ub, u = rand_bf16(rng, n, 2.0)
    dzb, dz = rand_bf16(rng, n)
    ud, dzd = dev_u16(ub), dev_u16(dzb)
    z = torch.zeros(n, dtype=torch.int16, device=DEV)
    assert sp.spk_gelu(stream_ptr(), ptr(ud), ptr(z), n) == sp.SP_OK
    assert sp.spk_gelu_bwd(stream_ptr(), ptr(dzd), ptr(ud), n) == sp.SP_OK
    sync()
    zr = O.gelu(u)
    assert np.all(np.abs(bf16_vals(host_u16(z)) - zr) <= BF16_EPS * np.abs(zr) + 2e-7)
    # the derivative by central differences of the oracle's gelu in fp64
    e = 1e-6
    dref = dz * (O.gelu(u + e) - O.gelu(u - e)) / (2 * e)
    got = bf16_vals(host_u16(ud))
    assert np.all(np.abs(got - dref) <= BF16_EPS * np.abs(dref) + 1e-6 * np.abs(dz) + 1e-9)
    assert sp.spk_gelu(stream_ptr(), ptr(ud), ptr(z), 12) == sp.SP_ERR_INVALID_ARG


@pytest.mark.parametrize("T,n,ld", [(300, 256, 256), (1000, 3840, 3840), (37, 1280, 2560), (5, 2, 8)])
def test_column_sums(T, n, ld):
    rng = np.random.default_rng(T + n)
    sb, s = rand_bf16(rng, (T, ld))
    sd = dev_u16(sb)
    scratch = torch.zeros(256 * n, dtype=torch.float32, device=DEV)
    out = torch.zeros(n, dtype=torch.float32, device=DEV)
    assert sp.spk_colsum_bf16(stream_ptr(), ptr(sd), ld, T, n, ptr(scratch), ptr(out)) == sp.SP_OK
    sync()
    ref = s[:, :n].sum(axis=0)
    assert np.max(np.abs(out.cpu().numpy() - ref)) <= 1e-5 * np.sqrt(T) * max(np.max(np.abs(ref)), 1.0)
    assert sp.spk_colsum_bf16(stream_ptr(), ptr(sd), ld, T, 3, ptr(scratch), ptr(out)) == sp.SP_ERR_INVALID_ARG


@pytest.mark.parametrize("T,n,ld", [(8224, 1280, 1280), (4100, 264, 264), (31, 1280, 1280), (33, 520, 1040), (1, 8, 8),
                                    (257, 40, 48), (1000, 3844, 3844), (700, 264, 266)])
def test_column_sums_sixteen_byte_rows(T, n, ld):
    """Rows on 16 bytes: one and several column blocks, a ragged last one, fewer rows than a load round; widths
    and strides that are no multiple of eight stay with the 4-byte kernel."""
    test_column_sums(T, n, ld)
