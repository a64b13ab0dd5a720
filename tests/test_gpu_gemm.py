"""Dense projection GEMM parity (darts_gemm) against float64 products of the
same bf16 operands, over the decode batch sizes of a rollout (1 .. 512 rows,
prefill-sized M) and the decoder shapes, for every epilogue."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda"

from workload.gen import bf16_bits_from_f32, f32_from_bf16_bits


def _b():
    from paper_2605_30859_amd import binding
    binding.load_library()
    return binding


def silu(x):
    return x / (1.0 + np.exp(-x))


def _mk(rng, rows, cols, scale):
    bits = bf16_bits_from_f32((rng.standard_normal((rows, cols)) * scale).astype(np.float32))
    return bits, f32_from_bf16_bits(bits).astype(np.float64)


def _run(M, N, K, epi, seed=0, sample_rows=None):
    B = _b()
    rng = np.random.default_rng(seed + M * 7 + N + K)
    ab, a = _mk(rng, M, K, 1.0)
    wb, w = _mk(rng, N, K, 1.0 / np.sqrt(K))
    at = torch.from_numpy(ab.view(np.int16)).to(DEV)
    wt = torch.from_numpy(wb.view(np.int16)).to(DEV)
    if epi == 3:
        out = torch.zeros((M, N // 2), dtype=torch.int16, device=DEV)
    elif epi == 1:
        out = torch.zeros((M, N), dtype=torch.int16, device=DEV)
    else:
        init = rng.standard_normal((M, N)).astype(np.float32) if epi == 2 else np.zeros((M, N), np.float32)
        out = torch.from_numpy(init.copy()).to(DEV)
    wsb = B.darts_gemm_workspace_bytes(M, N, K)
    ws = torch.empty(max(wsb, 256), dtype=torch.uint8, device=DEV)
    B.darts_gemm(at, wt, out, M, N, K, B.DARTS_BF16, epi, ws)
    torch.cuda.synchronize()
    rows = np.arange(M) if sample_rows is None else np.unique(np.clip(sample_rows, 0, M - 1))
    ref = a[rows] @ w.T
    if epi == 3:
        got = f32_from_bf16_bits(out.cpu().numpy().view(np.uint16)[rows]).astype(np.float64)
        g = ref[:, [(c >> 4) * 32 + (c & 15) for c in range(N // 2)]]
        u = ref[:, [(c >> 4) * 32 + 16 + (c & 15) for c in range(N // 2)]]
        exp = silu(g) * u
        tol = 2 ** -7
    elif epi == 1:
        got = f32_from_bf16_bits(out.cpu().numpy().view(np.uint16)[rows]).astype(np.float64)
        exp = ref
        tol = 2 ** -7
    else:
        got = out.cpu().numpy()[rows].astype(np.float64)
        exp = ref + (init[rows] if epi == 2 else 0.0)
        tol = 1e-4
    scale = np.maximum(np.abs(exp).max(axis=1, keepdims=True), 1e-3)
    err = (np.abs(got - exp) / scale).max()
    assert err <= tol, (M, N, K, epi, err)


@pytest.mark.parametrize("M", [1, 5, 16, 17, 33, 64, 65, 100, 128, 129, 200, 256, 300, 512])
def test_gemm_qkv_shape_all_batch_sizes(M):
    print(f"gemm M={M}", flush=True)
    _run(M, 6144, 4096, 0)


@pytest.mark.parametrize("M,N,K,epi", [(512, 4096, 4096, 2), (37, 4096, 4096, 2),
                                       (512, 24576, 4096, 3), (9, 24576, 4096, 3), (130, 24576, 4096, 3),
                                       (512, 4096, 12288, 2), (3, 4096, 12288, 2), (200, 4096, 12288, 2),
                                       (64, 1536, 1024, 1), (300, 32000, 1024, 0), (1024, 5120, 2048, 0),
                                       # small-batch exact-fill tiles (64 and 128 rows, 64 and 96 wide),
                                       # every epilogue, with and without a K split
                                       (64, 4096, 4096, 2), (100, 4096, 4096, 2), (16, 4096, 12288, 2),
                                       (64, 4096, 12288, 2), (50, 24576, 4096, 3), (128, 24576, 4096, 3),
                                       (60, 6144, 4096, 1), (97, 6144, 4096, 1), (40, 8192, 1024, 3),
                                       (33, 2048, 4096, 2),
                                       # the Qwen3-30B-A3B attention projections (QKV, O with the
                                       # residual add) at 100-513 rows, with and without a K split
                                       (128, 5120, 2048, 0), (200, 5120, 2048, 0), (354, 5120, 2048, 0),
                                       (513, 5120, 2048, 0), (100, 2048, 4096, 2), (200, 2048, 4096, 2),
                                       (256, 2048, 4096, 2), (354, 2048, 4096, 2), (512, 2048, 4096, 2)])
def test_gemm_decoder_shapes(M, N, K, epi):
    print(f"gemm M={M} N={N} K={K} epi={epi}", flush=True)
    _run(M, N, K, epi)


def test_gemm_lm_head_full_size_sampled_rows():
    """LM head at the Qwen3-8B shape (151936 x 4096), 512 rows; sampled rows."""
    _run(512, 151936, 4096, 0, sample_rows=np.array([0, 1, 63, 64, 255, 256, 300, 511]))


def test_gemm_prefill_size_sampled_rows():
    """Prefill-sized M (32 prompts x 512 tokens) on the QKV shape; sampled rows."""
    _run(16384, 6144, 4096, 0, sample_rows=np.array([0, 1, 127, 128, 8191, 16000, 16383]))


@pytest.mark.parametrize("M,N,K,epi", [(4133, 6144, 512, 0), (4096, 4096, 256, 2), (8203, 6144, 256, 1),
                                       (4133, 8192, 1024, 3), (8195, 4096, 256, 3), (300, 24576, 4096, 3),
                                       (1030, 4096, 4096, 2), (2049, 4096, 12288, 2), (257, 24576, 256, 1)])
def test_gemm_large_tiles_every_row(M, N, K, epi):
    """256-row tiles on persistent blocks: several tiles per block, the last row
    tile nearly empty or full, the shortest K ranges, with and without a split.
    Every row against float64; rows past M are not written.  Tolerances: fp32
    sums of K products of order 1/sqrt(K), K*2^-24 at worst; bf16 results 2^-8,
    and the SwiGLU product's inputs as much again."""
    print(f"gemm large tiles M={M} N={N} K={K} epi={epi}", flush=True)
    B = _b()
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    a = torch.randn(M, K, device=DEV, generator=g).bfloat16()
    w = (torch.randn(N, K, device=DEV, generator=g) / K ** 0.5).bfloat16()
    cols = N // 2 if epi == 3 else N
    dt = torch.bfloat16 if epi in (1, 3) else torch.float32
    out = torch.full((M + 256, cols), 7.0, dtype=dt, device=DEV)
    init = out[:M].double()
    ws = torch.empty(max(B.darts_gemm_workspace_bytes(M, N, K), 256), dtype=torch.uint8, device=DEV)
    B.darts_gemm(a, w, out, M, N, K, B.DARTS_BF16, epi, ws)
    torch.cuda.synchronize()
    ref = a.double() @ w.double().T
    if epi == 3:
        ref = ref.view(M, N // 32, 2, 16)
        ref = (torch.nn.functional.silu(ref[:, :, 0]) * ref[:, :, 1]).reshape(M, cols)
    elif epi == 2:
        ref = ref + init
    err = (out[:M].double() - ref).abs()
    tol = 2 ** -8 * ref.abs() + 1e-3 if epi in (1, 3) else K * 2.0 ** -24 * (ref.abs() + 1.0)
    assert bool((err <= tol).all()), (M, N, K, epi, float((err - tol).max()))
    assert bool((out[M:] == 7.0).all())


@pytest.mark.parametrize("M,N,K,epi", [(1, 5, 1, 0), (17, 33, 7, 0), (16, 16, 130, 2), (33, 48, 516, 2), (2, 64, 20, 3),
                                       (35, 96, 1027, 3), (64, 1024, 128, 1)])
@pytest.mark.parametrize("shift", [0, 1])
def test_gemm_f32_any_size(M, N, K, epi, shift):
    """fp32 operands: tile remainders, K shorter and longer than the wavefronts'
    share, K and addresses that are not multiples of four (shift: A starts 4
    bytes off).  Against float64; tolerance K*2^-24 relative to the sum of
    magnitudes (the bound for a sum of K rounded products in any order), and
    four ulp more for the SwiGLU function."""
    print(f"gemm f32 M={M} N={N} K={K} epi={epi} shift={shift}", flush=True)
    B = _b()
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    buf = torch.randn(M * K + 1, device=DEV, generator=g)
    a = buf[shift:shift + M * K].view(M, K)
    w = torch.randn(N, K, device=DEV, generator=g)
    cols = N // 2 if epi == 3 else N
    out = torch.full((M + 16, cols), 3.0, device=DEV)
    B.darts_gemm(a, w, out, M, N, K, B.DARTS_F32, epi)
    torch.cuda.synchronize()
    ref, mag = a.double() @ w.double().T, a.double().abs() @ w.double().abs().T
    tol = (K + 2) * 2.0 ** -24 * mag
    if epi == 3:
        ref, tol = ref.view(M, N // 32, 2, 16), tol.view(M, N // 32, 2, 16)
        sg = torch.nn.functional.silu(ref[:, :, 0])
        # |silu'| <= 1.1
        tol = (1.1 * tol[:, :, 0] + 2.0 ** -21 * sg.abs()) * ref[:, :, 1].abs() + sg.abs() * tol[:, :, 1] + 1e-6
        ref, tol = (sg * ref[:, :, 1]).reshape(M, cols), tol.reshape(M, cols)
    elif epi == 2:
        ref, tol = ref + 3.0, tol + 2.0 ** -22 * (ref.abs() + 3.0)
    err = (out[:M].double() - ref).abs()
    assert bool((err <= tol).all()), float((err - tol).max())
    assert bool((out[M:] == 3.0).all())


@pytest.mark.parametrize("M,N,K,epi", [(259, 4500096, 2048, 0), (256, 4500096, 256, 2), (259, 8601600, 256, 1),
                                       (300, 256, 4 * 2 ** 21 + 2048, 0)])
def test_gemm_rows_beyond_32_bit_offsets(M, N, K, epi):
    """Rows of C or of the operands so long that 256 of them pass 4 GiB: every
    column of the rows at both ends of the tiles, and sampled columns of every
    row, against float64."""
    print(f"gemm long rows M={M} N={N} K={K} epi={epi}", flush=True)
    B = _b()
    g = torch.Generator(device=DEV).manual_seed(N + K)
    a = torch.empty(M, K, device=DEV, dtype=torch.bfloat16).normal_(generator=g)
    w = torch.empty(N, K, device=DEV, dtype=torch.bfloat16).normal_(0.0, K ** -0.5, generator=g)
    dt = torch.bfloat16 if epi == 1 else torch.float32
    out = torch.full((M, N), 7.0, dtype=dt, device=DEV)
    ws = torch.empty(max(B.darts_gemm_workspace_bytes(M, N, K), 256), dtype=torch.uint8, device=DEV)
    B.darts_gemm(a, w, out, M, N, K, B.DARTS_BF16, epi, ws)
    torch.cuda.synchronize()

    def check(rows, cols):
        ref = torch.zeros(len(rows), len(cols), dtype=torch.float64, device=DEV)
        for k0 in range(0, K, 1 << 16):     # float64 copies of a piece of K at a time
            ref += a[rows, k0:k0 + (1 << 16)].double() @ w[cols, k0:k0 + (1 << 16)].double().T
        if epi == 2:
            ref += 7.0
        err = (out[rows][:, cols].double() - ref).abs()
        # K roundings of partial sums of order 1, each within 2^-24: 16 times the
        # standard deviation of their sum; 16-bit results 2^-8 more
        tol = 16 * K ** 0.5 * 2.0 ** -24 * (ref.abs() + 1.0)
        if epi == 1:
            tol = tol + 2.0 ** -8 * ref.abs()
        assert bool((err <= tol).all()), (M, N, K, epi, float((err - tol).max()))

    every = torch.arange(M, device=DEV)
    cols = torch.randint(0, N, (min(N, 512),), device=DEV, generator=g)
    cols[0], cols[1] = 0, N - 1
    check(every, cols)
    ends = torch.tensor([r for r in (0, 239, 240, 255, 256, M - 1) if r < M], device=DEV)
    for c0 in range(0, N, 1 << 20):
        check(ends, torch.arange(c0, min(N, c0 + (1 << 20)), device=DEV))


@pytest.mark.parametrize("M,kind", [(129, 3), (300, 5), (1100, 4)])
@pytest.mark.parametrize("scale", [1.0, 30.0])
def test_swiglu_rows_do_not_depend_on_the_tile(M, kind, scale):
    """The SwiGLU projection in 256-row tiles (256x128, 256x192, 256x256) and in
    128-row tiles: while neither plan splits K, the sums run over K in the same
    order and a row's results are the same bit for bit.  scale 30: gates down to
    -100, where the quotient g / (1 + e^-g) becomes small and then zero."""
    print(f"swiglu tiles M={M} kind={kind} scale={scale}", flush=True)
    B = _b()
    N, K, part = 24576, 512, 100
    assert B.darts_debug_gemm_plan(M, N, K, 3)[::4] == (kind, 1)      # alternating groups
    assert B.darts_debug_gemm_plan(M, N, K, 3)[3] == 1 and B.darts_debug_gemm_plan(part, N, K, 3)[3:5] == (1, 0)
    g = torch.Generator(device=DEV).manual_seed(M)
    a = (torch.randn(M, K, device=DEV, generator=g) * scale).bfloat16()
    w = (torch.randn(N, K, device=DEV, generator=g) / K ** 0.5).bfloat16()
    whole = torch.empty(M, N // 2, dtype=torch.bfloat16, device=DEV)
    rows = torch.empty(part, N // 2, dtype=torch.bfloat16, device=DEV)
    B.darts_gemm(a, w, whole, M, N, K, B.DARTS_BF16, 3)
    for r0 in (0, M - part):
        B.darts_gemm(a[r0:r0 + part], w, rows, part, N, K, B.DARTS_BF16, 3)
        torch.cuda.synchronize()
        same = whole[r0:r0 + part].view(torch.int16) == rows.view(torch.int16)
        assert bool(same.all()), (M, kind, scale, r0, int((~same).sum()))


@pytest.mark.parametrize("M,epi", [(300, 1), (1100, 1), (300, 3), (1100, 3)])
def test_gemm_16_bit_results_at_any_element(M, epi):
    """16-bit results that start at an odd element: those of the large tiles are
    stored 16 bytes at a time and have to lie where an aligned call's lie."""
    print(f"gemm unaligned results M={M} epi={epi}", flush=True)
    B = _b()
    N, K = 24576, 512
    assert B.darts_debug_gemm_plan(M, N, K, epi)[3:5] == (1, 1)
    g = torch.Generator(device=DEV).manual_seed(M)
    a = torch.randn(M, K, device=DEV, generator=g).bfloat16()
    w = (torch.randn(N, K, device=DEV, generator=g) / K ** 0.5).bfloat16()
    cols = N // 2 if epi == 3 else N
    out = torch.empty(M * cols, dtype=torch.bfloat16, device=DEV)
    B.darts_gemm(a, w, out, M, N, K, B.DARTS_BF16, epi)
    for shift in (1, 2, 7):
        buf = torch.full((M * cols + 16,), 3.0, dtype=torch.bfloat16, device=DEV)
        B.darts_gemm(a, w, buf[shift:], M, N, K, B.DARTS_BF16, epi)
        torch.cuda.synchronize()
        assert bool((buf[shift:shift + M * cols] == out).all()), shift
        assert bool((buf[:shift] == 3.0).all()) and bool((buf[shift + M * cols:] == 3.0).all()), shift
