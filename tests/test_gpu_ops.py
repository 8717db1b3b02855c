"""Single-operator parity: each HIP kernel, called through the C ABI, against the oracle's plain
definition on the same seeded inputs (sizes span several tiles and ragged tails)."""
import pytest
import torch

from oracle import prefill_oracle as O
from paper_2602_16603_amd import inputs as I
from tests.util import TOL, max_rel_err

pytestmark = pytest.mark.gpu

DT = {"fp32": (0, torch.float32), "bf16": (1, torch.bfloat16)}


def _binding():
    from paper_2602_16603_amd import binding
    return binding


@pytest.mark.parametrize("name", ["bf16", "fp32"])
@pytest.mark.parametrize("m,n,k", [
    (1, 8, 8), (37, 520, 264), (256, 512, 256), (300, 1408, 256), (256, 256, 704),
    (1000, 256, 704), (513, 776, 1000), (4113, 4096, 512),
])
def test_gemm_matches_definition(name, m, n, k):
    B = _binding()
    code, td = DT[name]
    print(f"gemm {name} m={m} n={n} k={k}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 11, td, "cuda")
    w = I.normal_tensor((n, k), 0.05, 12, td, "cuda")
    c = torch.full((m, n), float("nan"), dtype=td, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_gemm(code, a.data_ptr(), w.data_ptr(), c.data_ptr(), m, n, k, False)
    torch.cuda.synchronize()
    ref = O.linear(a.cpu(), w.cpu())
    assert max_rel_err(c, ref) <= TOL[name]


@pytest.mark.parametrize("name", ["bf16", "fp32"])
@pytest.mark.parametrize("m,n,k", [(300, 264, 520), (4113, 4096, 256)])
def test_gemm_residual_accumulates_into_fp32(name, m, n, k):
    B = _binding()
    code, td = DT[name]
    print(f"gemm-residual {name} m={m} n={n} k={k}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 13, td, "cuda")
    w = I.normal_tensor((n, k), 0.05, 14, td, "cuda")
    x = I.normal_tensor((m, n), 1.0, 15, torch.float32, "cuda")
    x0 = x.clone()
    torch.cuda.synchronize()
    B.fp_op_gemm(code, a.data_ptr(), w.data_ptr(), x.data_ptr(), m, n, k, True)
    torch.cuda.synchronize()
    ref = x0.cpu().double() + O.linear(a.cpu(), w.cpu())
    assert max_rel_err(x, ref) <= TOL[name]


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m,n,k", [
    (2304, 2816, 64), (2304, 2816, 128), (2304, 2816, 192), (2560, 2560, 448), (2560, 2560, 576),
    (2560, 2560, 1088), (2561, 2568, 704), (2049, 3080, 1600),
])
def test_gemm_fast_path_trip_counts_and_ragged_edges(residual, m, n, k):
    """The 256x256-tile MFMA kernel on every path of its K loop (1, 2, 3, 7, 9, 11, 17 and 25
    k-tiles: single tiles, pairs, the eight-tile trip and their mixes), with a last row tile of
    one row and a last column tile of eight columns; rows behind the output must stay untouched."""
    B = _binding()
    print(f"gemm fast path residual={residual} m={m} n={n} k={k}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 21, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.05, 22, torch.bfloat16, "cuda")
    td = torch.float32 if residual else torch.bfloat16
    guard = 300
    buf = torch.full((m + guard, n), 7.0, dtype=td, device="cuda")
    if residual:
        buf[:m] = I.normal_tensor((m, n), 1.0, 23, torch.float32, "cuda")
    x0 = buf[:m].clone()
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), buf.data_ptr(), m, n, k, residual)
    torch.cuda.synchronize()
    ref = O.linear(a.cpu(), w.cpu())
    if residual:
        ref = ref + x0.cpu().double()
    assert max_rel_err(buf[:m], ref) <= TOL["bf16"]
    assert torch.all(buf[m:] == 7.0)


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m,n,k", [
    (512, 6144, 64), (300, 6152, 128), (257, 6152, 192), (512, 6152, 448), (257, 6152, 576), (130, 12296, 704),
    (257, 6152, 1088), (1, 12296, 1600),
])
def test_gemm_narrow_tile_trip_counts_and_ragged_edges(residual, m, n, k):
    """The 128-column tile that requests of up to two row tiles run on, uncut (no workspace), on
    every path of its K loop (1, 2, 3, 7, 9, 11, 17 and 25 k-tiles), with a last row tile of one
    row and a last column tile of eight columns; rows behind the output must stay untouched."""
    B = _binding()
    assert B.fp_op_gemm_workspace_bytes(1, m, n, k) == 0 or k >= 1024   # (short K: not cut even with a workspace)
    print(f"gemm narrow tile residual={residual} m={m} n={n} k={k}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 24, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.05, 25, torch.bfloat16, "cuda")
    td = torch.float32 if residual else torch.bfloat16
    guard = 300
    buf = torch.full((m + guard, n), 7.0, dtype=td, device="cuda")
    if residual:
        buf[:m] = I.normal_tensor((m, n), 1.0, 26, torch.float32, "cuda")
    x0 = buf[:m].clone()
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), buf.data_ptr(), m, n, k, residual)
    torch.cuda.synchronize()
    ref = O.linear(a.cpu(), w.cpu())
    if residual:
        ref = ref + x0.cpu().double()
    assert max_rel_err(buf[:m], ref) <= TOL["bf16"]
    assert torch.all(buf[m:] == 7.0)


def _random_gemm_shapes(count, seed):
    import random
    rng = random.Random(seed)
    ms = [1, 7, 63, 64, 65, 127, 128, 129, 255, 256, 257, 300, 511, 513, 777, 1024, 1500, 2049, 2560, 3001]
    ns = [8, 16, 64, 120, 128, 136, 248, 256, 264, 512, 520, 1000, 1024, 2048, 2056, 3072, 4104]
    ks = [8, 16, 24, 64, 72, 128, 192, 256, 320, 512, 1024, 1088, 2048, 4096]
    out = []
    while len(out) < count:
        m, n, k = rng.choice(ms), rng.choice(ns), rng.choice(ks)
        if m * n * k <= 6e9:
            out.append((m, n, k, rng.random() < 0.5))
    return out


@pytest.mark.parametrize("m,n,k,residual", _random_gemm_shapes(32, 20260216))
def test_gemm_seeded_random_shapes(m, n, k, residual):
    """Shapes drawn (seeded) across the dispatches of the bf16 GEMM that need no workspace -- the
    small-problem kernel and the 256x256-tile kernel -- with ragged rows, columns and K; rows
    before and behind the output must stay untouched.  (The split-K form is reached through
    fp_op_gemm_ws: test_gemm_split_k_with_workspace.)"""
    B = _binding()
    print(f"gemm random m={m} n={n} k={k} residual={residual}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 31, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.05, 32, torch.bfloat16, "cuda")
    td = torch.float32 if residual else torch.bfloat16
    g = 3
    buf = torch.full((m + 2 * g, n), 7.0, dtype=td, device="cuda")
    if residual:
        buf[g:g + m] = I.normal_tensor((m, n), 1.0, 33, torch.float32, "cuda")
    x0 = buf[g:g + m].clone()
    out = buf[g:g + m]
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), out.data_ptr(), m, n, k, residual)
    torch.cuda.synchronize()
    ref = O.linear(a.cpu(), w.cpu())
    if residual:
        ref = ref + x0.cpu().double()
    assert max_rel_err(out, ref) <= TOL["bf16"]
    assert torch.all(buf[:g] == 7.0) and torch.all(buf[g + m:] == 7.0)


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m,n,k", [
    (256, 6144, 4096), (1, 4096, 4096), (130, 4096, 14336), (1000, 4096, 4096), (512, 6144, 4096),
    (513, 4104, 1024), (200, 14336, 4096), (64, 5120, 27648), (777, 2056, 2048),
])
def test_gemm_split_k_with_workspace(residual, m, n, k):
    """Short requests (the 128-1024-token prompts of the trace) leave too few output tiles to fill
    the chip; with a workspace the GEMM is cut over K and a second kernel adds the partial sums in
    a fixed order.  Ragged M and N, guard rows before and behind the output, the workspace's own
    guard region untouched, the result against the definition and against the uncut form."""
    B = _binding()
    ws_bytes = B.fp_op_gemm_workspace_bytes(1, m, n, k)
    print(f"gemm split-K m={m} n={n} k={k} residual={residual} workspace={ws_bytes}", flush=True)
    assert ws_bytes > 0, "shape chosen for the split-K path does not split"
    a = I.normal_tensor((m, k), 1.0, 35, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.05, 36, torch.bfloat16, "cuda")
    td = torch.float32 if residual else torch.bfloat16
    g = 3
    buf = torch.full((m + 2 * g, n), 7.0, dtype=td, device="cuda")
    if residual:
        buf[g:g + m] = I.normal_tensor((m, n), 1.0, 37, torch.float32, "cuda")
    x0 = buf[g:g + m].clone()
    plain = x0.clone()
    out = buf[g:g + m]
    pad = 4096
    ws = torch.full((ws_bytes + pad,), 0x5A, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), out.data_ptr(), m, n, k, residual, ws.data_ptr(), ws_bytes)
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), plain.data_ptr(), m, n, k, residual)
    torch.cuda.synchronize()
    ref = O.linear(a.cpu(), w.cpu())
    if residual:
        ref = ref + x0.cpu().double()
    assert max_rel_err(out, ref) <= TOL["bf16"]
    assert max_rel_err(out, plain.cpu().double()) <= 1e-2          # same sums, another fp32 order
    assert torch.all(buf[:g] == 7.0) and torch.all(buf[g + m:] == 7.0)
    assert torch.all(ws[ws_bytes:] == 0x5A)
    again = x0.clone()                                              # fixed-order reduction: repeats bit for bit
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), again.data_ptr(), m, n, k, residual, ws.data_ptr(), ws_bytes)
    torch.cuda.synchronize()
    assert torch.equal(again, out)


@pytest.mark.parametrize("m,n,k", [(256, 4096, 4096), (1000, 4096, 14336), (130, 5120, 27648), (1, 4096, 4096), (513, 2056, 2048)])
def test_split_k_reduction_fused_with_rmsnorm_equals_the_two_operators(m, n, k):
    """Residual projection cut over K whose reduction kernel also normalises the updated row: the
    residual and the normalised rows carry the bits of fp_op_gemm_ws followed by fp_op_rmsnorm,
    and agree with the definition."""
    B = _binding()
    ws_bytes = B.fp_op_gemm_workspace_bytes(1, m, n, k)
    assert ws_bytes > 0
    a = I.normal_tensor((m, k), 1.0, 45, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.02, 46, torch.bfloat16, "cuda")
    gain = (1.0 + I.normal_tensor((n,), 0.1, 47, torch.float32, "cuda")).to(torch.bfloat16)
    x0 = I.normal_tensor((m, n), 1.0, 48, torch.float32, "cuda")
    ws = torch.empty((ws_bytes,), dtype=torch.uint8, device="cuda")
    x_two, x_fused = x0.clone(), x0.clone()
    h_two = torch.empty((m, n), dtype=torch.bfloat16, device="cuda")
    h_fused = torch.full((m + 2, n), 7.0, dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), x_two.data_ptr(), m, n, k, True, ws.data_ptr(), ws_bytes)
    B.fp_op_rmsnorm(1, x_two.data_ptr(), gain.data_ptr(), h_two.data_ptr(), m, n, 1e-5)
    B.fp_op_gemm_tail(a.data_ptr(), w.data_ptr(), x_fused.data_ptr(), m, n, k, True, ws.data_ptr(), ws_bytes,
                      B.FP_TAIL_RMSNORM, gain.data_ptr(), h_fused[1:].data_ptr(), 1e-5)
    torch.cuda.synchronize()
    assert torch.equal(x_fused, x_two) and torch.equal(h_fused[1:m + 1], h_two)
    assert torch.all(h_fused[0] == 7.0) and torch.all(h_fused[m + 1] == 7.0)
    x_ref = x0.cpu().double() + O.linear(a.cpu(), w.cpu())
    assert max_rel_err(x_fused, x_ref) <= TOL["bf16"]
    assert max_rel_err(h_fused[1:m + 1], O.rmsnorm(x_ref, gain.cpu(), 1e-5)) <= TOL["bf16"]


@pytest.mark.parametrize("m,f,k", [(256, 7168, 4096), (100, 2048, 4096), (64, 6912, 5120)])
def test_split_k_reduction_fused_with_swiglu_equals_the_two_operators(m, f, k):
    """gate_up projection cut over K whose reduction kernel applies SiLU(gate)*up: the bits of
    fp_op_gemm_ws into [M, 2F] followed by fp_op_silu_mul, without that intermediate."""
    B = _binding()
    ws_bytes = B.fp_op_gemm_workspace_bytes(1, m, 2 * f, k)
    assert ws_bytes > 0
    a = I.normal_tensor((m, k), 1.0, 49, torch.bfloat16, "cuda")
    w = I.normal_tensor((2 * f, k), 0.02, 50, torch.bfloat16, "cuda")
    ws = torch.empty((ws_bytes,), dtype=torch.uint8, device="cuda")
    gu = torch.empty((m, 2 * f), dtype=torch.bfloat16, device="cuda")
    two = torch.empty((m, f), dtype=torch.bfloat16, device="cuda")
    fused = torch.full((m + 1, f), 7.0, dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), gu.data_ptr(), m, 2 * f, k, False, ws.data_ptr(), ws_bytes)
    B.fp_op_silu_mul(1, gu.data_ptr(), two.data_ptr(), m, f)
    B.fp_op_gemm_tail(a.data_ptr(), w.data_ptr(), 0, m, 2 * f, k, False, ws.data_ptr(), ws_bytes,
                      B.FP_TAIL_SWIGLU, 0, fused.data_ptr())
    torch.cuda.synchronize()
    assert torch.equal(fused[:m], two) and torch.all(fused[m] == 7.0)
    ref = O.silu_mul(O.linear(a.cpu(), w.cpu()))
    assert max_rel_err(fused[:m], ref) <= TOL["bf16"]


def test_fused_tail_is_refused_when_the_problem_is_not_cut():
    B = _binding()
    m, n, k = 4096, 4096, 4096                        # fills the chip with output tiles: no split-K, no tail
    a = torch.zeros((m, k), dtype=torch.bfloat16, device="cuda")
    x = torch.zeros((m, n), dtype=torch.float32, device="cuda")
    ws = torch.empty((1 << 20,), dtype=torch.uint8, device="cuda")
    with pytest.raises(B.FlowPrefillError) as e:
        B.fp_op_gemm_tail(a.data_ptr(), a.data_ptr(), x.data_ptr(), m, n, k, True, ws.data_ptr(), 1 << 20,
                          B.FP_TAIL_RMSNORM, a.data_ptr(), a.data_ptr(), 1e-5)
    assert e.value.status == B.FP_ERR_INVALID


@pytest.mark.parametrize("name", ["bf16", "fp32"])
@pytest.mark.parametrize("t,d", [(1, 256), (77, 4096), (5, 5120), (3, 8200), (2, 20000)])
def test_rmsnorm_matches_definition(name, t, d):
    B = _binding()
    code, td = DT[name]
    x = I.normal_tensor((t, d), 3.0, 16, torch.float32, "cuda")
    g = (1.0 + I.normal_tensor((d,), 0.1, 17, torch.float32, "cuda")).to(td)
    out = torch.empty((t, d), dtype=td, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_rmsnorm(code, x.data_ptr(), g.data_ptr(), out.data_ptr(), t, d, 1e-5)
    torch.cuda.synchronize()
    ref = O.rmsnorm(x.cpu(), g.cpu(), 1e-5)
    assert max_rel_err(out, ref) <= TOL[name]


@pytest.mark.parametrize("name", ["bf16", "fp32"])
@pytest.mark.parametrize("t,f", [(1, 8), (33, 704), (7, 14336)])
def test_silu_mul_matches_definition(name, t, f):
    B = _binding()
    code, td = DT[name]
    gu = I.normal_tensor((t, 2 * f), 2.0, 18, td, "cuda")
    out = torch.empty((t, f), dtype=td, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_silu_mul(code, gu.data_ptr(), out.data_ptr(), t, f)
    torch.cuda.synchronize()
    ref = O.silu_mul(gu.cpu())
    assert max_rel_err(out, ref) <= TOL[name]


@pytest.mark.parametrize("m,f,k", [(8192, 14336, 4096), (1000, 14336, 4096), (3000, 1000, 256), (700, 27648, 5120),
                                   (2304, 1536, 64), (2305, 1544, 576),
                                   (256, 14336, 4096), (130, 14336, 4096), (200, 6152, 1024), (500, 3080, 512)])
def test_fused_gate_up_swiglu_equals_the_two_operators(m, f, k):
    """The gate_up GEMM with SiLU(gate)*up in its epilogue gives the bits of the GEMM followed by
    the stand-alone silu_mul (ragged M, an FFN width that is not a multiple of the 128-column
    tile, both 8B and 32B shapes; the last four shapes run on the 64-column tile of short
    requests), and both agree with the definition."""
    B = _binding()
    a = I.normal_tensor((m, k), 1.0, 40, torch.bfloat16, "cuda")
    w = I.normal_tensor((2 * f, k), 0.02, 41, torch.bfloat16, "cuda")
    gu = torch.empty((m, 2 * f), dtype=torch.bfloat16, device="cuda")
    two = torch.empty((m, f), dtype=torch.bfloat16, device="cuda")
    fused = torch.full((m, f), float("nan"), dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), gu.data_ptr(), m, 2 * f, k, False)
    B.fp_op_silu_mul(1, gu.data_ptr(), two.data_ptr(), m, f)
    B.fp_op_gemm_swiglu(a.data_ptr(), w.data_ptr(), fused.data_ptr(), m, f, k)
    torch.cuda.synchronize()
    assert torch.equal(fused, two)
    rows = torch.tensor(sorted(r for r in {0, 1, 255, 256, m // 2, m - 1} if r < m))
    ref = O.silu_mul(O.linear(a[rows].cpu().double(), w.cpu().double()))
    assert max_rel_err(fused[rows], ref) <= TOL["bf16"]


def test_fused_swiglu_rejects_small_problems():
    B = _binding()
    a = torch.zeros(64 * 64, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.FlowPrefillError):
        B.fp_op_gemm_swiglu(a.data_ptr(), a.data_ptr(), a.data_ptr(), 16, 64, 64)


def test_bad_sizes_are_rejected_not_launched():
    B = _binding()
    a = torch.zeros(64, device="cuda")
    with pytest.raises(B.FlowPrefillError):
        B.fp_op_gemm(1, a.data_ptr(), a.data_ptr(), a.data_ptr(), 4, 8, 12, False)   # K % 8
    with pytest.raises(B.FlowPrefillError):
        B.fp_op_gemm(1, a.data_ptr(), a.data_ptr(), a.data_ptr(), 0, 8, 8, False)
    with pytest.raises(B.FlowPrefillError):
        B.fp_op_rmsnorm(1, a.data_ptr(), a.data_ptr(), a.data_ptr(), 1, 12, 1e-5)


def test_mfma_ceiling_diagnostic_reports_a_plausible_rate():
    """The register-only MFMA loop cannot beat the vendor's dense bf16 peak and, on an idle chip,
    does not fall below a third of it."""
    B = _binding()
    rate = B.fp_diag_mfma_ceiling(100)
    assert 800.0 < rate < 2600.0
    with pytest.raises(B.FlowPrefillError):
        B.fp_diag_mfma_ceiling(0)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m,n,k", [(1, 8, 8), (31, 72, 40), (33, 64, 32), (300, 4096, 96), (65, 520, 72), (1024, 2056, 104), (1153, 5128, 136)])
def test_fp32_gemm_tiles_and_alignment(m, n, k, residual, offset):
    """The fp32 MFMA kernel on its three tiles (32x64, 64x64, 128x128: one row, one row more than a tile,
    eight columns more; one, two, three and more k-tiles with tails of 8 to 32), and, one float off the
    16-byte alignment, the plain kernel.  Rows before and behind the output stay untouched."""
    B = _binding()

    def put(t):
        buf = torch.empty(t.numel() + 4, device="cuda")
        view = buf[offset:offset + t.numel()].view(t.shape)
        view.copy_(t)
        return view

    a = put(I.normal_tensor((m, k), 1.0, 51, torch.float32, "cuda"))
    w = put(I.normal_tensor((n, k), 0.05, 52, torch.float32, "cuda"))
    c = put(torch.full((m + 2, n), 7.0, device="cuda"))
    if residual:
        c[1:m + 1] = I.normal_tensor((m, n), 1.0, 53, torch.float32, "cuda")
    x0 = c[1:m + 1].cpu().double()
    print(f"fp32 gemm m={m} n={n} k={k} residual={residual} offset={offset}", flush=True)
    torch.cuda.synchronize()
    B.fp_op_gemm(0, a.data_ptr(), w.data_ptr(), c[1:].data_ptr(), m, n, k, residual)
    torch.cuda.synchronize()
    ref = O.linear(a.cpu(), w.cpu())
    if residual:
        ref = ref + x0
    # k <= 136 fp32 products and sums: at most (k + 1) roundings of 2^-24 of the sum of magnitudes, itself
    # under 12 sqrt(k) times an element's spread (about 1e-4 of the largest result); observed 1e-7 .. 5e-7.
    assert max_rel_err(c[1:m + 1], ref) <= 1e-5
    assert torch.all(c[0] == 7.0) and torch.all(c[m + 1] == 7.0)


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m", [1, 31, 33, 64, 65, 128])
@pytest.mark.parametrize("n,k", [(12296, 64), (12296, 192), (4104, 1088), (2056, 4096)])
def test_gemm_of_few_rows(m, n, k, residual):
    """The kernel of up to 128 rows on its three row tiles (one row, a row less, a row more, all), uncut
    where the columns alone occupy the chip and cut over K otherwise, k-tiles behind the end of K (one and
    three of 64: the ring holds more) and a last column tile of eight columns: against the definition, and
    the uncut form bit for bit against the kernel of larger requests (the same sums in the same order, as for every
    projection whose columns all start at the beginning of K)."""
    B = _binding()
    print(f"few rows m={m} n={n} k={k} residual={residual}", flush=True)
    a = torch.zeros((200, k), dtype=torch.bfloat16, device="cuda")
    a[:m] = I.normal_tensor((m, k), 1.0, 61, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.05, 62, torch.bfloat16, "cuda")
    td = torch.float32 if residual else torch.bfloat16
    buf = torch.full((m + 200, n), 7.0, dtype=td, device="cuda")
    if residual:
        buf[:m] = I.normal_tensor((m, n), 1.0, 63, torch.float32, "cuda")
    x0 = buf[:m].clone()
    large = torch.zeros((200, n), dtype=td, device="cuda")
    large[:m] = x0 if residual else 0
    ws_bytes = B.fp_op_gemm_workspace_bytes(1, m, n, k)
    ws = torch.full((ws_bytes + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), buf.data_ptr(), m, n, k, residual, ws.data_ptr(), ws_bytes)
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), large.data_ptr(), 200, n, k, residual)
    torch.cuda.synchronize()
    ref = O.linear(a[:m].cpu(), w.cpu())
    if residual:
        ref = ref + x0.cpu().double()
    assert max_rel_err(buf[:m], ref) <= TOL["bf16"]
    assert torch.all(buf[m:] == 7.0) and torch.all(ws[ws_bytes:] == 0x5A)
    if ws_bytes == 0:
        assert torch.equal(buf[:m], large[:m])


@pytest.mark.parametrize("m,f,k", [(m, f, k) for f, k in [(6152, 128), (7176, 704)] for m in (1, 32, 64, 127)] +
                                  [(m, 20488, k) for m in (65, 127, 128) for k in (64, 320, 1216)] +
                                  [(m, 6152, 448) for m in (70, 180, 370)])
def test_fused_gate_up_swiglu_of_few_rows(m, f, k):
    """SiLU(gate)*up in the epilogue of the few-rows kernel (up to 64 rows; 65 to 128 where 20488 outputs fill the chip with wide tiles,
    the plain projection then on the large kernel up to K = 1152) and of the 128-column tile on 96, 128 and 192 rows: the bits of
    the two operators."""
    B = _binding()
    a = I.normal_tensor((m, k), 1.0, 64, torch.bfloat16, "cuda")
    w = I.normal_tensor((2 * f, k), 0.02, 65, torch.bfloat16, "cuda")
    gu = torch.empty((m, 2 * f), dtype=torch.bfloat16, device="cuda")
    two = torch.empty((m, f), dtype=torch.bfloat16, device="cuda")
    fused = torch.full((m + 1, f), 7.0, dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), gu.data_ptr(), m, 2 * f, k, False)
    B.fp_op_silu_mul(1, gu.data_ptr(), two.data_ptr(), m, f)
    B.fp_op_gemm_swiglu(a.data_ptr(), w.data_ptr(), fused.data_ptr(), m, f, k)
    torch.cuda.synchronize()
    assert torch.equal(fused[:m], two) and torch.all(fused[m] == 7.0)
    assert max_rel_err(fused[:m], O.silu_mul(O.linear(a.cpu(), w.cpu()))) <= TOL["bf16"]


@pytest.mark.parametrize("m", [1, 32, 33, 64, 65, 256, 257, 512])
@pytest.mark.parametrize("f,k", [(6272, 2048), (6272, 3200), (7168, 3136), (6400, 16384)])
def test_gate_up_whose_columns_start_at_different_k(m, f, k):
    """Up to two row tiles on the few-rows and the 128-column tile, long rows: every group of 128 columns starts at another k (49
    and 50 groups over 16, 25 and 128 starts; none where K is no multiple of 128, whose last k-tile of 128 is half empty). The
    fused form has the bits of the two operators, and each value is as near its definition as its roundings are."""
    B = _binding()
    print(f"starts m={m} f={f} k={k}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 104, torch.bfloat16, "cuda")
    w = I.normal_tensor((2 * f, k), 0.02, 105, torch.bfloat16, "cuda")
    gu = torch.full((m + 1, 2 * f), 7.0, dtype=torch.bfloat16, device="cuda")
    two = torch.empty((m, f), dtype=torch.bfloat16, device="cuda")
    fused = torch.full((m + 1, f), 7.0, dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), gu.data_ptr(), m, 2 * f, k, False)
    B.fp_op_silu_mul(1, gu.data_ptr(), two.data_ptr(), m, f)
    B.fp_op_gemm_swiglu(a.data_ptr(), w.data_ptr(), fused.data_ptr(), m, f, k)
    torch.cuda.synchronize()
    assert torch.equal(fused[:m], two) and torch.all(fused[m] == 7.0) and torch.all(gu[m] == 7.0)
    ref = a.double() @ w.double().T
    # bf16 rounding 2^-9 of a row's values; sums of up to 16384 products of about 0.02 in fp32, 32 at a time: 1e-6.  A k-tile left out or
    # taken twice is 1/256 of K or more, 6e-2 of a row.
    err = (gu[:m].double() - ref).norm(dim=1) / ref.norm(dim=1)
    assert err.max().item() <= 4e-3, (err.argmax().item(), err.max().item())
    assert max_rel_err(fused[:m], torch.nn.functional.silu(ref[:, :f]) * ref[:, f:]) <= TOL["bf16"]


@pytest.mark.parametrize("n,k,last", [(12544, 2048, 512), (12544, 3200, 512), (14336, 4096, 512), (20736, 2048, 256)])
def test_a_row_has_one_result_for_all_sizes_that_start_alike(n, k, last):
    """An uncut projection whose columns start at different k (49, 49, 56 and 81 groups) adds a row's products up in one order for
    all sizes that do so (up to two row tiles, up to one where two fill the chip with wide tiles), whatever tile they run on: the
    same bits from 1 to 512 or 256 rows.  Larger ones start at the beginning, and so does a residual one of any size: another
    order of the same sums."""
    B = _binding()
    a = I.normal_tensor((600, k), 1.0, 106, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.02, 107, torch.bfloat16, "cuda")
    ref = a.double() @ w.double().T
    rows = {}
    for m in (last, last + 1, 1, 20, 32, 50, 64, 65, 100, 128, 200, 256, 300, 512, 600):
        print(f"one result m={m} n={n} k={k}", flush=True)
        rows[m] = torch.full((m + 1, n), 7.0, dtype=torch.bfloat16, device="cuda")
        torch.cuda.synchronize()
        B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), rows[m].data_ptr(), m, n, k, False)
        torch.cuda.synchronize()
        assert torch.all(rows[m][m] == 7.0)
        alike = rows[last if m <= last else last + 1]
        both = min(m, alike.shape[0] - 1)
        assert torch.equal(rows[m][:both], alike[:both]), m
    # Sums of up to 4096 products in fp32, 32 at a time: a random walk of 128 roundings of 2^-24 of the running sum, 7e-7 of a row;
    # at bf16's 2^-9 that moves one value in a thousand or so to the neighbouring one.
    assert (rows[600][:last] != rows[last][:last]).float().mean().item() <= 4e-3
    for m in (last, 600):
        err = (rows[m][:m].double() - ref[:m]).norm(dim=1) / ref[:m].norm(dim=1)
        assert err.max().item() <= 4e-3                # bf16 rounding: 2^-9 at most of a value, 2^-9 / sqrt(3) in the mean square
    one, many = (torch.zeros((m, n), device="cuda") for m in (50, 600))
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), one.data_ptr(), 50, n, k, True)
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), many.data_ptr(), 600, n, k, True)
    torch.cuda.synchronize()
    assert torch.equal(one, many[:50]) and torch.equal(many.bfloat16()[:600], rows[600][:600])


@pytest.mark.parametrize("m,n,k", [(777, 6144, 1088), (513, 7824, 2048), (1024, 4096, 1600), (600, 5136, 1024)])
@pytest.mark.parametrize("residual", [False, True])
def test_three_and_four_row_tiles_on_the_narrow_tile(m, n, k, residual):
    """Problems of three and four row tiles with a short K run on the 128-column tile in fewer K ranges,
    or uncut: against the definition; uncut, the bits of the call without a workspace.  The workspace
    asked for is still enough and its guard stays untouched."""
    B = _binding()
    ws_bytes = B.fp_op_gemm_workspace_bytes(1, m, n, k)
    assert ws_bytes > 0
    a = I.normal_tensor((m, k), 1.0, 66, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.05, 67, torch.bfloat16, "cuda")
    td = torch.float32 if residual else torch.bfloat16
    x0 = I.normal_tensor((m, n), 1.0, 68, td, "cuda")
    buf = torch.full((m + 2, n), 7.0, dtype=td, device="cuda")
    buf[1:m + 1] = x0
    plain = x0.clone()
    ws = torch.full((ws_bytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    print(f"narrow cut m={m} n={n} k={k} residual={residual}", flush=True)
    torch.cuda.synchronize()
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), buf[1:].data_ptr(), m, n, k, residual, ws.data_ptr(), ws_bytes)
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), plain.data_ptr(), m, n, k, residual)
    torch.cuda.synchronize()
    ref = O.linear(a.cpu(), w.cpu())
    if residual:
        ref = ref + x0.cpu().double()
    assert max_rel_err(buf[1:m + 1], ref) <= TOL["bf16"]
    assert torch.all(buf[0] == 7.0) and torch.all(buf[m + 1] == 7.0) and torch.all(ws[ws_bytes:] == 0x5A)
    if not residual and 184 <= ((m + 255) // 256) * ((n + 127) // 128) <= 256:       # the tiles alone occupy the chip: one range
        assert torch.equal(buf[1:m + 1], plain)
    if not residual:                                              # the SwiGLU tail, cut or not: the two operators' bits
        two = torch.empty((m, n // 2), dtype=torch.bfloat16, device="cuda")
        fused = torch.empty_like(two)
        B.fp_op_silu_mul(1, buf[1:].data_ptr(), two.data_ptr(), m, n // 2)
        B.fp_op_gemm_tail(a.data_ptr(), w.data_ptr(), 0, m, n, k, False, ws.data_ptr(), ws_bytes, B.FP_TAIL_SWIGLU, 0, fused.data_ptr())
        torch.cuda.synchronize()
        assert torch.equal(fused, two)


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m,n,k", [(2560, 2560, 8), (2305, 2568, 72), (2304, 2816, 136), (2305, 2568, 200), (2049, 3080, 632), (4100, 1544, 1016), (8200, 520, 2040),
                                   (3329, 3080, 8), (3329, 3080, 72), (3329, 3080, 136), (3329, 3080, 200), (3329, 3080, 632), (4100, 2568, 1016), (8200, 1288, 2040)])
def test_gemm_odd_k_on_the_large_tile(m, n, k, residual):
    """K not a multiple of 64 on the 256x256 tile (0, 1, 2, 3, 9, 15 and 31 whole k-tiles and a tail of 8 or 56
    columns), a last row tile of one row and a last column tile of eight columns: the columns of W and A
    behind K belong to the next row and must not enter.  The first seven problems, of about 100 such tiles, run on the
    128x128 tiles that are ahead there, the others on the large one (tests/test_gemm_plan.py)."""
    B = _binding()
    print(f"gemm odd k m={m} n={n} k={k} residual={residual}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 72, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.05, 73, torch.bfloat16, "cuda")
    td = torch.float32 if residual else torch.bfloat16
    buf = torch.full((m + 300, n), 7.0, dtype=td, device="cuda")
    if residual:
        buf[:m] = I.normal_tensor((m, n), 1.0, 74, torch.float32, "cuda")
    x0 = buf[:m].clone()
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), buf.data_ptr(), m, n, k, residual)
    torch.cuda.synchronize()
    ref = O.linear(a.cpu(), w.cpu())
    if residual:
        ref = ref + x0.cpu().double()
    assert max_rel_err(buf[:m], ref) <= TOL["bf16"]
    # One dropped or foreign column would be off by sqrt(1/k) of the result: far above the bf16 rounding of 2^-9.
    assert ((buf[:m].cpu().double() - ref).norm() / ref.norm()).item() <= 4e-3
    assert torch.all(buf[m:] == 7.0)


def _at(tensor, offset):
    """A copy of the tensor whose first element lies `offset` elements behind a 256-byte boundary, and its buffer."""
    buf = torch.full((offset + tensor.numel() + 64,), 7.0, dtype=tensor.dtype, device="cuda")
    view = buf[offset:offset + tensor.numel()].view(tensor.shape)
    view.copy_(tensor)
    return view, buf


@pytest.mark.parametrize("offset", [1, 2, 4])
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m,n,k", [(50, 4104, 1088), (100, 12296, 64), (300, 2056, 4096), (600, 5136, 1024), (2560, 2568, 128), (2305, 2568, 72), (33, 72, 40)])
def test_bf16_gemm_operands_off_the_16_byte_grid(m, n, k, residual, offset):
    """Operands 2, 4 and 8 bytes off (views of a larger buffer): few rows, cut over K on either tile, uncut large, odd K,
    small.  Against the definition; what lies before and behind the output stays untouched."""
    B = _binding()
    a, _ = _at(I.normal_tensor((m, k), 1.0, 81, torch.bfloat16, "cuda"), offset)
    w, _ = _at(I.normal_tensor((n, k), 0.05, 82, torch.bfloat16, "cuda"), offset)
    x0 = I.normal_tensor((m, n), 1.0, 83, torch.float32 if residual else torch.bfloat16, "cuda")
    c, buf = _at(x0, offset)
    ws_bytes = B.fp_op_gemm_workspace_bytes(1, m, n, k)
    ws = torch.full((ws_bytes + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    print(f"unaligned gemm m={m} n={n} k={k} residual={residual} offset={offset}", flush=True)
    torch.cuda.synchronize()
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), c.data_ptr(), m, n, k, residual, ws.data_ptr(), ws_bytes)
    torch.cuda.synchronize()
    ref = O.linear(a.cpu(), w.cpu())
    if residual:
        ref = ref + x0.cpu().double()
    assert max_rel_err(c, ref) <= TOL["bf16"]
    # bf16 rounding of the result is 2^-9 at most; a chunk fetched from a neighbouring address would be off by its share of K.
    assert ((c.cpu().double() - ref).norm() / ref.norm()).item() <= 4e-3
    assert torch.all(buf[:offset] == 7.0) and torch.all(buf[offset + c.numel():] == 7.0) and torch.all(ws[ws_bytes:] == 0x5A)


@pytest.mark.parametrize("offset", [1, 2, 4])
@pytest.mark.parametrize("m", [50, 200, 300])
def test_bf16_fused_operators_off_the_16_byte_grid(m, offset):
    """The fused gate_up projection and both tails of a cut projection on operands 2, 4 and 8 bytes off: the bits of the
    separate operators on the same operands."""
    B = _binding()
    f, k = 7176, 704
    a, _ = _at(I.normal_tensor((m, k), 1.0, 84, torch.bfloat16, "cuda"), offset)
    w, _ = _at(I.normal_tensor((2 * f, k), 0.02, 85, torch.bfloat16, "cuda"), offset)
    gu, _ = _at(torch.zeros((m, 2 * f), dtype=torch.bfloat16, device="cuda"), offset)
    two = torch.empty((m, f), dtype=torch.bfloat16, device="cuda")
    fused, buf = _at(torch.zeros((m, f), dtype=torch.bfloat16, device="cuda"), offset)
    print(f"unaligned fused m={m} offset={offset}", flush=True)
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), gu.data_ptr(), m, 2 * f, k, False)
    gu_copy = gu.clone()
    torch.cuda.synchronize()
    B.fp_op_silu_mul(1, gu_copy.data_ptr(), two.data_ptr(), m, f)
    B.fp_op_gemm_swiglu(a.data_ptr(), w.data_ptr(), fused.data_ptr(), m, f, k)
    torch.cuda.synchronize()
    assert torch.equal(fused, two)
    assert torch.all(buf[:offset] == 7.0) and torch.all(buf[offset + fused.numel():] == 7.0)

    n, k = 4096, 4096                                  # cut over K: the tails of the reduction
    ws_bytes = B.fp_op_gemm_workspace_bytes(1, m, n, k)
    assert ws_bytes > 0
    ws = torch.full((ws_bytes + 256,), 0x5A, dtype=torch.uint8, device="cuda")
    a, _ = _at(I.normal_tensor((m, k), 1.0, 86, torch.bfloat16, "cuda"), offset)
    w, _ = _at(I.normal_tensor((n, k), 0.05, 87, torch.bfloat16, "cuda"), offset)
    gain = I.normal_tensor((n,), 1.0, 88, torch.bfloat16, "cuda")
    x = I.normal_tensor((m, n), 1.0, 89, torch.float32, "cuda")
    plain, tailed = x.clone(), x.clone()
    h, h_tail = (torch.empty((m, n), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    gu, _ = _at(torch.zeros((m, n), dtype=torch.bfloat16, device="cuda"), offset)
    act, act_tail = (torch.empty((m, n // 2), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), plain.data_ptr(), m, n, k, True, ws.data_ptr(), ws_bytes)
    B.fp_op_rmsnorm(1, plain.data_ptr(), gain.data_ptr(), h.data_ptr(), m, n, 1e-5)
    B.fp_op_gemm_tail(a.data_ptr(), w.data_ptr(), tailed.data_ptr(), m, n, k, True, ws.data_ptr(), ws_bytes, B.FP_TAIL_RMSNORM, gain.data_ptr(), h_tail.data_ptr(), 1e-5)
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), gu.data_ptr(), m, n, k, False, ws.data_ptr(), ws_bytes)
    gu_copy = gu.clone()
    torch.cuda.synchronize()
    B.fp_op_silu_mul(1, gu_copy.data_ptr(), act.data_ptr(), m, n // 2)
    B.fp_op_gemm_tail(a.data_ptr(), w.data_ptr(), 0, m, n, k, False, ws.data_ptr(), ws_bytes, B.FP_TAIL_SWIGLU, 0, act_tail.data_ptr())
    torch.cuda.synchronize()
    assert torch.equal(tailed, plain) and torch.equal(h_tail, h) and torch.equal(act_tail, act)
    ref = O.linear(a.cpu(), w.cpu()) + x.cpu().double()
    assert max_rel_err(tailed, ref) <= TOL["bf16"] and torch.all(ws[ws_bytes:] == 0x5A)


LARGE_TILE_SIZES = [          # rows of the tile, epilogue, m (one to three rows past the last whole tile, or as many short of one), n, k
    (128, "bf16", 2051, 7184, 64), (160, "bf16", 1283, 6672, 64), (192, "bf16", 5762, 1544, 64), (224, "bf16", 5379, 2064, 64),
    (256, "bf16", 5634, 2320, 64), (128, "bf16", 2430, 6408, 576), (160, "bf16", 5759, 1544, 576),
    (192, "bf16", 4029, 2320, 576), (224, "bf16", 1566, 7176, 576), (256, "bf16", 5631, 2320, 576),
    (128, "residual", 2049, 7184, 64), (160, "residual", 1282, 6920, 64), (192, "residual", 5761, 1560, 64),
    (224, "residual", 4931, 2312, 64), (256, "residual", 5633, 2312, 64), (128, "residual", 4990, 3088, 576),
    (160, "residual", 1117, 7960, 576), (192, "residual", 1342, 7176, 576), (224, "residual", 4927, 2312, 576),
    (256, "residual", 2047, 6424, 576), (128, "swiglu", 1537, 4616, 64), (160, "swiglu", 801, 5112, 64),
    (192, "swiglu", 3073, 1552, 64), (224, "swiglu", 1346, 4112, 64), (256, "swiglu", 1795, 3600, 64),
    (128, "swiglu", 1406, 5400, 576), (160, "swiglu", 799, 5112, 576), (192, "swiglu", 4607, 1040, 576),
    (224, "swiglu", 4478, 1288, 576), (256, "swiglu", 1022, 6664, 576),
    (128, "bf16", 258, 20232, 832), (160, "bf16", 801, 10000, 832), (128, "residual", 257, 20232, 832), (160, "residual", 799, 9992, 832),
    (128, "swiglu", 258, 10120, 832), (160, "swiglu", 798, 5008, 832), (128, "bf16", 259, 20232, 896), (160, "bf16", 801, 10256, 896),
    (128, "residual", 257, 20504, 896), (160, "residual", 801, 10008, 896), (128, "swiglu", 382, 10264, 896), (160, "swiglu", 803, 5272, 896),
    (128, "bf16", 383, 20504, 1536), (160, "bf16", 1118, 7944, 1536), (128, "residual", 383, 20496, 1536), (160, "residual", 798, 9992, 1536),
    (128, "swiglu", 259, 10264, 1536), (160, "swiglu", 799, 5008, 1536), (128, "bf16", 257, 20232, 2560), (160, "bf16", 798, 9992, 2560),
    (128, "residual", 257, 20496, 2560), (160, "residual", 802, 10000, 2560), (128, "swiglu", 258, 10128, 2560), (160, "swiglu", 802, 5000, 2560)]


@pytest.mark.parametrize("rows,epilogue,m,n,k", LARGE_TILE_SIZES)
def test_large_tile_of_every_height(rows, epilogue, m, n, k):
    """An uncut projection on the large tile of 128 to 256 rows (tests/test_gemm_plan.py checks which): one k-tile and nine, a
    nearly empty and a nearly full last row tile, a last column tile of one or two column blocks; on 128 and 160 rows also 13
    and 14 k-tiles, and 24 and 40 with the L2 warm-up; rows behind M stay."""
    B = _binding()
    print(f"large tile rows={rows} {epilogue} m={m} n={n} k={k}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 91, torch.bfloat16, "cuda")
    w = I.normal_tensor((2 * n if epilogue == "swiglu" else n, k), 0.1, 92, torch.bfloat16, "cuda")
    c = torch.full((m + 256, n), 7.0, dtype=torch.float32 if epilogue == "residual" else torch.bfloat16, device="cuda")
    ref = a.double() @ w.double().T
    if epilogue == "residual":
        c[:m] = I.normal_tensor((m, n), 1.0, 93, torch.float32, "cuda")
        ref += c[:m].double()
    elif epilogue == "swiglu":
        ref = torch.nn.functional.silu(ref[:, :n]) * ref[:, n:]
    torch.cuda.synchronize()
    if epilogue == "swiglu":
        B.fp_op_gemm_swiglu(a.data_ptr(), w.data_ptr(), c.data_ptr(), m, n, k)
    else:
        B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), c.data_ptr(), m, n, k, epilogue == "residual")
    torch.cuda.synchronize()
    # bf16 results: 2^-9 relative each; SiLU(gate) * up of gate and up rounded to bf16: three such roundings, the gate's
    # amplified by at most 1 + |g|/4 or so.  fp32 results: sums of up to 2560 products in fp32, 32 at a time in the matrix unit: 1e-6 at most.
    bound = {"bf16": 4e-3, "swiglu": 1e-2, "residual": 1e-5}[epilogue]
    err = (c[:m].double() - ref).norm(dim=1) / ref.norm(dim=1)
    assert err.max().item() <= bound, (err.argmax().item(), err.max().item())
    assert torch.all(c[m:] == 7.0)


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m,n,k", [(m, 2056, 1088) for m in (65, 96, 97, 128, 129, 160, 161, 192, 193, 224, 225, 257, 321, 385, 450, 511)] +
                                  [(m, 2056, 6208) for m in (513, 576, 577, 672, 673, 771, 1023)] +
                                  [(m, 21000, 192) for m in (65, 95, 127, 159, 191, 223, 255)] + [(128, 1032, 17408)])
def test_few_row_tiles_of_every_height(m, n, k, residual):
    """Problems of one to four row tiles, cut over K on both widths of the large tile and (21000 columns) uncut on the narrow
    one: row tiles of 96 to 256 rows, as few as hold m (and 128 rows of a long K on the few-rows kernel); rows behind M and the workspace's guard stay."""
    B = _binding()
    print(f"few row tiles m={m} n={n} k={k} residual={residual}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 94, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.05, 95, torch.bfloat16, "cuda")
    c = torch.full((m + 256, n), 7.0, dtype=torch.float32 if residual else torch.bfloat16, device="cuda")
    ref = a.double() @ w.double().T
    if residual:
        c[:m] = I.normal_tensor((m, n), 1.0, 96, torch.float32, "cuda")
        ref += c[:m].double()
    ws_bytes = B.fp_op_gemm_workspace_bytes(1, m, n, k)
    assert (ws_bytes > 0) == (k != 192)
    ws = torch.full((ws_bytes + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_gemm_ws(1, a.data_ptr(), w.data_ptr(), c.data_ptr(), m, n, k, residual, ws.data_ptr(), ws_bytes)
    torch.cuda.synchronize()
    err = (c[:m].double() - ref).norm(dim=1) / ref.norm(dim=1)
    # bf16 results: 2^-9 relative each; fp32: sums of up to 17408 products in fp32, 32 at a time in the matrix unit: 1e-5 at most.
    assert err.max().item() <= (1e-5 if residual else 4e-3), (err.argmax().item(), err.max().item())
    assert torch.all(c[m:] == 7.0) and torch.all(ws[ws_bytes:] == 0x5A)


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("m,n,k", [(65, 40968, 1152), (128, 40968, 1216), (65, 65800, 64), (97, 65800, 192), (128, 65536, 128)])
def test_wide_projections_of_65_to_128_rows(m, n, k, residual):
    """Columns that fill the chip with wide tiles: the large kernel (one round of tiles, K up to 1152), else the few-rows kernel; the
    bits of 200 rows, which run on the former, and every row behind M stays."""
    B = _binding()
    print(f"wide projection m={m} n={n} k={k} residual={residual}", flush=True)
    a = I.normal_tensor((200, k), 1.0, 101, torch.bfloat16, "cuda")
    w = I.normal_tensor((n, k), 0.05, 102, torch.bfloat16, "cuda")
    td = torch.float32 if residual else torch.bfloat16
    c = torch.full((200, n), 7.0, dtype=td, device="cuda")
    if residual:
        c[:m] = I.normal_tensor((m, n), 1.0, 103, td, "cuda")
    all_rows = c.clone()
    ref = a[:m].double() @ w.double().T
    if residual:
        ref += c[:m].double()
    assert B.fp_op_gemm_workspace_bytes(1, m, n, k) == 0
    torch.cuda.synchronize()
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), c.data_ptr(), m, n, k, residual)
    B.fp_op_gemm(1, a.data_ptr(), w.data_ptr(), all_rows.data_ptr(), 200, n, k, residual)
    torch.cuda.synchronize()
    err = (c[:m].double() - ref).norm(dim=1) / ref.norm(dim=1)
    # bf16 results: 2^-9 relative each; fp32: sums of up to 1216 products in fp32, 32 at a time in the matrix unit: 1e-5 at most.
    assert err.max().item() <= (1e-5 if residual else 4e-3), (err.argmax().item(), err.max().item())
    assert torch.equal(c[:m], all_rows[:m]) and torch.all(c[m:] == 7.0)


F32_TILE_SIZES = [            # rows of the tile, m (one row past the last whole tile, or one short of one), n, k, residual
    (16, 431, 24, 520, 0), (16, 417, 8, 520, 0), (16, 31, 72, 520, 1), (16, 1, 104, 304, 1), (32, 63, 416, 40, 0), (32, 1, 2784, 40, 0),
    (32, 31, 576, 8, 1), (48, 95, 5496, 40, 0), (48, 385, 1384, 40, 0), (48, 335, 1528, 8, 1), (48, 97, 4616, 8, 1),
    (64, 255, 16, 8, 0), (64, 255, 2720, 8, 1), (64, 193, 3768, 8, 1), (80, 159, 5840, 8, 0), (80, 321, 2808, 8, 0),
    (80, 300, 4096, 4096, 1), (80, 321, 2824, 8, 1), (128, 1151, 3360, 136, 0), (128, 639, 5712, 8, 1), (128, 897, 3912, 8, 1)]


@pytest.mark.parametrize("rows,m,n,k,residual", F32_TILE_SIZES)
def test_fp32_gemm_on_tiles_of_every_height(rows, m, n, k, residual):
    """The fp32 MFMA kernel on 16 to 128 rows (tests/test_gemm_plan.py checks which), among them heights that are no
    multiple of the 32 rows a round of DMA fills; rows before and behind the output stay."""
    B = _binding()
    print(f"fp32 tile rows={rows} m={m} n={n} k={k} residual={residual}", flush=True)
    a = I.normal_tensor((m, k), 1.0, 97, torch.float32, "cuda")
    w = I.normal_tensor((n, k), 0.05, 98, torch.float32, "cuda")
    c = torch.full((m + 256, n), 7.0, device="cuda")
    ref = a.double() @ w.double().T
    if residual:
        c[128:m + 128] = I.normal_tensor((m, n), 1.0, 99, torch.float32, "cuda")
        ref += c[128:m + 128].double()
    torch.cuda.synchronize()
    B.fp_op_gemm(0, a.data_ptr(), w.data_ptr(), c[128:].data_ptr(), m, n, k, bool(residual))
    torch.cuda.synchronize()
    err = (c[128:m + 128].double() - ref).norm(dim=1) / ref.norm(dim=1)
    # Sums of k products, four at a time: a random walk of k / 4 roundings of 2^-24, 2e-6 at k = 4096 (a row of few columns: twice that).
    assert err.max().item() <= 4e-6, (err.argmax().item(), err.max().item())
    assert torch.all(c[:128] == 7.0) and torch.all(c[m + 128:] == 7.0)
