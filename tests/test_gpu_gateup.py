"""GPU parity of the fused gate-up projection (ppas_gateup_proj) against the fp64
oracle (oracle/gemm.py), through the C ABI.

Bound per output element, derived from the kernel's arithmetic: the products of
two bf16 values are exact in fp32, the fp32 accumulation over H features moves
the sum s by at most H 2^-24 A (A = sum_k |x_k w_k|, from the oracle; doubled to
cover any internal order of the matrix cores), and rounding s to bf16 nearest
moves it by at most 2^-8 |s|:
    |gpu - y| <= 2^-8 |y| + (1 + 2^-8) 2 H 2^-24 A.
Ragged shapes (token rows and output columns not multiples of the 256 x 256 tile)
are compared on every element; the full Qwen2.5-3B sizes (hidden 2048, 22016
stacked gate/up rows) at 2,048 and 16,384 tokens on every element as well.
"""
import numpy as np
import pytest

import oracle.gemm as OG
from paper_2608_15171_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2608_15171_amd import ppas, step
    return ppas, step, torch


def run(lib, xb, wb, split=True):
    """split: give the call the workspace it asks for (reductions split across workgroups
    when the output has fewer tiles than compute units); False: no workspace, no split."""
    ppas, step, torch = lib
    x = step.to_device_bf16(xb)
    w = step.to_device_bf16(wb)
    y = torch.full((xb.shape[0], wb.shape[0]), float("nan"), dtype=torch.bfloat16, device="cuda")
    n = ppas.gateup_workspace_bytes(xb.shape[0], xb.shape[1], wb.shape[0]) if split else 0
    ws = torch.full((max(n // 4, 1),), float("nan"), dtype=torch.float32, device="cuda") if n else None
    ppas.gateup_proj(x, w, y, ws)
    torch.cuda.synchronize()
    return y


def check(g, xb, wb, rows=None, label=""):
    """g: the GPU output of all rows, or of `rows` in that order."""
    y, a = OG.gate_up(xb, wb, rows=rows, with_abs=True)
    assert np.isfinite(g).all(), f"{label}: non-finite output"
    H = xb.shape[1]
    bound = 2.0 ** -8 * np.abs(y) + (1 + 2.0 ** -8) * 2 * H * 2.0 ** -24 * a + 1e-30
    err = np.abs(g - y)
    worst = float((err / bound).max())
    print(f"{label}: max_abs={err.max():.3e} err/bound={worst:.3f}", flush=True)
    assert worst <= 1.0, f"{label}: {int((err > bound).sum())} elements beyond the bound"


def f64(lib, y):
    return y.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("T,H,N", [(1, 64, 1), (5, 64, 300), (31, 128, 33), (257, 128, 513), (300, 192, 520),
                                   (256, 256, 256), (513, 2048, 600), (700, 640, 1030),
                                   # split reductions: the decoder layer's other projections at decode and
                                   # chunk sizes (down 11008 -> 2048, QKV 2048 -> 2560, output 2048 -> 2048)
                                   (16, 11008, 2048), (3, 11008, 2050), (100, 2048, 2560), (2048, 11008, 2048),
                                   (600, 2048, 2048),
                                   # just over one round of workgroups' tiles, 64-row tail tiles among them
                                   (1125, 128, 15300)])
@pytest.mark.parametrize("split", [True, False])
def test_ragged_shapes_every_element(lib, T, H, N, split):
    ppas = lib[0]
    print(f"gate-up T={T} H={H} N={N} split={split} workspace={ppas.gateup_workspace_bytes(T, H, N)}", flush=True)
    xb = I.gateup_tokens(1, T, 0, hidden=H)
    wb = I.gateup_weight(1, hidden=H, inter=(N + 1) // 2)[:N]
    check(f64(lib, run(lib, xb, wb, split)), xb, wb, label=f"T{T} H{H} N{N} split={split}")


def test_split_reduction_is_deterministic(lib):
    ppas, step, torch = lib
    xb = I.gateup_tokens(2, 40, 0, hidden=11008)
    wb = I.gateup_weight(2, hidden=11008, inter=1024)
    a, b = run(lib, xb, wb), run(lib, xb, wb)
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("T", [2048, 16384])
def test_qwen25_3b_sizes_every_row(lib, T):
    """Every element at the full sizes, checked in blocks of 2,048 token rows."""
    print(f"gate-up T={T} H={I.GATEUP_HIDDEN} N={2 * I.GATEUP_INTER}", flush=True)
    xb = I.gateup_tokens(0, T)
    wb = I.gateup_weight(0)
    y = run(lib, xb, wb)
    for r0 in range(0, T, 2048):
        rows = np.arange(r0, min(T, r0 + 2048))
        check(f64(lib, y[r0:rows[-1] + 1]), xb, wb, rows=rows, label=f"T{T} rows {r0}..{rows[-1]}")


def test_chunks_equal_whole_prompt_rows(lib):
    """Eight 2,048-token chunks projected one by one give the same bits as the rows of
    the 16,384-token prompt projected at once: each output element is the same
    sequence of MFMA k-steps wherever its row sits in a tile."""
    ppas, step, torch = lib
    wb = I.gateup_weight(0)
    whole = run(lib, I.gateup_tokens(0, 16384), wb)
    for c in range(8):
        part = run(lib, I.gateup_tokens(0, 2048, 2048 * c), wb)
        assert torch.equal(part.view(torch.int16), whole[2048 * c:2048 * (c + 1)].view(torch.int16)), c


def test_zero_tokens_is_a_no_op_and_bad_sizes_are_refused(lib):
    ppas, step, torch = lib
    x = torch.zeros((0, 64), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((8, 64), dtype=torch.bfloat16, device="cuda")
    y = torch.zeros((0, 8), dtype=torch.bfloat16, device="cuda")
    ppas.gateup_proj(x, w, y)
    x = torch.zeros((4, 96), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((8, 96), dtype=torch.bfloat16, device="cuda")
    y = torch.zeros((4, 8), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ppas.PPASError) as ex:
        ppas.gateup_proj(x, w, y)
    assert ex.value.status == ppas.PPAS_EUNSUPPORTED


@pytest.mark.parametrize("T,H,N", [
    # one row over a tile; single-stage tiles, several per workgroup
    (65, 64, 300), (449, 64, 22016), (1790, 64, 9000),
    # a few rows after whole tiles; three stages; splits
    (130, 2048, 22010), (513, 192, 22000), (700, 11008, 2048),
    # 64-row tiles dealt to the workgroups with fewer large ones; a narrow output
    (321, 2048, 22016), (577, 1024, 16000), (2048, 11008, 300)])
def test_tile_shapes_every_element(lib, T, H, N):
    """Ragged rows, columns and stage counts of the tile kernels."""
    print(f"gate-up tiles T={T} H={H} N={N}", flush=True)
    xb = I.gateup_tokens(6, T, 0, hidden=H)
    wb = I.gateup_weight(6, hidden=H, inter=(N + 1) // 2)[:N]
    check(f64(lib, run(lib, xb, wb)), xb, wb, label=f"T{T} H{H} N{N}")


@pytest.mark.parametrize("which", ["x", "w"])
def test_operands_off_the_16_byte_grid(lib, which):
    """Operands that start 8 bytes off a 16-byte boundary take the general kernel."""
    ppas, step, torch = lib
    T, H, N = 300, 256, 520
    xb = I.gateup_tokens(7, T, 0, hidden=H)
    wb = I.gateup_weight(7, hidden=H, inter=N // 2)

    def off(bits):
        flat = torch.zeros(bits.size + 4, dtype=torch.bfloat16, device="cuda")
        flat[4:] = step.to_device_bf16(bits).flatten()
        return flat[4:].view(*bits.shape)

    x = off(xb) if which == "x" else step.to_device_bf16(xb)
    w = off(wb) if which == "w" else step.to_device_bf16(wb)
    assert (x.data_ptr() | w.data_ptr()) % 16 == 8
    y = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ppas.gateup_proj(x, w, y)
    check(f64(lib, y), xb, wb, label=f"{which} off by 8 bytes")


@pytest.mark.parametrize("T,H,N", [
    # few rows: 16-, 32- and 64-row tiles and their edges, several of them; a last block of one chunk; fewer
    # chunks than waves; more blocks than are kept in order
    (1, 2048, 22016), (16, 2048, 2050), (17, 64, 300), (24, 11008, 2048), (33, 576, 256), (48, 2048, 11010),
    (64, 128, 40), (65, 2048, 2048), (100, 2112, 130), (256, 2048, 250), (20, 192, 9001)])
def test_few_rows_every_element(lib, T, H, N):
    print(f"gate-up rows T={T} H={H} N={N}", flush=True)
    xb = I.gateup_tokens(9, T, 0, hidden=H)
    wb = I.gateup_weight(9, hidden=H, inter=(N + 1) // 2)[:N]
    check(f64(lib, run(lib, xb, wb)), xb, wb, label=f"T{T} H{H} N{N}")


# Every kernel variant, with the choice that names it: few rows by token rows per workgroup, weight-row tiles and
# their rows; tiles by the rows of a main tile (64: small tiles only), whether the reduction is split and whether
# small tiles follow. Columns, rows and stages are ragged where the variant allows it.
VARIANTS = [
    ("rows", 16, 1, 8, 16, 11008, 1697), ("rows", 16, 1, 16, 10, 11008, 2730), ("rows", 16, 2, 16, 10, 5504, 5445),
    ("rows", 16, 4, 16, 14, 2048, 10463), ("rows", 16, 6, 16, 16, 2048, 22016), ("rows", 32, 1, 8, 18, 11008, 1516),
    ("rows", 32, 1, 16, 30, 3584, 2790), ("rows", 32, 2, 16, 18, 3008, 5541), ("rows", 32, 4, 16, 29, 1024, 10102),
    ("rows", 32, 6, 16, 24, 2048, 22016), ("rows", 64, 1, 8, 250, 3008, 399), ("rows", 64, 1, 16, 168, 1600, 1116),
    ("rows", 64, 2, 16, 172, 1024, 1703), ("rows", 64, 4, 16, 187, 576, 2784), ("rows", 64, 6, 16, 67, 576, 8270),
    ("rows", 64, 6, 16, 48, 2048, 22016),
    ("tiles", 64, False, True, 193, 192, 8096), ("tiles", 64, True, True, 545, 3008, 183),
    ("tiles", 128, False, False, 256, 128, 16872), ("tiles", 128, False, True, 131, 128, 21995),
    ("tiles", 128, True, False, 1408, 2048, 360), ("tiles", 128, True, True, 1190, 11008, 23),
    ("tiles", 256, False, False, 768, 320, 10756), ("tiles", 256, False, True, 583, 320, 21776),
    ("tiles", 256, True, False, 1792, 11008, 1064), ("tiles", 256, True, True, 513, 11008, 3102)]


def variant_of(c):
    if c["kernel"] == "rows":
        return "rows", c["rows"], c["weight_tiles"], c["weight_rows"]
    return c["kernel"], c["rows"] if c["main_tiles"] else 64, c["splits"] > 1, c["small_tiles"] > 0


@pytest.mark.parametrize("kind,rows,p,q,T,H,N", VARIANTS)
def test_every_variant_every_element(lib, kind, rows, p, q, T, H, N):
    ppas = lib[0]
    assert variant_of(ppas.gateup_choice(T, H, N, num_cus=256)) == (kind, rows, p, q)
    print(f"gate-up {kind} {rows} {p} {q} T={T} H={H} N={N}", flush=True)
    xb = I.gateup_tokens(12, T, 0, hidden=H)
    wb = I.gateup_weight(12, hidden=H, inter=(N + 1) // 2)[:N]
    check(f64(lib, run(lib, xb, wb)), xb, wb, label=f"{kind} {rows} {p} {q}")


@pytest.mark.parametrize("T,H,N,split", [(1, 64, 1, False), (257, 128, 513, True), (40, 2048, 520, True),
                                         (40, 2048, 520, False), (300, 11008, 1030, True), (700, 640, 1031, True)])
@pytest.mark.parametrize("which", ["x", "w", "xw"])
def test_general_kernel_every_element(lib, which, T, H, N, split):
    """Operands off the 16-byte grid, with and without the workspace: one chain per split."""
    ppas, step, torch = lib
    nbytes = ppas.gateup_workspace_bytes(T, H, N) if split else 0
    c = ppas.gateup_choice(T, H, N, aligned=False, workspace_bytes=nbytes)
    assert c["kernel"] == "general" and (c["splits"] > 1) == (split and H > 256 and T * N > 1), c
    print(f"gate-up general {which} T={T} H={H} N={N} splits={c['splits']}", flush=True)
    xb = I.gateup_tokens(13, T, 0, hidden=H)
    wb = I.gateup_weight(13, hidden=H, inter=(N + 1) // 2)[:N]

    def put(bits, off):
        flat = torch.zeros(bits.size + 4, dtype=torch.bfloat16, device="cuda")
        v = flat[4:] if off else flat[:-4]
        v.copy_(step.to_device_bf16(bits).flatten())
        return v.view(*bits.shape)

    x, w = put(xb, "x" in which), put(wb, "w" in which)
    assert (x.data_ptr() | w.data_ptr()) % 16 == 8
    y = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda") if nbytes else None
    ppas.gateup_proj(x, w, y, ws)
    torch.cuda.synchronize()
    check(f64(lib, y), xb, wb, label=f"general {which} T{T} H{H} N{N} split={split}")


@pytest.mark.parametrize("H,N", [(2048, 256), (2048, 512), (1024, 500), (256, 128)])
def test_narrow_output_does_not_depend_on_the_rows_beside_it(lib, H, N):
    """The K and V projections (up to 512 columns over one to eight 256-feature blocks) add the
    same block sums in the same order in every kernel: a row's bits are the same in calls of
    any size."""
    ppas, step, torch = lib
    wb = I.gateup_weight(10, hidden=H, inter=N // 2)
    xb = I.gateup_tokens(10, 2500, 0, hidden=H)
    whole = run(lib, xb, wb)
    for n in (1, 16, 40, 200, 256, 300, 700, 1100):
        part = run(lib, xb[:n], wb)
        assert torch.equal(part.view(torch.int16), whole[:n].view(torch.int16)), n
