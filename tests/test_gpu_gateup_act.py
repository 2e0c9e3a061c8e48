"""GPU parity of the gate-up projection with the gated activation (ppas_gateup_act)
against the fp64 oracle (oracle.gemm.gate_up_act), through the C ABI.

Bound per output element, derived from the kernel's arithmetic. The gate and up
sums g~ and u~ carry the projection's accumulation error, at most
d_g = (1 + 2^-8) 2 H 2^-24 A_g (A_g = sum_k |x_k w_k| over the gate row; d_u the
same over the up row), and are not rounded before the activation. silu has slope
at most 1.1 in magnitude, so
    |silu(g~) u~ - silu(g) u| <= 1.1 d_g (|u| + d_u) + |silu(g)| d_u = D.
The fp32 evaluation of silu(g~) u~ (the exponential of a rounded argument, one
division, one product) adds at most 2^-24 (|g| + 4) |silu(g) u|, and the final
rounding to bf16 nearest at most 2^-8 of the stored value, so
    |gpu - z| <= (2^-8 |z| + D + 2^-24 (|g| + 4) |z|) / (1 - 2^-8).
Ragged shapes (token rows not multiples of 256, features not multiples of the
128 a tile covers, split and unsplit reductions) are compared on every element;
the Qwen2.5-3B sizes (hidden 2048, 11008 features) on every element as well.
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
    ppas, step, torch = lib
    x = step.to_device_bf16(xb)
    w = step.to_device_bf16(wb)
    n_inter = wb.shape[0] // 2
    y = torch.full((xb.shape[0], n_inter), float("nan"), dtype=torch.bfloat16, device="cuda")
    n = ppas.gateup_act_workspace_bytes(xb.shape[0], xb.shape[1], n_inter) if split else 0
    ws = torch.full((max(n // 4, 1),), float("nan"), dtype=torch.float32, device="cuda") if n else None
    ppas.gateup_act(x, w, y, ws)
    torch.cuda.synchronize()
    return y


def f64(y):
    return y.float().cpu().numpy().astype(np.float64)


def check(g, xb, wb, rows=None, label=""):
    z, gate, up, ag, au = OG.gate_up_act(xb, wb, rows=rows, with_terms=True)
    assert np.isfinite(g).all(), f"{label}: non-finite output"
    H = xb.shape[1]
    dg = (1 + 2.0 ** -8) * 2 * H * 2.0 ** -24 * ag
    du = (1 + 2.0 ** -8) * 2 * H * 2.0 ** -24 * au
    D = 1.1 * dg * (np.abs(up) + du) + np.abs(OG.silu(gate)) * du
    bound = (2.0 ** -8 * np.abs(z) + D + 2.0 ** -24 * (np.abs(gate) + 4) * np.abs(z)) / (1 - 2.0 ** -8) + 1e-30
    err = np.abs(g - z)
    worst = float((err / bound).max())
    print(f"{label}: max_abs={err.max():.3e} err/bound={worst:.3f}", flush=True)
    assert worst <= 1.0, f"{label}: {int((err > bound).sum())} elements beyond the bound"


@pytest.mark.parametrize("T,H,NI", [(1, 64, 1), (5, 64, 150), (31, 128, 17), (257, 128, 256), (300, 192, 260),
                                    (256, 256, 128), (513, 2048, 300), (700, 640, 515),
                                    # split reductions: decode-sized and small-chunk calls
                                    (16, 2048, 11008), (3, 2048, 1025), (100, 2048, 1280), (2048, 2048, 1024),
                                    # just over one round of workgroups' tiles, tail tiles among them
                                    (1125, 128, 7650)])
@pytest.mark.parametrize("split", [True, False])
def test_ragged_shapes_every_element(lib, T, H, NI, split):
    ppas = lib[0]
    print(f"gate-up-act T={T} H={H} I={NI} split={split} workspace={ppas.gateup_act_workspace_bytes(T, H, NI)}",
          flush=True)
    xb = I.gateup_tokens(3, T, 0, hidden=H)
    wb = I.gateup_weight(3, hidden=H, inter=NI)
    check(f64(run(lib, xb, wb, split)), xb, wb, label=f"T{T} H{H} I{NI} split={split}")


def test_split_reduction_is_deterministic(lib):
    torch = lib[2]
    xb = I.gateup_tokens(4, 40, 0, hidden=2048)
    wb = I.gateup_weight(4, hidden=2048, inter=2048)
    a, b = run(lib, xb, wb), run(lib, xb, wb)
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("T", [2048, 16384])
def test_qwen25_3b_sizes_every_row(lib, T):
    """Every element at the full sizes, checked in blocks of 2,048 token rows."""
    print(f"gate-up-act T={T} H={I.GATEUP_HIDDEN} I={I.GATEUP_INTER}", flush=True)
    xb = I.gateup_tokens(0, T)
    wb = I.gateup_weight(0)
    y = run(lib, xb, wb)
    for r0 in range(0, T, 2048):
        rows = np.arange(r0, min(T, r0 + 2048))
        check(f64(y[r0:rows[-1] + 1]), xb, wb, rows=rows, label=f"T{T} rows {r0}..{rows[-1]}")


def test_chunks_equal_whole_prompt_rows(lib):
    """Eight 2,048-token chunks give the same bits as the rows of the 16,384-token
    prompt at once (the same k-steps for every element, wherever its row sits)."""
    torch = lib[2]
    wb = I.gateup_weight(0)
    whole = run(lib, I.gateup_tokens(0, 16384), wb)
    for c in range(8):
        part = run(lib, I.gateup_tokens(0, 2048, 2048 * c), wb)
        assert torch.equal(part.view(torch.int16), whole[2048 * c:2048 * (c + 1)].view(torch.int16)), c


def test_shapes_and_sizes_are_refused(lib):
    ppas, step, torch = lib
    x = torch.zeros((4, 64), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((9, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ValueError):                          # odd weight rows
        ppas.gateup_act(x, w, torch.zeros((4, 4), dtype=torch.bfloat16, device="cuda"))
    w = torch.zeros((8, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ValueError):                          # y must be [T, I]
        ppas.gateup_act(x, w, torch.zeros((4, 8), dtype=torch.bfloat16, device="cuda"))
    ppas.gateup_act(x[:0], w, torch.zeros((0, 4), dtype=torch.bfloat16, device="cuda"))   # no tokens
    x = torch.zeros((4, 96), dtype=torch.bfloat16, device="cuda")
    w = torch.zeros((8, 96), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(ppas.PPASError) as ex:
        ppas.gateup_act(x, w, torch.zeros((4, 4), dtype=torch.bfloat16, device="cuda"))
    assert ex.value.status == ppas.PPAS_EUNSUPPORTED


@pytest.mark.parametrize("T,H,NI", [(65, 64, 150), (130, 2048, 11005), (513, 192, 11000), (321, 2048, 11008),
                                    (577, 1024, 8000), (700, 2048, 1030)])
def test_tile_shapes_every_element(lib, T, H, NI):
    """Ragged rows, features and stage counts of the tile kernels."""
    print(f"gate-up-act tiles T={T} H={H} I={NI}", flush=True)
    xb = I.gateup_tokens(8, T, 0, hidden=H)
    wb = I.gateup_weight(8, hidden=H, inter=NI)
    check(f64(run(lib, xb, wb)), xb, wb, label=f"act T{T} H{H} I{NI}")


@pytest.mark.parametrize("T,H,NI", [(1, 2048, 11008), (16, 64, 500), (17, 1024, 3001), (24, 2048, 5504),
                                    (64, 576, 1500), (65, 128, 700), (200, 2048, 640)])
def test_few_rows_every_element(lib, T, H, NI):
    """Few rows: tiles of 16, 32 and 64 rows and their edges."""
    print(f"gate-up-act rows T={T} H={H} I={NI}", flush=True)
    xb = I.gateup_tokens(11, T, 0, hidden=H)
    wb = I.gateup_weight(11, hidden=H, inter=NI)
    check(f64(run(lib, xb, wb)), xb, wb, label=f"act T{T} H{H} I{NI}")


# Every kernel variant, with the choice that names it: few rows by token rows per workgroup, weight-row tiles and
# their rows; tiles by the rows of a main tile (64: small tiles only), whether the reduction is split and whether
# small tiles follow.
VARIANTS = [
    ("rows", 16, 2, 8, 9, 11008, 1514), ("rows", 16, 2, 16, 13, 3008, 3836), ("rows", 16, 4, 16, 8, 3008, 6233),
    ("rows", 16, 6, 16, 8, 2112, 8874), ("rows", 32, 2, 8, 30, 3584, 1395), ("rows", 32, 2, 16, 21, 3008, 2375),
    ("rows", 32, 4, 16, 25, 1024, 5864), ("rows", 32, 6, 16, 24, 2048, 11008), ("rows", 64, 2, 8, 208, 5504, 131),
    ("rows", 64, 2, 16, 88, 1024, 1665), ("rows", 64, 4, 16, 139, 576, 1873), ("rows", 64, 6, 16, 70, 576, 4183),
    ("rows", 64, 6, 16, 48, 2048, 11008),
    ("tiles", 64, False, True, 228, 320, 2056), ("tiles", 64, True, True, 775, 3584, 54),
    ("tiles", 128, False, False, 256, 128, 8197), ("tiles", 128, False, True, 129, 128, 10982),
    ("tiles", 128, True, False, 1024, 11008, 133), ("tiles", 128, True, True, 1136, 11008, 12),
    ("tiles", 256, False, False, 768, 320, 5600), ("tiles", 256, False, True, 611, 320, 10889),
    ("tiles", 256, True, False, 1280, 5504, 1549), ("tiles", 256, True, True, 2076, 11008, 387)]


@pytest.mark.parametrize("kind,rows,p,q,T,H,NI", VARIANTS)
def test_every_variant_every_element(lib, kind, rows, p, q, T, H, NI):
    c = lib[0].gateup_choice(T, H, 2 * NI, activation=True, num_cus=256)
    got = (c["rows"], c["weight_tiles"], c["weight_rows"]) if c["kernel"] == "rows" else \
        (c["rows"] if c["main_tiles"] else 64, c["splits"] > 1, c["small_tiles"] > 0)
    assert (c["kernel"], *got) == (kind, rows, p, q)
    print(f"gate-up-act {kind} {rows} {p} {q} T={T} H={H} I={NI}", flush=True)
    xb = I.gateup_tokens(14, T, 0, hidden=H)
    wb = I.gateup_weight(14, hidden=H, inter=NI)
    check(f64(run(lib, xb, wb)), xb, wb, label=f"act {kind} {rows} {p} {q}")


@pytest.mark.parametrize("T,H,NI,split", [(1, 64, 1, False), (257, 128, 257, True), (40, 2048, 260, True),
                                          (40, 2048, 260, False), (300, 11008, 515, True), (700, 640, 513, True)])
@pytest.mark.parametrize("which", ["x", "w", "xw"])
def test_general_kernel_every_element(lib, which, T, H, NI, split):
    """Operands off the 16-byte grid, with and without the workspace: one chain per split."""
    ppas, step, torch = lib
    nbytes = ppas.gateup_act_workspace_bytes(T, H, NI) if split else 0
    c = ppas.gateup_choice(T, H, 2 * NI, activation=True, aligned=False, workspace_bytes=nbytes)
    assert c["kernel"] == "general" and (c["splits"] > 1) == (split and H > 256), c
    print(f"gate-up-act general {which} T={T} H={H} I={NI} splits={c['splits']}", flush=True)
    xb = I.gateup_tokens(15, T, 0, hidden=H)
    wb = I.gateup_weight(15, hidden=H, inter=NI)

    def put(bits, off):
        flat = torch.zeros(bits.size + 4, dtype=torch.bfloat16, device="cuda")
        v = flat[4:] if off else flat[:-4]
        v.copy_(step.to_device_bf16(bits).flatten())
        return v.view(*bits.shape)

    x, w = put(xb, "x" in which), put(wb, "w" in which)
    assert (x.data_ptr() | w.data_ptr()) % 16 == 8
    y = torch.full((T, NI), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda") if nbytes else None
    ppas.gateup_act(x, w, y, ws)
    torch.cuda.synchronize()
    check(f64(y), xb, wb, label=f"act general {which} T{T} H{H} I{NI} split={split}")
