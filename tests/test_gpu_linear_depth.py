"""The projection kernel's k loop at the sizes where its pipeline can go wrong:
fewer k-tiles than the loop keeps in flight, every remainder of its four-tile
body, ragged last k-tiles, each row-block height and workgroup width, idle
column groups. Compared with float64 on every element: a sum of k products of
bf16 numbers accumulated in fp32 is within 2^-20 of sum |x w| of the exact one,
plus half a bf16 spacing (2^-9 of the value) where the output is bf16."""

import re

import pytest
import torch

from gpu_helpers import kernels_of

pytestmark = pytest.mark.gpu


def _run(lib, m, n, k, epi, x):
    g = torch.Generator(device="cuda").manual_seed(m * 31 + n + k * 7 + epi)
    w = [(0.02 * torch.randn(n, k, device="cuda", generator=g)).bfloat16() for _ in range(2 if epi == 2 else 1)]
    cols = 2 * (-(-n // 32) * 32) if epi == 2 else n
    packed = torch.empty(lib.sidp_packed_bytes(cols, k), dtype=torch.uint8, device="cuda")
    if epi == 2:
        lib.sidp_pack_gate_up(w[0], w[1], n, k, packed)
    else:
        lib.sidp_pack_linear(w[0], n, k, packed)
    out = torch.full((m, n), float("nan"), device="cuda", dtype=torch.float32 if epi == 1 else torch.bfloat16)
    resid = torch.randn(m, n, device="cuda", generator=g) if epi == 1 else None
    lib.sidp_linear_noalloc(x, m, k, packed, n, epi, None, resid, out)
    torch.cuda.synchronize()
    return out.double(), [v.double() for v in w], resid


def _check(lib, m, n, k, epi, x):
    got, w, resid = _run(lib, m, n, k, epi, x)
    xd = x.double()
    if epi == 2:
        gate, up = xd @ w[0].t(), xd @ w[1].t()
        want = torch.nn.functional.silu(gate) * up
        # |silu'| <= 1.1: the gate's error passes through scaled by |up|
        tol = 2.0 ** -20 * (1.1 * (xd.abs() @ w[0].abs().t()) * up.abs()
                            + torch.nn.functional.silu(gate).abs() * (xd.abs() @ w[1].abs().t()))
    else:
        want, tol = xd @ w[0].t(), 2.0 ** -20 * (xd.abs() @ w[0].abs().t())
        if resid is not None:
            want, tol = want + resid.double(), tol + 2.0 ** -23 * resid.double().abs()
    if epi != 1:
        tol = tol + 2.0 ** -8 * want.abs() + 2.0 ** -133
    bad = ~((got - want).abs() <= tol)
    assert not bool(bad.any()), (m, n, k, epi, int(bad.sum()))


def _x(m, k, seed=0):
    g = torch.Generator(device="cuda").manual_seed(m + k + seed)
    return (0.5 * torch.randn(m, k, device="cuda", generator=g)).bfloat16()


@pytest.mark.parametrize("m", [1, 32, 33, 64, 65, 128, 129, 300])
def test_every_depth_and_row_block(lib, m):
    for k in (8, 64, 72, 128, 192, 200, 256, 320, 328, 384, 448, 456, 520, 1000, 4104, 7264):
        _check(lib, m, 1000, k, 0, _x(m, k))
    _check(lib, m, 1000, 2056, 1, _x(m, 2056))
    _check(lib, m, 3032, 7264, 2, _x(m, 7264))


@pytest.mark.parametrize("m,n,k,epi", [(200, 28672, 520, 2), (129, 29568, 1032, 2), (260, 28672, 64, 2),
                                       (200, 45056, 264, 0), (512, 28672, 584, 1), (200, 8192, 25608, 1),
                                       # 158 MB of weights: ragged, whole and nearly empty second row blocks
                                       (161, 8192, 9672, 1), (256, 8192, 9672, 1), (129, 8192, 9672, 1), (160, 8192, 9672, 1)])
def test_wide_workgroups_and_large_weights(lib, m, n, k, epi):
    _check(lib, m, n, k, epi, _x(m, k))


@pytest.mark.parametrize("m", [20, 50, 97, 129, 200])
def test_rows_stay_apart_with_infinities_and_a_ragged_k(lib, m):
    """A row of infinities or NaN reaches its own outputs only, also where the
    pieces of a ragged k-tile run on into the next row."""
    x = _x(m, 456)
    ref, _, _ = _run(lib, m, 1000, 456, 0, x)
    y = x.clone()
    y[7] = float("nan")
    y[m - 1] = float("inf")
    got, _, _ = _run(lib, m, 1000, 456, 0, y)
    keep = [r for r in range(m) if r not in (7, m - 1)]
    assert torch.equal(got[keep], ref[keep])
    assert not bool(torch.isfinite(got[7]).any())


def test_activations_at_an_odd_eight_bytes(lib):
    """Activations that are not 16-byte aligned take the register-staged kernel: the same bits."""
    x = _x(100, 1032)
    ref, _, _ = _run(lib, 100, 1000, 1032, 0, x)
    buf = torch.empty(x.numel() + 4, dtype=torch.bfloat16, device="cuda")
    y = buf[4:].view(100, 1032)
    y.copy_(x)
    assert y.data_ptr() % 16 == 8
    got, _, _ = _run(lib, 100, 1000, 1032, 0, y)
    assert torch.equal(got, ref)


@pytest.mark.parametrize("n,epi", [(1001, 0), (999, 1), (3030, 2), (1002, 0), (4, 1), (1, 0)])
def test_split_reduction_of_odd_widths(lib, n, epi):
    """Split-K outputs whose width is no multiple of four columns are reduced one column a thread."""
    assert lib.sidp_linear_plan(17, n, 4104, epi)["splits"] > 1
    _check(lib, 17, n, 4104, epi, _x(17, 4104))


def _kernel(lib, m, n, k, epi):
    """The projection kernel that a call launches."""
    cols = 2 * (-(-n // 32) * 32) if epi == 2 else n
    packed = torch.zeros(lib.sidp_packed_bytes(cols, k), dtype=torch.uint8, device="cuda")
    x = torch.zeros(m, k, dtype=torch.bfloat16, device="cuda")
    out = torch.empty(m, n, dtype=torch.float32 if epi == 1 else torch.bfloat16, device="cuda")
    resid = torch.zeros(m, n, device="cuda") if epi == 1 else None
    ran = kernels_of(lambda: lib.sidp_linear_noalloc(x, m, k, packed, n, epi, None, resid, out))
    return re.search(r"k_gemm\w*", next(name for name in ran if "k_gemm" in name)).group(0)


@pytest.mark.parametrize("m,n,k,epi,kernel", [
    # a thin second row block: 24 rows, 14336 k and 150 MiB
    (152, 8192, 14336, 1, "k_gemm"), (153, 8192, 14336, 1, "k_gemm_deep"), (152, 8192, 14272, 1, "k_gemm_deep"),
    (152, 5120, 14336, 1, "k_gemm_deep"), (128, 8192, 14336, 1, "k_gemm_deep"),
    # few k-tiles on a full chip: 16 a split with two row blocks, 8 with four
    (200, 4096, 8192, 0, "k_gemm"), (200, 4096, 8256, 0, "k_gemm_deep"), (128, 4096, 4096, 0, "k_gemm_deep"),
    (512, 2048, 4096, 0, "k_gemm"), (512, 2048, 4160, 0, "k_gemm_deep"), (200, 12544, 1024, 0, "k_gemm_deep"),
    # one row block on every CU, 8 or 16 k-tiles a split
    (64, 8192, 8192, 0, "k_gemm"), (33, 8192, 4096, 0, "k_gemm"), (32, 8192, 8192, 0, "k_gemm_deep"),
    (64, 8192, 8256, 0, "k_gemm_deep"), (64, 8192, 12288, 0, "k_gemm_deep"), (64, 10240, 8192, 0, "k_gemm_deep"),
    # two 4-wave workgroups on some CUs: 288 of them, whole row blocks or 32 k-tiles
    (384, 24576, 2112, 0, "k_gemm"), (383, 24576, 2112, 0, "k_gemm_deep"), (383, 24576, 2048, 0, "k_gemm"),
    (384, 18304, 2112, 0, "k_gemm_deep"), (512, 28672, 1024, 2, "k_gemm_deep"),
])
def test_the_deep_pipeline_runs_where_it_is_the_faster_one(lib, m, n, k, epi, kernel):
    assert _kernel(lib, m, n, k, epi) == kernel


@pytest.mark.parametrize("m,n,k,epi", [(152, 8192, 14336, 1), (200, 4096, 2056, 0), (512, 2048, 1032, 1),
                                       (384, 24576, 328, 0), (300, 24576, 1032, 0), (257, 11008, 264, 2),
                                       (100, 8192, 4096, 1)])
def test_row_blocks_on_the_shallow_kernel(lib, m, n, k, epi):
    assert _kernel(lib, m, n, k, epi) == "k_gemm"
    _check(lib, m, n, k, epi, _x(m, k))


@pytest.mark.parametrize("m,n,k,columns", [(100, 4096, 2056, 4), (99, 4096, 2056, 1), (128, 2048, 1032, 1), (200, 2049, 1032, 1)])
def test_split_reduction_reads_four_columns_a_thread_of_large_outputs(lib, m, n, k, columns):
    """From 409600 outputs on, in rows of a multiple of four columns."""
    packed = torch.zeros(lib.sidp_packed_bytes(n, k), dtype=torch.uint8, device="cuda")
    x = torch.zeros(m, k, dtype=torch.bfloat16, device="cuda")
    out = torch.empty(m, n, dtype=torch.bfloat16, device="cuda")
    ran = kernels_of(lambda: lib.sidp_linear_noalloc(x, m, k, packed, n, 0, None, None, out))
    assert any(f"k_splitk_reduce<0, {columns}>" in name for name in ran), ran
    _check(lib, m, n, k, 0, _x(m, k))
