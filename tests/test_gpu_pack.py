"""Weight packing against the packed order written out as a torch permutation:
[k-tile][column group][k step][column half][k half][row][8], zero padded to
64 x 64. Sizes around one 64 x 64 tile, odd row lengths and sources that are
not 16-byte aligned (gathered by elements), and nothing written past the end."""

import pytest
import torch

pytestmark = pytest.mark.gpu


def _packed(w):
    n, k = w.shape
    N, K = -(-n // 64) * 64, -(-k // 64) * 64
    p = torch.zeros(N, K, dtype=torch.int16)
    p[:n, :k] = w.view(torch.int16)
    return p.reshape(N // 64, 2, 32, K // 64, 4, 2, 8).permute(3, 0, 4, 1, 5, 2, 6).contiguous().reshape(-1)


def _weights(n, k, offset, seed):
    g = torch.Generator().manual_seed(seed)
    buf = torch.randn(n * k + 8, generator=g).to(torch.bfloat16)
    return buf[offset:offset + n * k].view(n, k), buf.cuda()[offset:offset + n * k].view(n, k)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n,k", [(1, 1), (64, 64), (63, 40), (65, 257), (200, 1000), (1000, 2052)])
def test_pack_linear_order(lib, n, k, offset):
    host, dev = _weights(n, k, offset, n + k)
    out = torch.full((lib.sidp_packed_bytes(n, k) + 256,), 7, dtype=torch.uint8, device="cuda")
    lib.sidp_pack_linear(dev, n, k, out)
    torch.cuda.synchronize()
    assert torch.equal(out[:-256].view(torch.int16).cpu(), _packed(host))
    assert bool((out[-256:] == 7).all())


@pytest.mark.parametrize("f,k,offset", [(16, 64, 0), (48, 100, 0), (33, 8, 1), (688, 256, 0)])
def test_pack_gate_up_order(lib, f, k, offset):
    gh, gd = _weights(f, k, offset, f)
    uh, ud = _weights(f, k, offset, f + 1)
    f32 = -(-f // 32) * 32
    rows = torch.zeros(2, f32, k, dtype=torch.bfloat16)
    rows[0, :f], rows[1, :f] = gh, uh
    rows = rows.reshape(2, f32 // 32, 32, k).transpose(0, 1).reshape(2 * f32, k)
    out = torch.full((lib.sidp_packed_bytes(2 * f32, k) + 256,), 7, dtype=torch.uint8, device="cuda")
    lib.sidp_pack_gate_up(gd, ud, f, k, out)
    torch.cuda.synchronize()
    assert torch.equal(out[:-256].view(torch.int16).cpu(), _packed(rows))
    assert bool((out[-256:] == 7).all())
