"""Branches of the small kernels: the RMSNorm whose row stays in registers at
both ends of its range, and the KV append on inputs that are not 16-byte
aligned (element loads), which must give the aligned call's bits."""

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_helpers import assert_bf16_within_ulp, bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,n", [(2, 4092), (2, 4096), (3, 4100), (5, 16384), (2, 16388)])
def test_rmsnorm_row_lengths(lib, rows, n):
    g = torch.Generator().manual_seed(rows + n)
    x = torch.randn(rows, n, generator=g) * 3.0
    gain = (1 + 0.1 * torch.randn(n, generator=g)).to(torch.bfloat16)
    out = torch.empty(rows, n, dtype=torch.bfloat16, device="cuda")
    lib.sidp_rmsnorm(x.cuda(), gain.cuda(), 1e-5, out, rows, n)
    torch.cuda.synchronize()
    want = oracle.rms_norm(x.double().numpy(), oracle.bf16_bits_to_f64(bits(gain)), 1e-5)
    assert_bf16_within_ulp(bits(out), want, what="rmsnorm")


def _fma(a, b, c):
    """float32 a * b + c rounded once (but for a double rounding one time in 2^29)."""
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(np.float32)


def _butterfly_sum(v):
    for o in (32, 16, 8, 4, 2, 1):
        v = v + v[..., np.arange(64) ^ o]
    return v[..., 0]


@pytest.mark.parametrize("rows,n", [(64, 1024), (256, 8192), (64, 5120), (16, 16384), (16, 16388), (64, 4100)])
def test_rmsnorm_sums_every_row_length_in_one_order(lib, rows, n):
    """Both kernels sum thread t's chunks 1024 columns apart, then the wave's
    threads pairwise, then the four waves: the same float32 roundings, hence the
    same bits as written out here, whichever kernel takes the row."""
    g = torch.Generator().manual_seed(rows + n)
    x = torch.randn(rows, n, generator=g) * 3.0
    gain = (1 + 0.1 * torch.randn(n, generator=g)).to(torch.bfloat16)
    out = torch.empty(rows, n, dtype=torch.bfloat16, device="cuda")
    lib.sidp_rmsnorm(x.cuda(), gain.cuda(), 1e-5, out, rows, n)
    torch.cuda.synchronize()
    v = x.numpy()
    padded = np.zeros((rows, -(-n // 1024) * 1024), np.float32)
    padded[:, :n] = v
    q = padded.reshape(rows, -1, 256, 4)  # [row, turn, thread, column of the chunk]
    q = _fma(q[..., 3], q[..., 3], _fma(q[..., 2], q[..., 2], _fma(q[..., 0], q[..., 0], q[..., 1] * q[..., 1])))
    ss = np.zeros((rows, 256), np.float32)
    for k in range(q.shape[1]):
        ss = ss + q[:, k]
    w = _butterfly_sum(ss.reshape(rows, 4, 64))
    total = ((w[:, 0] + w[:, 1]) + w[:, 2]) + w[:, 3]
    r = (np.float32(1) / np.sqrt(total / np.float32(n) + np.float32(1e-5))).astype(np.float32)
    want = (v * r[:, None]) * gain.float().numpy()
    assert torch.equal(out.cpu(), torch.from_numpy(want).to(torch.bfloat16))


@pytest.mark.parametrize("name", ["tiny_layer", "qwen3_32b_layer"])
def test_rope_append_unaligned_inputs_bitexact(lib, name):
    cfg = synth.get_config(name, qk_norm=1, num_layers=1)
    Hq, Hkv, D = cfg["num_q_heads"], cfg["num_kv_heads"], cfg["head_dim"]
    ctx = np.array([0, 5, 16, 200], np.int32)
    B, nblk, width = len(ctx), 40, 16
    bt = torch.tensor(lib.sidp_kv_alloc(ctx, 1, 16, nblk, 3, width), dtype=torch.int32, device="cuda")
    pos = torch.tensor(ctx, dtype=torch.int32, device="cuda")
    g = torch.Generator().manual_seed(5)
    src = [torch.randn(n, generator=g).to(torch.bfloat16) for n in (B * (Hq + 2 * Hkv) * D, D, D)]
    outs = []
    for offset in (0, 1):
        t = [torch.zeros(s.numel() + 8, dtype=torch.bfloat16, device="cuda") for s in src]
        qkv, gq, gk = (b[offset:offset + s.numel()].copy_(s) for b, s in zip(t, src))
        qbuf = torch.zeros(B * Hq * D + 8, dtype=torch.bfloat16, device="cuda")
        q = qbuf[offset:offset + B * Hq * D]
        kc = torch.zeros(nblk, Hkv, D // 8, 16, 8, dtype=torch.bfloat16, device="cuda")
        vc = torch.zeros(nblk, Hkv, D, 16, dtype=torch.bfloat16, device="cuda")
        h = lib.sidp_create(lib.make_config(cfg, B, 2048))
        try:
            lib.sidp_kv_attach(h, kc, vc, nblk, 1)
            lib.sidp_rope_append(h, qkv, pos, bt, width, B, gq, gk, 0, q)
            lib.sidp_sync(h)
        finally:
            lib.sidp_destroy(h)
        outs.append((q.clone(), kc, vc))
    assert bool((outs[0][0] != 0).any())
    assert all(torch.equal(a, b) for a, b in zip(*outs))


@pytest.mark.parametrize("name,batch", [("tiny_layer", 64), ("qwen3_32b_layer", 32)])
def test_qk_norm_sums_a_head_in_one_order(lib, name, batch):
    """A head's squares are summed as pairs (i, i + D/2) and then pairwise from
    the highest bit of i down: the float32 roundings written out here, so the
    queries at position 0 (no rotation) come out bit for bit."""
    cfg = synth.get_config(name, qk_norm=1, num_layers=1)
    Hq, Hkv, D = cfg["num_q_heads"], cfg["num_kv_heads"], cfg["head_dim"]
    g = torch.Generator().manual_seed(9)
    qkv = torch.randn(batch, Hq + 2 * Hkv, D, generator=g).to(torch.bfloat16)
    gain = (1 + 0.1 * torch.randn(D, generator=g)).to(torch.bfloat16)
    q = torch.empty(batch, Hq, D, dtype=torch.bfloat16, device="cuda")
    kc = torch.zeros(batch, Hkv, D // 8, 16, 8, dtype=torch.bfloat16, device="cuda")
    vc = torch.zeros(batch, Hkv, D, 16, dtype=torch.bfloat16, device="cuda")
    pos = torch.zeros(batch, dtype=torch.int32, device="cuda")
    bt = torch.arange(batch, dtype=torch.int32, device="cuda").view(batch, 1)
    h = lib.sidp_create(lib.make_config(cfg, batch, 2048))
    try:
        lib.sidp_kv_attach(h, kc, vc, batch, 1)
        lib.sidp_rope_append(h, qkv.cuda(), pos, bt, 1, batch, gain.cuda(), gain.cuda(), 0, q)
        lib.sidp_sync(h)
    finally:
        lib.sidp_destroy(h)
    x = qkv.float().numpy()
    t = np.zeros((batch, Hq + 2 * Hkv, 64), np.float32)
    t[..., :D // 2] = _fma(x[..., D // 2:], x[..., D // 2:], x[..., :D // 2] * x[..., :D // 2])
    r = np.float32(1) / np.sqrt(_butterfly_sum(t) / np.float32(D) + np.float32(cfg["qk_norm_eps"]))
    want = torch.from_numpy((x * r[..., None].astype(np.float32)) * gain.float().numpy()).to(torch.bfloat16)
    assert torch.equal(q.cpu(), want[:, :Hq])
    k = lib.k_blocks_from_lib(kc)[:, :, 0].cpu()
    assert torch.equal(k, want[:, Hq:Hq + Hkv])
