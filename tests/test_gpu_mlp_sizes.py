"""Sizes and alignments at which the network kernels change their split.

Forward: one wave per 16 states up to 16,384 states, 64 states per wave above; ragged tails; parameters
and activations that are not 16-byte aligned.  Backward: chunks of 64 states, one slice per work group,
256 slices at most.  Loss: one work group up to 8,192 states.  Bounds as in test_gpu_mlp: 1e-2 relative
for outputs and gradients (BF16 activations), FP32 rounding for the loss.
"""
import ctypes

import numpy as np
import pytest

from oracle import mlp as ref
from tests._gpu import torch_cuda, to_host
from tests.test_gpu_mlp import _net, _occ, _states, _gradient_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [15, 17, 16384, 16385, 16384 + 256 * 3 + 33])
def test_forward_at_tile_edges(n):
    net, theta = _net(11)
    up, dn = _states(np.random.default_rng(n), n)
    out = to_host(net.forward(_occ(up, dn))).astype(np.float64)
    expect, _ = ref.forward(theta, up, dn, round_bf16=True)
    err = np.abs(out - expect)
    assert np.all(err <= 1e-2 * np.maximum(1.0, np.abs(expect))), float(err.max())
    assert np.median(err) < 1e-3


def test_both_forward_kernels_give_the_same_bits():
    # the same products in the same order: only the states per wave differ
    torch = torch_cuda()
    net, _ = _net(12)
    n = 20000
    occ = _occ(*_states(np.random.default_rng(1), n))
    act, few = (torch.empty(k * 384, dtype=torch.int16, device="cuda") for k in (n, 1000))
    out = net.forward(occ, act=act)
    part = net.forward(occ[:1000].contiguous(), act=few)
    assert torch.equal(out[:1000], part)
    assert torch.equal(act[:1000 * 128], few[:1000 * 128])
    assert torch.equal(act[2 * n * 128:2 * n * 128 + 1000 * 128], few[2000 * 128:])
    assert torch.equal(act[n * 128:2 * n * 128].view(128, n)[:, :1000], few[1000 * 128:2000 * 128].view(128, 1000))


@pytest.mark.parametrize("n", [48, 16400])
def test_unaligned_parameters_and_activations(n):
    torch = torch_cuda()
    net, _ = _net(13)
    occ = _occ(*_states(np.random.default_rng(2), n))
    act = torch.empty(n * 384, dtype=torch.int16, device="cuda")
    out = net.forward(occ, act=act)
    wb = torch.empty(net.wb.numel() + 1, dtype=torch.int16, device="cuda")
    wb[1:].copy_(net.wb)
    shifted = torch.empty(n * 384 + 1, dtype=torch.int16, device="cuda")
    aligned, net.wb = net.wb, wb[1:]
    got = net.forward(occ, act=shifted[1:])
    net.wb = aligned
    assert torch.equal(out, got)
    assert torch.equal(act, shifted[1:])


@pytest.mark.parametrize("n,seed", [(64, 5), (96, 6), (160, 7), (64 * 256, 8), (64 * 256 + 32, 9)])
def test_backward_at_chunk_and_slice_edges(n, seed):
    g, e = _gradient_case(n, seed)
    for name, part in ref.unpack(np.arange(ref.N_PARAMS)).items():
        k = part.ravel()
        rel = np.linalg.norm(g[k] - e[k]) / max(np.linalg.norm(e[k]), 1e-30)
        assert rel <= 1e-2, (name, rel)


@pytest.mark.parametrize("n", [1, 1023, 8192, 8193])
def test_loss_at_work_group_edges(n):
    torch = torch_cuda()
    from paper_1707_03974_amd import _lib
    rng = np.random.default_rng(n)
    out = rng.normal(0.0, 2.0, (n, 2)).astype(np.float32)
    tgt = np.stack([rng.normal(-5, 1, n), rng.choice([-1.0, 1.0], n)], axis=1).astype(np.float32)
    o, t = torch.from_numpy(out).cuda(), torch.from_numpy(tgt).cuda()
    d = torch.empty_like(o)
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    L = _lib.load()
    nb = ctypes.c_size_t()
    _lib.check(L.pdz_mlp_workspace_size(n, ctypes.byref(nb)))
    ws = torch.empty(nb.value, dtype=torch.uint8, device="cuda")
    p = [ctypes.c_void_p(x.data_ptr()) for x in (o, t, d, loss, ws)]
    _lib.check(L.pdz_mlp_loss(p[0], p[1], n, p[2], p[3], p[4], ws.numel(), None))
    torch.cuda.synchronize()
    expect, dout = ref.loss_and_dout(out.astype(np.float64), tgt[:, 0].astype(np.float64), tgt[:, 1])
    assert abs(loss.item() - expect) <= 1e-6 * abs(expect)
    assert np.allclose(to_host(d), dout, rtol=1e-5, atol=1e-9)
