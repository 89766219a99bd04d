"""Sizes and alignments at which the network kernels change their split.

Forward: one wave per 16 states up to 16,384 states, 64 states per wave above; ragged tails; parameters
and activations that are not 16-byte aligned.  Bounds as in test_gpu_mlp: 1e-2 relative (BF16
activations).
"""
import numpy as np
import pytest

from oracle import mlp as ref
from tests._gpu import torch_cuda, to_host
from tests.test_gpu_mlp import _net, _occ, _states

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
