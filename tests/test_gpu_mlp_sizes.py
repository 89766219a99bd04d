"""Sizes and alignments at which the network kernels change their split.

Forward: one wave per 16 states up to 32,768 states, 64 states per wave above; ragged tails; parameters
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


@pytest.mark.parametrize("sites", [(0, 17), (3, 9)])
def test_a_state_that_is_not_a_number_stays_alone(sites):
    """Two opposite infinities in a row of W1 cancel to NaN where the two sites agree and saturate where they do
    not: every state's outputs are those it has on its own (one wave per 16 states, one tile)."""
    torch = torch_cuda()
    import paper_1707_03974_amd as pdz
    from paper_1707_03974_amd import mlp
    net, _ = _net(14)
    w = net.w.cpu()
    w[5 * 32 + sites[0]], w[5 * 32 + sites[1]] = float("inf"), float("-inf")
    net = mlp.Net(params=w)
    n = 200_000 + 77
    up, dn = _states(np.random.default_rng(3), n)
    occ = _occ(up, dn)
    out = net.forward(occ)
    alone = torch.cat([net.forward(occ[k:k + 10_000].contiguous()) for k in range(0, n, 10_000)])
    bits = np.concatenate([(up[:, None] >> np.arange(16)) & 1, (dn[:, None] >> np.arange(16)) & 1], axis=1)
    nan = torch.from_numpy(bits[:, sites[0]] == bits[:, sites[1]]).cuda()
    assert 0.2 < nan.float().mean().item() < 0.8
    assert torch.equal(torch.isnan(out), nan[:, None].expand(n, 2)) and torch.equal(torch.isnan(alone), torch.isnan(out))
    assert torch.equal(out[~nan], alone[~nan])
    # the start vector of a state that is a number: sign * exp(min(o_0, 60))
    p = pdz.Problem(16, [(0, 1, 1.0)], 1.0, 4, 3)
    iu, idn = np.meshgrid(np.arange(p.info["D_up"]), np.arange(p.info["D_dn"]), indexing="ij")
    su = pdz.unrank(16, 4, torch.arange(p.info["D_up"], dtype=torch.int32, device="cuda"))
    sd = pdz.unrank(16, 3, torch.arange(p.info["D_dn"], dtype=torch.int32, device="cuda"))
    pairs = torch.stack([su[torch.from_numpy(iu.ravel()).cuda()], sd[torch.from_numpy(idn.ravel()).cuda()]], dim=1)
    o = torch.cat([net.forward(pairs[k:k + 10_000].contiguous()) for k in range(0, p.D, 10_000)]).double()
    v = mlp.start_vector(p, net, torch.float64)
    ok = ~torch.isnan(o[:, 0])
    expect = torch.exp(o[:, 0].clamp(max=60.0)) * torch.where(o[:, 1] >= 0, 1.0, -1.0)
    assert 0.2 < ok.double().mean().item() < 0.8
    assert torch.allclose(v[ok], expect[ok], rtol=1e-13, atol=0.0)


@pytest.mark.parametrize("n", [32767, 32768, 32769, 33000])
def test_forward_where_the_kernel_changes(n):
    """The kernel of long lists and the one of short lists (each list in two halves) give the same bits."""
    torch = torch_cuda()
    net, _ = _net(15)
    occ = _occ(*_states(np.random.default_rng(n), n))
    act = torch.empty(n * 384, dtype=torch.int16, device="cuda")
    out = net.forward(occ, act=act)
    for a, b in ((0, n // 2), (n // 2, n)):
        m = b - a
        part_act = torch.empty(m * 384, dtype=torch.int16, device="cuda")
        assert torch.equal(net.forward(occ[a:b].contiguous(), act=part_act), out[a:b])
        assert torch.equal(part_act[:m * 128], act[a * 128:b * 128])
        assert torch.equal(part_act[m * 128:2 * m * 128].view(128, m), act[n * 128:2 * n * 128].view(128, n)[:, a:b])
        assert torch.equal(part_act[2 * m * 128:], act[(2 * n + a) * 128:(2 * n + b) * 128])
