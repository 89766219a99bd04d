"""Launch plans with some fields left automatic: what a set field does not go with is not run.

The automatic up pass (16-byte lanes in FP32, batches of 16 hops in FP64) does not exist at every chunk
width, and the variants that preload a row or use wide lanes do not exist at the automatic width.  Every
accepted plan of one down family gives the automatic plan's y bit for bit.
"""
import itertools

import pytest

import synth
from tests._gpu import torch_cuda, to_dev

pytestmark = pytest.mark.gpu

WIDTHS = {"f32": (32, 64, 128, 256), "f64": (16, 32, 64, 128)}


def _ring(N):
    return [(i, (i + 1) % N, 1.0) for i in range(N)]


def _runs(name, cw, up):
    """Chunk widths and variants that have a kernel."""
    if up == 2:
        return cw <= 64
    return up != 4 or cw * (4 if name == "f32" else 8) <= 512


@pytest.mark.parametrize("name", ["f32", "f64"])
@pytest.mark.parametrize("n,nu,nd", [(9, 4, 4), (11, 5, 6), (13, 4, 5), (13, 9, 1)])
def test_partial_plans_run_a_kernel_of_their_width(name, n, nu, nd):
    torch = torch_cuda()
    import paper_1707_03974_amd as pdz
    g = pdz.Problem(n, _ring(n), 3.25, nu, nd)
    x = to_dev(synth.random_vector(g.D, 5), torch.float32 if name == "f32" else torch.float64)
    ref = g.hv(x)
    for cw, up, mp in itertools.product((0,) + WIDTHS[name], range(5), (0, 1, 2, 3)):
        if cw and up and not _runs(name, cw, up):
            with pytest.raises(pdz.PdzError):
                g.set_plan(name, 0, cw, up, mp)
            continue
        g.set_plan(name, 0, cw, up, mp)
        pl = g.get_plan(name)
        assert _runs(name, pl["up_cw"], pl["up"]), (cw, up, mp, pl)
        assert pl["up_cw"] == (cw or pl["up_cw"]) and pl["up"] == (up or pl["up"]) and pl["map"] == (mp or pl["map"])
        if mp in (0, 2):
            assert torch.equal(g.hv(x), ref), (cw, up, mp, pl)
        # what is set holds: the resolved plan, set whole, is the same plan
        g.set_plan(name, *(pl[k] for k in ("down", "up_cw", "up", "map")))
        assert g.get_plan(name) == pl


@pytest.mark.parametrize("cw,up", [(32, 4), (64, 4), (64, 0), (64, 2), (256, 0), (0, 0)])
def test_rows_past_32_bit_offsets_are_all_summed(cw, up):
    """A pitch that puts the last rows past 2^32 elements: one up pass, whatever the plan's (17 GB vectors)."""
    torch = torch_cuda()
    import paper_1707_03974_amd as pdz
    g = pdz.Problem(9, _ring(9), 3.25, 4, 4)
    x = to_dev(synth.random_vector(g.D, 6), torch.float32)
    ref = g.hv(x).view(g.info["D_up"], -1)
    rows, cols = ref.shape
    pitch = 2 ** 32 // rows + 1
    xp, yp = (torch.empty(rows * pitch, dtype=torch.float32, device="cuda") for _ in range(2))
    xp.view(rows, pitch)[:, :cols] = x.view(rows, cols)
    g.set_plan("f32", 0, cw, up, 0)
    g.hv_pitched(xp, pitch, yp)
    assert torch.equal(yp.view(rows, pitch)[:, :cols], ref)
