"""Whole-network forward kernels with two and four waves per workgroup (narrow layers, more rows than
the device holds at once) against the eight-wave form on parts of the batch: a row's outputs and
the gradients of a backward pass from the kept activations do not depend on the form, bit for bit.

Batches at the edge where the forms change (512 workgroups of 32 rows), one row more and a ragged
larger one; widths at the edges of two and four waves; with an input map.
"""
import pytest
import torch

pytestmark = pytest.mark.gpu

EDGE = 512 * 32


def _net(widths, batch, seed):
    from paper_2302_14344_amd.solver import Mlp
    g = torch.Generator().manual_seed(seed)
    m = Mlp(widths, batch)
    n = sum(a * b + b for a, b in zip(widths[:-1], widths[1:]))
    m.set_params((torch.randn(n, generator=g) * 0.3).cuda())
    m.set_input_affine(torch.rand(widths[0], generator=g).cuda() + 0.5, torch.randn(widths[0], generator=g).cuda())
    return m


@pytest.mark.parametrize("batch", [EDGE, EDGE + 1, 3 * EDGE + 77])
@pytest.mark.parametrize("widths", [[12, 64, 64, 6], [5, 33, 17, 3], [12, 65, 6], [27, 128, 100, 15], [27, 129, 64, 15]])
def test_rows_do_not_depend_on_the_form(widths, batch):
    print(widths, batch, flush=True)
    x = torch.randn(batch, widths[0], generator=torch.Generator().manual_seed(5)).cuda()
    whole = _net(widths, batch, 3)
    y, yi = whole.forward(x), whole.infer(x)
    part = _net(widths, EDGE // 2, 3)
    for r in range(0, batch, EDGE // 2):
        n = min(EDGE // 2, batch - r)
        ref = part.forward(x[r:r + n].contiguous())
        assert torch.equal(y[r:r + n], ref) and torch.equal(yi[r:r + n], ref)
    # the kept activations: gradients of the last rows alone (weights zero elsewhere) in both forms
    t = torch.zeros(batch, widths[-1]).cuda()
    wt = torch.zeros(batch, widths[-1]).cuda()
    wt[-100:] = 1.0
    whole.forward(x)
    g = whole.backward(t, wt, want_grad=True)[1]
    part.forward(x[-100:].contiguous())
    h = part.backward(t[-100:].contiguous(), wt[-100:].contiguous(), want_grad=True)[1]
    # sums of 100 rows in another split of the batch: FP32 rounding of sums of 100 products
    assert torch.allclose(g, h, rtol=0.0, atol=100 * 6e-8 * float(h.abs().max()) * 4)
