"""Saved-tensor hooks around the autograd functions."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _points():
    g = torch.Generator("cuda").manual_seed(2500)
    return (torch.randn((70, 3), device="cuda", dtype=torch.float64, generator=g),
            torch.randn((70, 36), device="cuda", dtype=torch.float64, generator=g))


# the saved values come back, in another layout
HOOKS = {"transposed": (lambda t: t.t().contiguous() if t.dim() == 2 else t, lambda t: t.t() if t.dim() == 2 else t),
         "host": (lambda t: t.cpu(), lambda t: t.cuda())}


@pytest.mark.parametrize("hooks", sorted(HOOKS))
@pytest.mark.parametrize("e3nn", [False, True])
def test_first_derivatives_under_hooks(e3nn, hooks):
    import paper_2302_08381_amd as sph
    x0, w = _points()
    f = (lambda x: sph.e3nn_spherical_harmonics(x, 5)) if e3nn else (lambda x: sph.spherical_harmonics(x, 5))
    grads = []
    for pack, unpack in (HOOKS[hooks], (lambda t: t, lambda t: t)):
        x = x0.clone().requires_grad_()
        with torch.autograd.graph.saved_tensors_hooks(pack, unpack):
            y = f(x)
        grads.append(torch.autograd.grad(y, x, w)[0])
    assert torch.equal(grads[0], grads[1])


@pytest.mark.parametrize("hooks", sorted(HOOKS))
def test_second_derivatives_under_hooks(hooks):
    import paper_2302_08381_amd as sph
    x0, w = _points()
    grads = []
    for pack, unpack in (HOOKS[hooks], (lambda t: t, lambda t: t)):
        x = x0.clone().requires_grad_()
        with torch.autograd.graph.saved_tensors_hooks(pack, unpack):
            g, = torch.autograd.grad(sph.spherical_harmonics(x, 5), x, w, create_graph=True)
        grads.append(torch.autograd.grad(g, x, x0)[0])
    assert torch.equal(grads[0], grads[1])
