"""Where torch follows the operations, the package leaves them to torch."""
import pytest
import torch
from torch.fx.experimental.proxy_tensor import make_fx
from torch.overrides import TorchFunctionMode
from torch.utils._python_dispatch import TorchDispatchMode

from paper_2503_16424_amd import bz, cnn


class Dispatch(TorchDispatchMode):
    def __init__(self):
        super().__init__()
        self.seen = []

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        self.seen.append(func)
        return func(*args, **(kwargs or {}))


class Function(TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def test_every_follower_is_seen():
    seen = []

    def look(x):
        seen.append(bz.followed())
        return x * 1.0

    x = torch.ones(3)
    look(x)
    assert seen == [False]
    with Dispatch():
        look(x)
    with Function():
        look(x)
    make_fx(look)(x)
    torch.func.vmap(look)(x)
    torch.func.jvp(look, (x,), (x,))
    with torch.autograd.forward_ad.dual_level():
        look(x)
    assert all(seen[1:]) and len(seen) >= 7 and not bz.followed()


@pytest.mark.gpu
def test_decode_under_modes_and_tracing():
    z = torch.randn((4, cnn.OUT), device="cuda")
    want = cnn.decode(z.clone().requires_grad_()).detach()     # torch's operations
    with Dispatch() as mode:
        got = cnn.decode(z)
    assert torch.ops.aten.sigmoid.default in mode.seen and torch.equal(got, want)
    graph = make_fx(lambda t: cnn.decode(t))(z)
    other = torch.randn_like(z)
    assert torch.equal(graph(other), cnn.decode(other.clone().requires_grad_()).detach())


@pytest.mark.gpu
def test_decode_on_another_device_is_left_to_torch(monkeypatch):
    z = torch.randn((4, cnn.OUT), device="cuda")
    monkeypatch.setattr(torch.cuda, "current_device", lambda: z.device.index + 1)
    monkeypatch.setattr(bz, "_check", lambda *a: pytest.fail("launched on another device"))
    assert torch.equal(cnn.decode(z), cnn.decode(z.clone().requires_grad_()).detach())


@pytest.mark.gpu
def test_fit_step_under_a_mode():
    from paper_2503_16424_amd import optim, scenes
    f = optim.Fitter(bz.Rasterizer(scenes.small_mixed(1)), optim.FitConfig())
    for d in (f.rast.d_ctrl, f.rast.d_color, f.rast.d_opacity, f.rast.d_width):
        d.fill_(1e-3)
    f.update()                                              # makes the optimiser's state
    assert f._update_in_one_launch()
    with Dispatch() as mode:
        f.update()
        updated = len(mode.seen)
        f.push()
    seen = {str(op) for op in mode.seen}
    assert any(s.startswith("aten.clamp_") for s in seen) and "aten.copy_.default" in seen
    assert len(mode.seen) > updated
