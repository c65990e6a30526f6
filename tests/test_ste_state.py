"""The state QuasarLinear.step keeps on the module, without a GPU: the library
call is replaced by one that records its arguments."""
import pytest
import torch

from paper_2608_13966_amd import quasar as Q
from paper_2608_13966_amd.ste import QuasarLinear


@pytest.fixture
def steps(monkeypatch):
    """The step numbers the library was called with."""
    calls = []

    def reconstruct(W, v, g, *, want_diag, **cfg):
        d = Q.Descriptor(*W.shape, w_dtype=Q.F32, g_dtype=Q.F32, **cfg)
        return dict(Q.alloc_outputs(d, W, want_r=False, want_diag=want_diag, has_amax=True), r=torch.zeros_like(W))

    monkeypatch.setattr(Q, "reconstruct", reconstruct)
    monkeypatch.setattr(Q, "adamw_reconstruct", lambda *a, step, **kw: calls.append(int(step)))
    return calls


def _step(layer):
    layer.weight.grad = torch.ones_like(layer.weight)
    layer.step()


def test_the_step_count_is_the_modules_own(steps):
    layer = QuasarLinear(128, 2, device="cpu")
    _step(layer)
    layer.t = 41
    _step(layer)
    assert steps == [1, 42] and layer.t == 42


def test_a_step_count_in_a_buffer_is_saved_with_the_state(steps):
    class Counted(QuasarLinear):
        def __init__(self, *a, **kw):
            super().__init__(*a, **kw)
            del self.t
            self.register_buffer("t", torch.tensor(7))

    layer = Counted(128, 2, device="cpu")
    _step(layer)
    assert steps == [8] and int(layer.state_dict()["t"]) == 8 and "t" not in layer.__dict__
    layer.load_state_dict({**layer.state_dict(), "t": torch.tensor(20)})
    _step(layer)
    assert steps == [8, 21]


def test_results_deleted_by_the_caller_come_back(steps):
    layer = QuasarLinear(128, 2, device="cpu")
    _step(layer)
    codes = layer.codes
    assert codes is layer._out["codes"] and layer.scales is layer._out["scales"]
    del layer.codes
    layer.zeros = None
    _step(layer)
    assert layer.codes is codes and layer.zeros is layer._out["zeros"]
