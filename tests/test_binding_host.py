"""The binding where its native short way is not there: every entry point goes the general way, nothing is compiled."""
import pytest


@pytest.fixture
def binding(monkeypatch):
    """The binding as it is before it has seen a GPU, on a torch that says it has one, without the native module."""
    import torch

    import paper_2002_12418_amd.binding as b
    import paper_2002_12418_amd.build as build

    def no_compiler(*args, **kw):
        raise RuntimeError("g++ failed")

    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(torch.cuda, "init", lambda: None)
    monkeypatch.setattr(b, "_current_stream", None)
    monkeypatch.setattr(b, "_float32", None)
    monkeypatch.setattr(b, "_fast_call", None)
    monkeypatch.setattr(build, "build_fast_call", no_compiler)
    monkeypatch.setattr(build, "fast_call_path", lambda: None)
    return b


def test_the_stream_is_found(binding):
    with pytest.warns(RuntimeWarning):
        assert binding._find_current_stream() is not None
    assert binding._fast_call is None and binding._float32 is not None


def test_a_static_call_and_a_plan_reach_the_library(binding, monkeypatch):
    """The library is asked, and its answer is the error that is raised: there is no device here."""
    import torch

    from conv_workloads import ConvLayer
    monkeypatch.setattr(binding, "_find_current_stream", lambda: setattr(binding, "_float32", torch.float32))
    layer = ConvLayer("l", 1, 4, 5, 5, 4, 3, 3, 1, 1)
    x, w, y = torch.zeros(1, 4, 5, 5), torch.zeros(4, 4, 3, 3), torch.zeros(1, 4, 5, 5)
    with pytest.raises(binding.MnnError):
        binding.conv_run_static(layer, -1, x, w, None, y)

    calls = []

    class Library:                          # plans without a device
        def __getattr__(self, name):
            def f(*args):
                calls.append(name)
                return 0
            return f

    monkeypatch.setattr(binding, "lib", Library())
    monkeypatch.setattr(binding.ConvPlan, "_check_tensors", lambda self, *a: None)
    monkeypatch.setattr(binding, "_stream_handle", lambda stream: 0)
    plan = binding.ConvPlan.for_layer(layer)
    y = torch.zeros(plan.out_shape)
    for _ in range(2):
        assert plan.run(x, w, None, y) is y
    w.add_(1)
    plan.run(x, w, None, y)                 # new values behind the same pointer
    plan.set_weights = None
    plan.close()
    assert calls.count("mnn_conv_run") == 3 and calls.count("mnn_conv_invalidate_weights") == 1
