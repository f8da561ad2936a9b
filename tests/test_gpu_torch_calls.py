"""The native form of the ordinary calls against the general path (an output tensor given): same results, same
refusals, the current stream, and nothing taken that the general path would not take."""
import threading

import pytest
import torch

from paper_1911_03458_amd import binding as mb

pytestmark = pytest.mark.gpu


def _h(*shape):
    return torch.randn(shape, device="cuda").half()


def _f(*shape):
    return torch.rand(shape, device="cuda")


def _u(*shape):
    return torch.randint(0, 256, shape, device="cuda", dtype=torch.uint8)


CALLS = {
    "conv2d": (lambda: mb.merit_plan_conv2d(2, 16, 9, 11, 24, 3, 3, 1, 1, 1, 1), mb.merit_conv2d,
               lambda: (_h(2, 16, 9, 11), _h(24, 16, 3, 3))),
    "residual": (lambda: mb.merit_plan_conv2d_residual(2, 16, 9, 11, 24, 3, 3, 1, 1, 1, 1), mb.merit_conv2d_residual,
                 lambda: (_h(2, 16, 9, 11), _h(24, 16, 3, 3), _h(2, 24, 9, 11))),
    "pool2d": (lambda: mb.merit_plan_pool2d(2, 3, 9, 11, 3, 3, 2, 2, 1, 1, 1), mb.merit_pool2d,
               lambda: (_f(2, 3, 9, 11),)),
    "depthwise": (lambda: mb.merit_plan_conv2d_depthwise(2, 8, 9, 11, 3, 3, 1, 1, 1, 1), mb.merit_conv2d_depthwise,
                  lambda: (_h(2, 8, 9, 11), _h(8, 3, 3))),
    "sepfilter": (lambda: mb.merit_plan_sepfilter(2, 20, 30, 5), mb.merit_sepfilter,
                  lambda: (_f(2, 20, 30), _f(5), _f(5))),
    "bilateral": (lambda: mb.merit_plan_bilateral(1, 20, 30, 5), mb.merit_bilateral,
                  lambda: (_f(1, 20, 30), _f(5) + 0.1, _f(5) + 0.1, -0.5)),
    "correlation": (lambda: mb.merit_plan_correlation(1, 16, 8, 16, 2, 1), mb.merit_correlation,
                    lambda: (_h(1, 16, 8, 16), _h(1, 16, 8, 16))),
    "sad": (lambda: mb.merit_plan_sad(40, 72, 8, 4), mb.merit_sad_search, lambda: (_u(40, 72), _u(40, 72))),
}


@pytest.mark.parametrize("name", list(CALLS))
def test_ordinary_calls_match_the_general_path(name):
    make, op, inputs = CALLS[name]
    plan, args = make(), inputs()
    got = op(plan, *args)
    pair = isinstance(got, tuple)
    want = op(plan, *args, *[torch.empty_like(t) for t in (got if pair else (got,))])
    for a, b in zip(got if pair else (got,), want if pair else (want,)):
        assert a.dtype == b.dtype and a.shape == b.shape and torch.equal(a, b)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):        # (results of a queue of work on the other stream must be in it)
        again = op(plan, *[(a * 1) if isinstance(a, torch.Tensor) else a for a in args])
    side.synchronize()
    for a, b in zip(again if pair else (again,), want if pair else (want,)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("name", list(CALLS))
def test_what_the_general_path_refuses_stays_refused(name):
    make, op, inputs = CALLS[name]
    plan, args = make(), inputs()
    first, rest = args[0], args[1:]
    with pytest.raises(TypeError):
        op(plan, first.cpu(), *rest)
    with pytest.raises(TypeError):
        op(plan, first.double(), *rest)
    with pytest.raises(ValueError):
        op(plan, first[:, :-1].contiguous(), *rest)
    with pytest.raises(ValueError):
        op(plan, torch.stack((first, first), -1)[..., 0], *rest)      # right shape, not contiguous
    flat = torch.zeros(first.numel() + 1, dtype=first.dtype, device="cuda")
    with pytest.raises(mb.MeritError) as e:                            # contiguous, off the 16-byte grid
        op(plan, flat[1:].view(first.shape), *rest)
    assert e.value.status == mb.MERIT_ERR_ALIGNMENT
    with pytest.raises(Exception):
        torch.vmap(lambda t: op(plan, t, *rest))(first[None])
    plan.destroy()
    with pytest.raises(ValueError):
        op(plan, *args)


@pytest.mark.parametrize("name", list(CALLS))
def test_without_the_module(name, monkeypatch):
    """A process that cannot load it: every call through ctypes, with the same results."""
    make, op, inputs = CALLS[name]
    args = inputs()
    want = op(make(), *args)
    monkeypatch.setattr(mb, "_calls", False)
    monkeypatch.setattr(mb, "_ops", {})
    got = op(make(), *args)
    for a, b in zip(got if isinstance(got, tuple) else (got,), want if isinstance(want, tuple) else (want,)):
        assert torch.equal(a, b)


def test_packed_weights_and_a_changed_tiling():
    plan = mb.merit_plan_conv2d(2, 40, 16, 16, 72, 3, 3, 1, 1, 1, 1)
    x, w = _h(2, 40, 16, 16), _h(72, 40, 3, 3)
    packed, want = mb.merit_conv2d_pack_weights(plan, w), mb.merit_conv2d(plan, x, w)
    assert torch.equal(mb.merit_conv2d_packed(plan, x, packed), want)
    with pytest.raises(ValueError):
        mb.merit_conv2d_packed(plan, x, packed[:-8])
    with pytest.raises(ValueError):
        mb.merit_conv2d_packed(plan, x[:1], packed)
    before = mb.merit_plan_packed_weights_bytes(plan)
    plan.set_tile((0, 0, 8, 32))                    # the same plan, another size of packed copy
    assert mb.merit_plan_packed_weights_bytes(plan) != before
    with pytest.raises(ValueError):
        mb.merit_conv2d_packed(plan, x, packed)
    assert torch.equal(mb.merit_conv2d_packed(plan, x, mb.merit_conv2d_pack_weights(plan, w)), want)


@pytest.mark.parametrize("name", list(CALLS))
def test_under_graph_capture(name):
    """The output comes from the graph's pool, the launch is in the graph: every replay sees the inputs of its time."""
    make, op, inputs = CALLS[name]
    plan, args = make(), inputs()
    op(plan, *args)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = op(plan, *args)
    got = got if isinstance(got, tuple) else (got,)
    for _ in range(4):
        for a, b in zip(args, inputs()):
            if isinstance(a, torch.Tensor):
                a.copy_(b)
        graph.replay()
        torch.cuda.synchronize()
        want = op(plan, *args)
        for a, b in zip(got, want if isinstance(want, tuple) else (want,)):
            assert torch.equal(a, b)


@pytest.mark.parametrize("name", list(CALLS))
def test_threads_share_a_plan(name):
    """Four threads, a stream each, one plan."""
    make, op, inputs = CALLS[name]
    plan = make()
    sets = [inputs() for _ in range(4)]
    wants = [op(plan, *args) for args in sets]
    torch.cuda.synchronize()
    wrong = []

    def work(args, want):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(20):
                    got = op(plan, *args)
                    stream.synchronize()
                    for a, b in zip(got if isinstance(got, tuple) else (got,), want if isinstance(want, tuple) else (want,)):
                        if not torch.equal(a, b):
                            wrong.append("differs")
        except Exception as e:          # (an assertion in a thread is lost)
            wrong.append(repr(e))

    threads = [threading.Thread(target=work, args=z) for z in zip(sets, wants)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def test_tensor_subclass_takes_the_general_path():
    class Sub(torch.Tensor):
        pass

    plan, x = mb.merit_plan_pool2d(1, 3, 8, 8, 3, 3, 2, 2, 1, 1, 0), _f(1, 3, 8, 8)
    assert torch.equal(mb.merit_pool2d(plan, x.as_subclass(Sub)), mb.merit_pool2d(plan, x))
    with torch.inference_mode():
        assert mb.merit_pool2d(plan, x).is_inference()
    assert not mb.merit_pool2d(plan, torch.nn.Parameter(x)).requires_grad
