"""The binding's compute calls: what the extension takes and what it leaves to the Python checks must be told apart."""
import ctypes

import pytest
import torch

import paper_1810_02272_amd as conv
from paper_1810_02272_amd import binding

DEV = "cuda:0"


def layer():
    d = conv.conv_desc_create(conv.ConvParams(2, 3, 9, 9, 5, 3, 3, pad_h=1, pad_w=1))
    gen = torch.Generator().manual_seed(3)
    x, w, b = (torch.randn(s, generator=gen).to(DEV) for s in ((2, 3, 9, 9), (5, 3, 3, 3), (5,)))
    ws = torch.empty(conv.conv_desc_workspace_bytes(d) // 4 + 1, device=DEV)
    return d, x, w, b, torch.full((2, 5, 9, 9), float("nan"), device=DEV), ws


def test_arguments_out_of_order_on_the_cpu():
    """Nothing here is a device tensor: the extension declines every call and the checks raise what they always raised."""
    d = conv.conv_desc_create(conv.ConvParams(2, 3, 9, 9, 5, 3, 3))
    t = torch.zeros(2, 3, 9, 9)
    with pytest.raises(TypeError, match="x: expected a CUDA/HIP tensor"):
        conv.conv_forward(d, t, t, t, t)
    with pytest.raises(conv.ConvError) as e:
        conv.conv_forward(d, None, None, None, None, stream=0)
    assert e.value.status == binding.CONV_EINVAL
    conv.conv_desc_destroy(d)
    with pytest.raises(conv.ConvError):
        conv.conv_forward(d, None, None, None, None, stream=0)
    with pytest.raises(TypeError, match="aprob"):
        conv.pg_sigmoid_sample_action(t, t, t)
    with pytest.raises(TypeError):
        conv.conv_forward(d, t)


def test_an_extension_that_cannot_be_had_leaves_the_python_checks(monkeypatch):
    """Built for another PyTorch or Python and not to be built again: a warning, and descriptors and checks as ever."""
    from paper_1810_02272_amd import build

    assert build.marshal_fits()

    def fails():
        raise RuntimeError("no compiler")

    monkeypatch.setattr(build, "marshal_target", lambda: "for torch 0.1 and Python 2.7.")
    assert not build.marshal_fits() and build.is_stale()
    monkeypatch.setattr(build, "build_marshal", fails)
    with pytest.warns(UserWarning, match="no compiler"):
        without = binding._load_marshal()
    monkeypatch.setattr(binding, "_marshal", without)
    d = conv.conv_desc_create(conv.ConvParams(2, 3, 9, 9, 5, 3, 3))
    conv.ip_desc_create(conv.IpParams(2, 3, 4))
    t = torch.zeros(2, 3, 9, 9)
    with pytest.raises(TypeError, match="x: expected a CUDA/HIP tensor"):
        conv.conv_forward(d, t, t, t, t)
    with pytest.raises(TypeError, match="aprob"):
        conv.pg_sigmoid_sample_action(t, t, t)


@pytest.mark.gpu
def test_calls_without_the_extension(monkeypatch):
    d, x, w, b, y, ws = layer()
    conv.conv_forward(d, x, w, b, y, ws)
    torch.cuda.synchronize()
    ref = y.clone()
    y.fill_(float("nan"))
    monkeypatch.setattr(binding, "_marshal", binding._NoMarshal())
    conv.conv_forward(d, x, w, b, y, ws)
    again = layer()  # a descriptor made without it
    conv.conv_forward(*again)
    torch.cuda.synchronize()
    assert torch.equal(y, ref) and torch.equal(again[4], ref)


@pytest.mark.gpu
def test_what_is_refused_and_what_is_accepted():
    d, x, w, b, y, ws = layer()
    conv.conv_forward(d, x, w, b, y, ws)
    torch.cuda.synchronize()
    ref = y.clone()
    ok = torch.nn.functional.conv2d(x.double().cpu(), w.double().cpu(), b.double().cpu(), padding=1)
    assert float((ref.double().cpu() - ok).norm() / ok.norm()) < 1e-6

    class Sub(torch.Tensor):
        pass

    side = torch.cuda.Stream()
    for args, kw in (((d, x, w, b, y, ws), {}), ((d,), dict(x=x, w=w, bias=b, y=y, ws=ws)), ((d, x.as_subclass(Sub), w, b, y, ws), {}),
                     ((d, torch.nn.Parameter(x), w, b, y, ws.double()), {}), ((d, x, w, b, y, ws), dict(stream=torch.cuda.current_stream())),
                     ((d, x, w, b, y, ws, torch.cuda.current_stream().cuda_stream), {}), ((d, x, w, b, y, ws, side), {})):
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        conv.conv_forward(*args, **kw)
        torch.cuda.synchronize()
        assert torch.equal(y, ref), (len(args), list(kw))
    with torch.cuda.stream(side):
        assert binding._stream(None) == side.cuda_stream
        y.fill_(float("nan"))
        conv.conv_forward(d, x, w, b, y, ws)  # behind the fill on the same stream
    side.synchronize()
    assert torch.equal(y, ref)
    y.fill_(7.0)
    for bad, error in (((x.double(), w, b), TypeError), ((x.cpu(), w, b), TypeError), ((x[:1], w, b), ValueError),
                       ((x.transpose(2, 3), w, b), TypeError), ((x, w.reshape(-1), b), ValueError), ((x, w, None), conv.ConvError),
                       ((x, "w", b), TypeError), ((x.to("meta"), w, b), TypeError)):
        with pytest.raises(error):
            conv.conv_forward(d, *bad, y, ws)
    with pytest.raises(conv.ConvError) as e:
        conv.conv_forward(d, x, w, b, y, torch.empty(0, device=DEV))
    assert e.value.status == binding.CONV_EWORKSPACE
    with pytest.raises(Exception):  # a transform's tensors have no storage
        torch.vmap(lambda v: conv.conv_forward(d, v, w, b, y, ws))(x[None])
    with pytest.raises(conv.ConvError):
        conv.conv_backward_filter(d, x, y, w.clone(), 0.5, ws)
    with pytest.raises((TypeError, ValueError)):
        conv.conv_backward_filter(d, x, y, w.clone(), "one", ws)
    dw = w.clone()
    conv.conv_backward_filter(d, x, ref, dw, ctypes.c_float(1.0).value, ws)
    torch.cuda.synchronize()
    assert (y == 7.0).all()


@pytest.mark.gpu
def test_every_call_through_both_ways():
    """Each compute call once with plain tensors and once with a subclass of one (the Python checks): the same bits."""

    class Sub(torch.Tensor):
        pass

    def both(fn, ins, outs, *rest):
        got = []
        for wrap in (lambda t: t, lambda t: t.as_subclass(Sub)):
            for o in outs:
                o.fill_(3)
            fn(*[wrap(a) if i == 0 and isinstance(a, torch.Tensor) else a for i, a in enumerate(ins)], *outs, *rest)
            torch.cuda.synchronize()
            got.append([o.clone() for o in outs])
        assert all(torch.equal(a, b) for a, b in zip(*got)), fn

    d, x, w, b, y, ws = layer()
    for dt, sfx in ((torch.float32, ""), (torch.float64, "_f64")):
        x, w, b, y = (t.to(dt) for t in (x, w, b, y))
        dy = torch.randn_like(y.nan_to_num())
        size = conv.conv_desc_workspace_bytes_f64(d) if sfx else conv.conv_desc_workspace_bytes(d)
        ws = torch.empty(size // 8 + 1, device=DEV, dtype=torch.float64)
        both(lambda v, *a: getattr(conv, "conv_forward" + sfx)(d, v, *a), (x, w, b), [y], ws)
        both(lambda v, *a: getattr(conv, "conv_backward_data" + sfx)(d, v, *a), (w, dy), [torch.empty_like(x)], ws)
        both(lambda v, *a: getattr(conv, "conv_backward_filter" + sfx)(d, v, *a), (x, dy), [torch.empty_like(w)], 0.0, ws)
        both(lambda v, *a: getattr(conv, "conv_backward_bias" + sfx)(d, v, *a), (dy,), [torch.empty_like(b)], 0, ws)
        if not sfx:
            both(lambda v, *a: conv.conv_backward_filter_bias(d, v, *a), (x, dy), [torch.empty_like(w), torch.empty_like(b)], 0.0, ws)
    m, k, o = 6, 70, 33
    p = conv.ip_desc_create(conv.IpParams(m, k, o, relu=1))
    x, w, b, dy = (torch.randn(s, device=DEV) for s in ((m, k), (o, k), (o,), (m, o)))
    ws = torch.empty(conv.ip_desc_workspace_bytes(p) // 4 + 1, device=DEV)
    both(lambda v, *a: conv.ip_forward(p, v, *a), (x, w, b), [torch.empty_like(dy)], ws)
    both(lambda v, *a: conv.ip_relu_backward(p, v, *a), (dy.abs(), dy), [torch.empty_like(dy)])
    both(lambda v, *a: conv.ip_backward_data(p, v, *a), (w, dy), [torch.empty_like(x)], ws)
    both(lambda v, *a: conv.ip_backward_filter(p, v, *a), (x, dy), [torch.empty_like(w)], 0.0, ws)
    both(lambda v, *a: conv.ip_backward_bias(p, v, *a), (dy,), [torch.empty_like(b)], 0.0, ws)
    aprob, rnd, reward = (torch.rand(50, device=DEV) for _ in range(3))
    action = torch.randint(0, 2, (50,), device=DEV, dtype=torch.int32)
    offsets = torch.tensor([0, 20, 50], device=DEV, dtype=torch.int32)
    logits = torch.randn(50, 6, device=DEV)
    both(conv.pg_sigmoid_sample_action, (aprob, rnd), [torch.empty_like(action)])
    both(lambda v, *a: conv.pg_discount_rewards(v, offsets, 0.9, *a), (reward,), [torch.empty_like(reward)])
    both(conv.pg_sigmoid_bottom_diff, (aprob, action, reward), [torch.empty_like(reward), torch.empty_like(reward)])
    both(conv.pg_softmax_bottom_diff, (logits, action, reward), [torch.empty_like(logits), torch.empty_like(logits)])
