"""The native module of the device calls against the ctypes path beside it: the same results, the same
exceptions, and nothing called when an argument is not what it takes."""
import numpy as np
import pytest

import paper_2511_15369_amd as ip
from paper_2511_15369_amd import binding


def _module():
    ip.load()
    return pytest.importorskip("paper_2511_15369_amd._call")


def test_arguments_it_does_not_take_are_left_alone():
    """CPU tensors, other classes and wrong counts: None, and no call (there is no GPU here)."""
    import torch
    call = _module()
    call.bind(*[1] * 8, ip.SoftmaxParams, ip.GeluParams, ip.Dyadic)      # addresses no call may reach
    try:
        x, y = torch.zeros(8, dtype=torch.int32), torch.zeros(8, dtype=torch.uint8)
        sp, gp, dy = ip.SoftmaxParams(), ip.GeluParams(), ip.Dyadic()
        assert call.softmax_i32(x, None, 0, y, 2, 4, sp) is None
        assert call.softmax_i32_windowed(x, None, 0, x, 1, 1, y, 2, 4, sp) is None
        assert call.softmax_i32_windowed_bits(x, None, 0, x, 1, 1, y, 2, 4, sp) is None
        assert call.gelu_i8(y.view(torch.int8), y.view(torch.int8), 8, gp) is None
        assert call.gelu_i32(x, y.view(torch.int8), 8, gp) is None
        assert call.requant(x, y, 8, 0, dy) is None
        assert call.softmax_i32_layers(x, 4, y, 4, 1, 4, 2, [sp, sp]) is None
        assert call.gelu_i8_layers(y.view(torch.int8), 4, y.view(torch.int8), 4, 4, 2, [gp, gp]) is None
        for args in ((), (1,), (None,) * 7, ("a",) * 4, (x, None, 0, y, 2 ** 70, 4, sp), (x, None, 0, y, 2, 4, gp)):
            assert call.softmax_i32(*args) is None
            assert call.gelu_i8(*args) is None
    finally:
        binding._forget_stream()                                  # bound again before the next device call
    with pytest.raises(TypeError):
        call.bind(1, 2, 3)


def test_the_library_builds_and_runs_without_it(monkeypatch, tmp_path, capfd):
    """Where torch's headers are missing the build says so and goes on, and takes an older module away;
    where the module cannot be loaded the binding says so and takes the ctypes path."""
    import sys
    from torch.utils import cpp_extension
    from paper_2511_15369_amd import build
    older = tmp_path / "_call.so"
    older.write_bytes(b"older")
    with monkeypatch.context() as m:
        m.setattr(build, "CALL_MODULE", str(older))
        m.setattr(cpp_extension, "include_paths", lambda *a, **k: [])
        assert build.build_call_module() == ""
        assert "_call.so was not built" in capfd.readouterr().err and not list(tmp_path.iterdir())
        m.setattr(build.subprocess, "check_call", lambda *a, **k: (_ for _ in ()).throw(FileNotFoundError("g++")))
        assert build.build_call_module() == "" and "g++" in capfd.readouterr().err
    ip.load()
    with monkeypatch.context() as m:
        m.setitem(sys.modules, "paper_2511_15369_amd._call", None)
        m.delattr(sys.modules["paper_2511_15369_amd"], "_call", raising=False)
        m.setattr(binding, "_fast", None)
        with pytest.warns(RuntimeWarning, match="ctypes"):
            binding._bind_calls()
        assert binding._fast is None


def _cases():
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    s = (torch.randn((2 * 4 * 49, 49), device="cuda", generator=g) * 900).to(torch.int32)
    x8 = torch.randint(-128, 128, (5000,), device="cuda", generator=g, dtype=torch.int8)
    acc = (torch.randn(5000, device="cuda", generator=g) * 30000).to(torch.int32)
    bias = (torch.randn((4 * 49, 49), device="cuda", generator=g) * 8).to(torch.int32)
    mask = torch.where(torch.rand((2, 49, 49), device="cuda", generator=g) < 0.3, -2 ** 31, 0).to(torch.int32)
    bits = torch.empty((2, 49, 1), dtype=torch.int64, device="cuda")
    ip.pack_window_mask(mask, 2, 49, bits)
    sp = ip.softmax_prepare(0.01, 49, 1, 0)
    g8, g32 = ip.gelu_prepare(0.02, 0.02, 0, 0, 1, 255), ip.gelu_prepare(0.02, 0.02, 0, 0, 1, 127)
    g32.pre_m, g32.pre_s = 20000, 24
    rows = s.shape[0]

    def out(n, dtype):
        return torch.zeros(n, dtype=dtype, device="cuda")

    return {
        "softmax_i32": lambda y=None: (s, bias, 196, out(s.numel(), torch.uint8), rows, 49, sp),
        "softmax_i32_windowed": lambda: (s, bias, 196, mask, 2, 4, out(s.numel(), torch.uint8), rows, 49, sp),
        "softmax_i32_windowed_bits": lambda: (s, bias, 196, bits, 2, 4, out(s.numel(), torch.uint8), rows, 49, sp),
        "gelu_i8": lambda: (x8, out(5000, torch.int8), 5000, g8),
        "gelu_i32": lambda: (acc, out(5000, torch.int8), 5000, g32),
        "requant": lambda: (acc, out(5000, torch.int8), 5000, 1, ip.Dyadic(20480, 25, 0, -128, 127)),
        "softmax_i32_layers": lambda: (s, 49 * 100, out(s.numel(), torch.uint8), 49 * 100, 100, 49, 3, [sp] * 3),
        "gelu_i8_layers": lambda: (x8, 1000, out(5000, torch.int8), 1000, 1000, 5, [g8] * 5),
    }


NAMES = ["softmax_i32", "softmax_i32_windowed", "softmax_i32_windowed_bits", "gelu_i8", "gelu_i32", "requant",
         "softmax_i32_layers", "gelu_i8_layers"]
OUT_AT = dict(softmax_i32=3, softmax_i32_windowed=6, softmax_i32_windowed_bits=6, gelu_i8=1, gelu_i32=1, requant=1,
              softmax_i32_layers=2, gelu_i8_layers=2)


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_the_two_paths_agree(name, monkeypatch):
    import torch
    make, fn, at = _cases()[name], getattr(ip, name), OUT_AT[name]
    assert binding._fast is not None                              # the first device call brought it up
    native = make()
    assert getattr(binding._fast, name)(*native) == 0             # taken, not left to the long way
    with monkeypatch.context() as m:
        m.setattr(binding, "_fast", None)
        long_way = make()
        assert fn(*long_way) is None
    torch.cuda.synchronize()
    assert torch.equal(native[at], long_way[at])
    assert int(long_way[at].ne(0).sum()) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
@pytest.mark.parametrize("native", [True, False])
def test_calls_go_to_the_current_stream(name, native, monkeypatch):
    """The input arrives late, on a side stream: a call that ran on any other stream would have read what
    was there before it (and its output is not the one of the input that arrives)."""
    import torch
    make, at = _cases()[name], OUT_AT[name]
    fn = getattr(binding._fast, name) if native else getattr(ip, name)
    if not native:
        monkeypatch.setattr(binding, "_fast", None)
    want, early, late = make(), list(make()), list(make())
    fn(*want)
    early[0] = torch.zeros_like(want[0])
    fn(*early)
    late[0] = torch.zeros_like(want[0])
    torch.cuda.synchronize()
    assert not torch.equal(early[at], want[at])
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        late[0].copy_(want[0])
        assert fn(*late) in (0, None)
    torch.cuda.default_stream().synchronize()
    side.synchronize()
    assert torch.equal(late[at], want[at])


@pytest.mark.gpu
@pytest.mark.parametrize("name", NAMES)
def test_the_two_paths_raise_alike(name, monkeypatch):
    import torch

    class Sub(torch.Tensor):
        pass

    make, fn, at = _cases()[name], getattr(ip, name), OUT_AT[name]
    bad = []
    for i, a in enumerate(make()):
        if isinstance(a, torch.Tensor):
            bad += [(i, a.cpu()), (i, a.reshape(-1)[:3]), (i, a.double()), (i, a.reshape(-1)[::2]), (i, "no tensor")]
            bad += [(i, a.as_subclass(Sub))]                      # accepted, the long way
        elif isinstance(a, int):
            bad += [(i, -1), (i, np.int64(a)), (i, 1.5), (i, None), (i, 2 ** 40)]
        elif isinstance(a, list):
            bad += [(i, a[:-1]), (i, [ip.Dyadic()] * len(a)), (i, tuple(a))]
        else:
            bad += [(i, ip.Metric()), (i, None), (i, type(a)())]  # the last: zeros, outside the domain

    def outcome(i, v):
        args = list(make())
        args[i] = v if i != at or not isinstance(v, torch.Tensor) else v.clone()
        try:
            r = fn(*args)
            torch.cuda.synchronize()
            return r, args[at].clone()
        except Exception as e:
            return type(e), str(e)

    for i, v in bad:
        got = outcome(i, v)
        with monkeypatch.context() as m:
            m.setattr(binding, "_fast", None)
            want = outcome(i, v)
        assert got[0] == want[0], (i, v, got, want)
        if isinstance(want[1], torch.Tensor):
            assert torch.equal(got[1], want[1]), (i, v)
