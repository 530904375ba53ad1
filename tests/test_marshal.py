"""The native argument marshalling of the binding: arguments of plain form reach the library as they
are, everything else is left to the general path (None, nothing called)."""
import ctypes as C

import pytest
import torch

from paper_1908_05033_amd import binding as B

vp, sz, i, f = C.c_void_p, C.c_size_t, C.c_int, C.c_float
desc_p = C.POINTER(B.dsq_conv_desc)
SIGNATURES = [
    ("quantize_act", [vp, i, i, i, i, i, f, f, i, vp, sz, vp, vp]),
    ("conv2d", [desc_p, vp, vp, f, f, vp, vp, vp, i, vp, vp]),
    ("conv2d_requant", [desc_p, vp, vp, f, f, vp, vp, vp, vp, i, f, f, i, vp, sz, vp, vp]),
    ("conv2d_wq", [desc_p, vp, i, vp, vp, vp, i, vp]),
    ("soft_quantize_fwd", [vp, sz, f, f, f, i, vp, vp]),
    ("soft_quantize_bwd", [vp, vp, sz, f, f, f, i, vp, vp, vp]),
]


@pytest.fixture
def recorded():
    """The module bound to functions that note their arguments and return 7."""
    module, calls, keep = B.load_marshal(), [], []
    for name, args in SIGNATURES:
        def note(*a, _name=name):
            calls.append((_name, [[getattr(x.contents, n) for n, _ in B.dsq_conv_desc._fields_] if isinstance(x, desc_p) else x for x in a]))
            return 7
        keep.append(C.CFUNCTYPE(i, *args)(note))
    module.init(B.dsq_conv_desc, *(C.cast(k, vp).value for k in keep))
    try:
        yield module, calls
    finally:
        B._marshal = None
        B.load_marshal()


DESC = (2, 64, 9, 8, 32, 3, 3, 1, 1, 4, 16)


def test_plain_arguments_arrive(recorded):
    m, calls = recorded
    d = B.make_desc(*DESC)
    big = (1 << 63) + 64                                     # an address above the signed range
    assert m.conv2d(d, big, 0x20, -0.5, 2, 0x30, 0x40, 0x50, 1, None, 0x60) == 7
    assert calls.pop() == ("conv2d", [list(DESC), big, 0x20, -0.5, 2.0, 0x30, 0x40, 0x50, 1, None, 0x60])
    assert m.conv2d(d, 1, 2, 0.0, 1.0, 3, 4, 5, False, 6, 0) == 7
    assert calls.pop() == ("conv2d", [list(DESC), 1, 2, 0.0, 1.0, 3, 4, 5, 0, 6, None])
    assert m.conv2d_wq(d, 1, 0, 2, 3, 4, 1, 5) == 7
    assert calls.pop() == ("conv2d_wq", [list(DESC), 1, 0, 2, 3, 4, 1, 5])
    assert not calls


def test_other_forms_are_left_alone(recorded):
    m, calls = recorded
    d = B.make_desc(*DESC)
    good = [d, 1, 2, 0.0, 1.0, 3, 4, 5, 0, None, 6]

    class Number(int):
        pass

    cpu = torch.zeros(8, dtype=torch.uint8)
    bad = [(0, None), (0, object()), (0, B), (1, None), (1, cpu), (1, 1.0), (1, "x"), (1, 1 << 70), (3, "x"), (3, None), (3, torch.tensor(1.0)),
           (8, 1.0), (8, 1 << 40), (8, Number(1)), (9, 2.0), (10, object()), (10, torch.zeros(1))]
    for at, value in bad:
        args = list(good)
        args[at] = value
        assert m.conv2d(*args) is None, (at, value)
    assert m.conv2d(*good[:-1]) is None and m.conv2d(*good, None) is None
    # a byte count is asked of the codes: an address does not do
    assert m.quantize_act(1, 0, 1, 64, 2, 2, 0.0, 1.0, 4, 2, 3, 4) is None
    assert m.soft_quantize_fwd(1, 0.0, 1.0, 0.2, 2, 3, 4) is None
    with torch.overrides.TorchFunctionMode():
        assert m.conv2d(*good) is None
    assert not calls
    assert m.conv2d(*good) == 7


def test_module_that_does_not_load(monkeypatch):
    """Without the module (missing, or built for another PyTorch) the calls work through ctypes, with one warning."""
    import sys
    import warnings
    import paper_1908_05033_amd as package
    monkeypatch.setattr(B, "_marshal", None)
    monkeypatch.delattr(package, "_marshal", raising=False)
    monkeypatch.setitem(sys.modules, "paper_1908_05033_amd._marshal", None)          # its import raises ImportError
    # (no codes, no descriptor: refused before anything is launched)
    calls = [lambda: B.dsq_quantize_act(64, 0, 0, 64, 2, 2, 0.0, 1.0, 4, None, 64, 0),
             lambda: B.dsq_conv2d(None, 64, 64, 0.0, 1.0, 64, 64, 64, 0, None, 0),
             lambda: B.dsq_conv2d_requant(None, 64, 64, 0.0, 1.0, 64, 64, None, None, True, 0.0, 1.0, 4, None, 64, 0),
             lambda: B.dsq_conv2d_wq(None, 64, 0, 64, 64, 64, 0, 0),
             lambda: B.dsq_soft_quantize_fwd(torch.zeros(0), 0.0, 1.0, 0.2, 2, None),
             lambda: B.dsq_soft_quantize_bwd(torch.zeros(0), None, 0.0, 1.0, 0.2, 2, None, None)]
    with pytest.warns(RuntimeWarning, match="_marshal"):
        with pytest.raises(B.DsqError):
            calls[0]()
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        for call in calls[1:4]:
            with pytest.raises(B.DsqError):
                call()
        for call in calls[4:]:
            with pytest.raises(TypeError):                   # (a host tensor: refused as ever)
                call()


@pytest.mark.gpu
def test_device_tensors_and_streams(recorded):
    m, calls = recorded
    x = torch.zeros(256, device="cuda")
    y = torch.nn.Parameter(torch.zeros(256, device="cuda"))
    assert m.soft_quantize_fwd(x, -1.0, 1.0, 0.2, 2, y, None) == 7
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        assert m.soft_quantize_fwd(y, -1.0, 1.0, 0.2, 2, x, None) == 7
    first, second = [c[1] for c in calls]
    assert first[0] == x.data_ptr() and first[1] == 256 and first[6] == y.data_ptr()
    assert (first[7] or 0) == torch.cuda.current_stream().cuda_stream
    assert second[0] == y.data_ptr() and second[6] == x.data_ptr() and second[7] == s.cuda_stream
    calls.clear()

    class Sub(torch.Tensor):
        pass

    for odd in (x.double(), x[::2], x.cpu(), x.as_subclass(Sub), torch.zeros(256, device="meta")):
        assert m.soft_quantize_fwd(odd, -1.0, 1.0, 0.2, 2, y, None) is None
    assert m.soft_quantize_fwd(x, -1.0, 1.0, 0.2, 2, y, s) is None          # (a Stream object: general path)

    def inner(row):
        assert m.soft_quantize_fwd(row, -1.0, 1.0, 0.2, 2, y, None) is None
        return row
    torch.func.vmap(inner)(torch.zeros(2, 256, device="cuda"))
    assert not calls


@pytest.mark.gpu
def test_both_paths_give_the_same_results(monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(2, 9, 8, 64, generator=g, device="cuda")
    out = []
    for native in (True, False):
        if not native:
            class General:
                def __getattr__(self, name):
                    return lambda *a: None
            monkeypatch.setattr(B, "_marshal", General())
        codes = torch.empty(B.dsq_act_packed_bytes(2, 9, 8, 64, 4), dtype=torch.uint8, device="cuda")
        sums = torch.empty(2 * 9 * 8, dtype=torch.int32, device="cuda")
        B.dsq_quantize_act(x, B.DSQ_NHWC, 2, 64, 9, 8, -1.0, 2.0, 4, codes, sums)
        y, gx, g3 = torch.empty_like(x), torch.empty_like(x), torch.empty(3, dtype=torch.float64, device="cuda")
        B.dsq_soft_quantize_fwd(x, -1.0, 1.0, 0.2, 2, y)
        B.dsq_soft_quantize_bwd(x, y, -1.0, 1.0, 0.2, 2, gx, g3, stream=torch.cuda.current_stream())
        out.append((codes, sums, y, gx))
        with pytest.raises(B.DsqError):
            B.dsq_quantize_act(x, B.DSQ_NHWC, 2, 64, 9, 8, 2.0, -1.0, 4, codes, sums)
        with pytest.raises(TypeError):
            B.dsq_quantize_act(x.double(), B.DSQ_NHWC, 2, 64, 9, 8, -1.0, 2.0, 4, codes, sums)
        with pytest.raises(B.DsqError):
            B.dsq_quantize_act(None, B.DSQ_NHWC, 2, 64, 9, 8, -1.0, 2.0, 4, codes, sums)
    for a, b in zip(*out):
        assert torch.equal(a, b)
