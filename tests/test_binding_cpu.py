"""The binding's checks of tensor operands, with stub tensors that answer like
device tensors and a stub library that records the call: operands of the right
size, type and device reach the C function in its argument order; one operand
wrong in one property raises ValueError before any call."""
import inspect

import pytest
import torch

import paper_2204_01701_amd as ql

DESCS = [ql.conv_desc(2, 16, 9, 8, 24, 3, 3, (2, 1), 1), ql.conv_desc(1, 3, 5, 5, 7, 1, 5, 3, (0, 2), ql.QL_F32),
         ql.conv_desc(2, 12, 7, 7, 12, 3, 3, 1, 1, ql.QL_F32, groups=12), ql.conv_desc(4, 1, 6, 6, 1, 3, 3, groups=1)]
CONV = ql.conv_desc(2, 16, 9, 8, 24, 3, 3, (2, 1), 1)
CONV_T2 = ql.conv_desc(2, 16, 9, 8, 24, 3, 3, (2, 1), 1, ql.QL_F32, ql.QL_NEURON_T2)
LINEAR = ql.linear_desc(5, 7, 9)
LINEAR_F32 = ql.linear_desc(5, 7, 9, ql.QL_F32)
CALLS = [(n, d) for n in ("conv2d_fwd", "conv2d_fwd_ex", "conv2d_bwd_data", "conv2d_bwd_data_ex", "conv2d_bwd_weight",
                          "conv2d_bwd_weight_noalloc", "conv2d_bwd_relu") for d in (CONV, CONV_T2)]
CALLS += [(n, d) for n in ("linear_fwd", "linear_fwd_ex", "linear_bwd", "linear_bwd_relu") for d in (LINEAR, LINEAR_F32)]
ids = [f"{n}-{'f32' if d.dtype == ql.QL_F32 else 'bf16'}" for n, d in CALLS]


class Stub:
    """A device tensor as far as the binding looks at one."""

    def __init__(self, ptr, count, dtype, index=0, contiguous=True):
        self.ptr, self.count, self.dtype, self.contiguous = ptr, count, dtype, contiguous
        self.is_cuda = index >= 0
        self.device = torch.device("cuda", index) if index >= 0 else torch.device("cpu")

    def numel(self):
        return self.count

    def is_contiguous(self):
        return self.contiguous

    def get_device(self):
        return self.device.index if self.is_cuda else -1

    def data_ptr(self):
        return self.ptr


def sizes(d):
    """Elements of X, a weight, an output-side map, a bias: from the shapes."""
    if isinstance(d, ql.LinearDesc):
        return d.batch * d.in_, d.out * d.in_, d.batch * d.out, d.out
    cw = 1 if d.groups == d.c and d.c > 1 else d.c
    return d.n * d.h * d.w * d.c, d.o * d.kh * d.kw * cw, d.n * d.ho * d.wo * d.o, d.o


def operands(name, d):
    """Argument name -> (element count, dtype) of the entry point's tensors, as the header lists them."""
    nx, nw, ny, no = sizes(d)
    dt = torch.float32 if d.dtype == ql.QL_F32 else torch.bfloat16
    kinds = {}
    for p in inspect.signature(getattr(ql, "qlayer_" + name)).parameters:
        if p in ("x", "dx"):
            kinds[p] = nx, dt
        elif p in ("y", "gy", "y_out", "ta", "tb"):
            kinds[p] = ny, dt
        elif p in ("wa", "wb", "wc"):
            kinds[p] = nw, dt
        elif p in ("dwa", "dwb", "dwc"):
            kinds[p] = nw, torch.float32
        elif p in ("ba", "bb", "bc", "dba", "dbb", "dbc"):
            kinds[p] = no, torch.float32
    if "bwd_data" in name and d.neuron == ql.QL_NEURON_T2:
        kinds["ta"] = nx, dt  # (T2's input gradient takes X there)
    return kinds


@pytest.fixture
def calls(monkeypatch):
    made = []

    class Lib:
        def __getattr__(self, f):
            return lambda *a: made.append((f, a)) or 0

    monkeypatch.setattr(ql, "lib", Lib)
    return made


def run(name, d, tensors, **kw):
    if "noalloc" not in name:
        kw.setdefault("workspace", (None, 0))
    getattr(ql, "qlayer_" + name)(d, **tensors, stream=77, **kw)


def good(name, d):
    return {n: Stub(4096 * (i + 1), c, t) for i, (n, (c, t)) in enumerate(operands(name, d).items())}


@pytest.mark.parametrize("d", DESCS + [LINEAR], ids=range(len(DESCS) + 1))
def test_sizes(d):
    needs = (ql._linear_needs if isinstance(d, ql.LinearDesc) else ql._conv_needs)(d)
    dt = torch.float32 if d.dtype == ql.QL_F32 else torch.bfloat16
    assert tuple(needs[r][0] for r in "xwyb") == sizes(d)
    assert [needs[r][1] for r in "xwytbg"] == [dt] * 4 + [torch.float32] * 2


@pytest.mark.parametrize("name,d", CALLS, ids=ids)
def test_right_operands_reach_the_call_in_order(name, d, calls):
    tensors = good(name, d)
    assert ql._pointers((ql._linear_needs if isinstance(d, ql.LinearDesc) else ql._conv_needs)(d),
                        ql._OPERANDS["qlayer_" + name][1], tuple(tensors.values())) is not None  # (in one pass)
    ptrs = [t.ptr for t in tensors.values()]
    run(name, d, tensors)
    # raw pointers, all or in part, pass unchecked
    run(name, d, {n: t.ptr for n, t in tensors.items()})
    run(name, d, {n: t.ptr if i % 2 else t for i, (n, t) in enumerate(tensors.items())})
    run(name, d, {n: None for n in tensors})
    for i, (f, a) in enumerate(calls):
        assert f == "qlayer_" + name
        assert list(a[1:1 + len(ptrs)]) == (ptrs if i < 3 else [None] * len(ptrs))
        assert a[-1] == 77 and ("noalloc" in name or a[-3:-1] == (None, 0))
    assert len(calls) == 4


@pytest.mark.parametrize("name,d", CALLS, ids=ids)
def test_one_wrong_operand_raises_before_the_call(name, d, calls):
    for arg, (count, dt) in operands(name, d).items():
        for wrong, match in ((Stub(64, count + 1, dt), "elements"), (Stub(64, count - 1, dt), "elements"),
                             (Stub(64, count, torch.float16), "dtype"), (Stub(64, count, dt, 1), "on cuda"),
                             (Stub(64, count, dt, -1), "CUDA device|on cpu"),
                             (Stub(64, count, dt, contiguous=False), "contiguous")):
            tensors = good(name, d)
            tensors[arg] = wrong
            with pytest.raises(ValueError, match=match):
                run(name, d, tensors)
    assert not calls


@pytest.mark.parametrize("name,d", [c for c in CALLS if c[0].endswith("_ex") and "fwd" in c[0]])
def test_epilogue_operands_are_checked(name, d, calls):
    no = sizes(d)[3]
    run(name, d, good(name, d), epi=ql.epilogue(*(Stub(64, no, torch.float32) for _ in range(2))))
    assert len(calls) == 1
    for bad in (Stub(64, no - 1, torch.float32), Stub(64, no, torch.bfloat16), Stub(64, no, torch.float32, 1)):
        for k in ("scale", "shift", "stat_sum", "stat_sumsq"):
            with pytest.raises(ValueError, match="epi"):
                run(name, d, good(name, d), epi=ql.epilogue(**{k: bad}))
    assert len(calls) == 1


def test_unknown_type_codes_are_left_to_the_library():
    d = ql.linear_desc(4, 8, 8, ql.QL_F32)
    d.dtype = 7
    assert ql._pointers(ql._linear_needs(d), ql._OPERANDS["qlayer_linear_fwd"][1], (Stub(64, 32, torch.float32),)) is None
    with pytest.raises(ql.QLError):
        ql.qlayer_linear_fwd(d, 4096, 4096, 4096, 4096, y=4096, ta=4096, tb=4096)
