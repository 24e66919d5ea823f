"""The depthwise row kernels (a thread walks down a segment of rows), forced on
maps smaller than those they serve by default: column groups that end past the
map, segments of unequal length, maps shorter than the filter's reach, one to
64 channel lanes, several channel slices, stride 2 in the forward, no padding,
every neuron type, against the fp64 oracle element by element; and the default
route on a map large enough for them against the column kernels."""
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

import qlh  # noqa: E402
import paper_2204_01701_amd as ql  # noqa: E402

DEV = qlh.DEV
QUADRA, T4, T4I, T3, T2 = range(5)
# N, C, H, W, stride, pad
SHAPES = [(2, 12, 31, 9, 1, 1), (1, 260, 5, 6, 1, 1), (3, 4, 29, 3, 1, 0), (2, 64, 1, 2, 1, 1), (2, 20, 30, 7, 2, 1),
          (1, 512, 4, 4, 1, 1)]
CASES = [(QUADRA, s) for s in SHAPES] + [(n, (2, 40, 17, 5, 1, 1)) for n in (T4, T4I, T3, T2)]


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("neuron,shape", CASES, ids=[f"n{n}-{'x'.join(map(str, s))}" for n, s in CASES])
def test_row_kernels_match_oracle(neuron, shape, bf16, monkeypatch):
    N, C, H, W, s, p = shape
    print(f"depthwise rows neuron {neuron} {shape} bf16={bf16}", flush=True)
    monkeypatch.setenv("QLAYER_DW_ROWS", "1")
    nt = ql.NEURON_TERMS[neuron]
    inp = synth.random_dwconv_case([990, neuron, N, C, H, W, s], N, C, H, W, 3, 3, s, p, bf16=bf16)
    d = ql.conv_desc(N, C, H, W, C, 3, 3, s, p, qlh.qdtype(bf16), neuron, groups=C)
    w = [inp[k] if i < nt else None for i, k in enumerate(("wa", "wb", "wc"))]
    b = [inp[k] if i < nt else None for i, k in enumerate(("ba", "bb", "bc"))]
    ry, rta, rtb = oracle.dwconv2d_fwd(neuron, inp["x"], *w, *b, stride=s, pad=p)
    ref = oracle.dwconv2d_bwd(neuron, inp["x"], *w, *b, inp["gy"], stride=s, pad=p)
    x, gy = qlh.nchw_to_dev(inp["x"], bf16), qlh.nchw_to_dev(inp["gy"], bf16)
    wd = [qlh.oihw_to_dev(v, bf16) if v is not None else None for v in w]
    y = torch.full((N, d.ho, d.wo, C), float("nan"), device=DEV, dtype=qlh.tdtype(bf16))
    ta = torch.full_like(y, float("nan")) if neuron != T2 else None
    tb = torch.full_like(y, float("nan")) if nt >= 2 else None
    dx = torch.full_like(x, float("nan"))
    ql.qlayer_conv2d_fwd(d, x, *wd, *(qlh.vec_to_dev(v) for v in b), y, ta, tb)
    ql.qlayer_conv2d_bwd_data(d, gy, x if neuron == T2 else ta, tb, *wd, dx)
    torch.cuda.synchronize()
    for k, got, want in (("y", y, ry), ("ta", ta, rta), ("tb", tb, rtb), ("dx", dx, ref["dx"])):
        if got is not None:
            e = qlh.relerr(qlh.nhwc_to_np(got), want)
            assert e <= qlh.tol(bf16, k == "dx"), f"{k}: normwise relative error {e:.3e}"


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
def test_default_route_on_a_large_map(bf16, monkeypatch):
    """Every output of a map that takes the row kernels, against the column
    kernels: the same sums of at most 27 products in another order."""
    N, C, HW = 64, 256, 56
    d = ql.conv_desc(N, C, HW, HW, C, 3, 3, 1, 1, qlh.qdtype(bf16), groups=C)
    g = torch.Generator(device=DEV).manual_seed(5)

    def rnd(*shape, dtype=qlh.tdtype(bf16)):
        return torch.randn(shape, generator=g, device=DEV).to(dtype)

    x, gy, w = rnd(N, HW, HW, C), rnd(N, HW, HW, C), [rnd(C, 3, 3, 1) for _ in range(3)]
    b = [rnd(C, dtype=torch.float32) for _ in range(3)]
    out = {}
    for rows in ("0", "-1"):
        monkeypatch.setenv("QLAYER_DW_ROWS", rows)
        m = [torch.full_like(x, float("nan")) for _ in range(4)]
        ql.qlayer_conv2d_fwd(d, x, *w, *b, *m[:3])
        t = out["0"] if rows == "-1" else m  # the same saved maps for both input gradients
        ql.qlayer_conv2d_bwd_data(d, gy, t[1], t[2], *w, m[3])
        out[rows] = m
    torch.cuda.synchronize()
    u = 2.0 ** -8 if bf16 else 2.0 ** -18  # one rounding of the output (bf16), 27 fp32 products and sums each side
    for a, c in zip(out["0"], out["-1"]):
        a, c = a.double(), c.double()
        assert torch.isfinite(c).all()
        assert float((a - c).norm() / a.norm()) <= u
