"""The depthwise row kernels (a thread walks down a segment of rows), forced on
maps smaller than those they serve by default: column groups that end past the
map, segments of unequal length, maps shorter than the filter's reach, one to
64 channel lanes, several channel slices, stride 2 in the forward, no padding,
every neuron type, against the fp64 oracle element by element; and the default
route on a map large enough for them against the column kernels."""
import numpy as np
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


def _magnitudes(neuron, inp, w, b, s, p):
    """Sums of the magnitudes of the terms of Y, T_a, T_b and dX: the oracle on absolute values."""
    a = [np.abs(v) if v is not None else None for v in (*w, *b)]
    x, gy = np.abs(inp["x"]), np.abs(inp["gy"])
    return (*oracle.dwconv2d_fwd(neuron, x, *a, stride=s, pad=p), oracle.dwconv2d_bwd(neuron, x, *a, gy, stride=s, pad=p)["dx"])


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
    my, mta, mtb, mdx = _magnitudes(neuron, inp, w, b, s, p)
    for k, got, want, mag in (("y", y, ry, my), ("ta", ta, rta, mta), ("tb", tb, rtb, mtb), ("dx", dx, ref["dx"], mdx)):
        if got is not None:
            # (T2 sums products with X o X rounded to the type: the bound of products of rounded operands)
            kind = "dx" if k == "y" and neuron == T2 else k
            qlh.check_elementwise(k, kind, qlh.nhwc_to_np(got), want, mag, bf16, 9 * nt + 1)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape", [(2, 12, 31, 9, 1, 1), (1, 324, 6, 5, 1, 1), (2, 20, 30, 7, 2, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_row_forward_epilogue_matches_oracle(shape, bf16, monkeypatch):
    """Scale, shift and ReLU at the end of the row forward, which stores Y alone."""
    N, C, H, W, s, p = shape
    print(f"depthwise rows epilogue {shape} bf16={bf16}", flush=True)
    monkeypatch.setenv("QLAYER_DW_ROWS", "1")
    inp = synth.random_dwconv_case([991, N, C, H, W, s], N, C, H, W, 3, 3, s, p, bf16=bf16)
    d = ql.conv_desc(N, C, H, W, C, 3, 3, s, p, qlh.qdtype(bf16), groups=C)
    w, b = [inp[k] for k in ("wa", "wb", "wc")], [inp[k] for k in ("ba", "bb", "bc")]
    ry, _, _ = oracle.dwconv2d_fwd(QUADRA, inp["x"], *w, *b, stride=s, pad=p)
    rng = np.random.default_rng(992)
    scale, shift = (rng.standard_normal(C).astype(np.float32) for _ in range(2))
    want, _, _ = oracle.epilogue(ry, scale, shift, True)
    y = torch.full((N, d.ho, d.wo, C), float("nan"), device=DEV, dtype=qlh.tdtype(bf16))
    ql.qlayer_conv2d_fwd_ex(d, qlh.nchw_to_dev(inp["x"], bf16), *(qlh.oihw_to_dev(v, bf16) for v in w),
                            *(qlh.vec_to_dev(v) for v in b), y,
                            epi=ql.epilogue(qlh.vec_to_dev(scale), qlh.vec_to_dev(shift), True))
    torch.cuda.synchronize()
    # (the magnitude sum through the epilogue; ReLU makes no error larger)
    mag = _magnitudes(QUADRA, inp, w, b, s, p)[0]
    mag = mag * np.abs(scale)[None, :, None, None] + np.abs(shift)[None, :, None, None]
    qlh.check_elementwise("y", "y", qlh.nhwc_to_np(y), want, mag, bf16, 9 * 3 + 3)


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
    # the sums of the terms' magnitudes, by the column kernels on absolute values
    monkeypatch.setenv("QLAYER_DW_ROWS", "0")
    mag = [torch.empty_like(x) for _ in range(4)]
    wm, t = [v.abs() for v in w], out["0"]
    ql.qlayer_conv2d_fwd(d, x.abs(), *wm, *(v.abs() for v in b), *mag[:3])
    ql.qlayer_conv2d_bwd_data(d, gy.abs(), t[1].abs(), t[2].abs(), *wm, mag[3])
    torch.cuda.synchronize()
    # Every element: each side rounds its output once, by u relative, and accumulates
    # at most 28 terms in fp32 (Y a product of two such sums), twice that with slack.
    u = 2.0 ** -8 if bf16 else 2.0 ** -24  # (half a unit in the last of 8 or 24 bits)
    for k, a, c, m in zip(("y", "ta", "tb", "dx"), out["0"], out["-1"], mag):
        assert bool(torch.isfinite(c).all()), k
        bound = 1.01 * u * (a.double().abs() + c.double().abs()) + 2 * 4 * 28 * 2.0 ** -24 * m.double()
        worst = float(((a.double() - c.double()).abs() / bound.clamp(min=1e-30)).max())
        assert worst <= 1.0, f"{k}: largest difference {worst:.3f} times the bound"
