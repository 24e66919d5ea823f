"""The input gradient at stride > 1, computed phase by phase (each input pixel
meets only the taps of its stride offset): maps that the strides do not
divide, strides that differ, phases without taps (a filter smaller than the
stride) or without pixels (a map smaller than it), split-K, the narrow kernel
(C <= 16), padded channels, strides with more phases than the narrow kernel's
arguments list, and one with too many, the tiles with channel-aligned steps,
against the fp64 oracle element by element."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

import qlh  # noqa: E402
import paper_2204_01701_amd as ql  # noqa: E402
from test_gpu_neurons import NAMES, T2, T24, T3, T4, TERMS, _run_conv_neuron  # noqa: E402

# N, C, H, W, O, K, stride, pad
SHAPES = [
    (2, 24, 11, 8, 32, 3, (2, 2), 1),     # odd height
    (3, 72, 7, 10, 40, 3, (2, 1), 1),     # strides that differ; O off the K step
    (2, 32, 9, 7, 64, 5, (3, 2), 2),
    (2, 16, 12, 11, 16, 3, (2, 2), 1),    # narrow
    (2, 12, 9, 9, 24, 2, (3, 3), 0),      # narrow; phases without taps
    (2, 40, 10, 10, 32, 1, (2, 2), 0),    # three of four phases without taps
    (1, 8, 1, 6, 32, 3, (2, 2), 1),       # phases without pixels
    (4, 256, 5, 5, 256, 3, (2, 2), 1),    # split-K
    (16, 20, 9, 9, 30, 3, (2, 2), 1),     # O off the vector: padded copies
    (1, 16, 20, 20, 16, 9, (9, 9), 0),    # narrow, 81 phases, 25 pixels each or fewer
    (8, 16, 45, 38, 32, 9, (10, 9), 3),   # narrow, 90 phases, some without taps
    (3, 40, 33, 20, 48, 10, (10, 10), 1), # tiles, 100 phases
    (1, 72, 12, 30, 64, 5, (5, 17), 2),   # tiles, 85 phases, most without taps or with few pixels
    (1, 24, 70, 70, 30, 1, (70, 70), 0),  # a filter much smaller than the stride: the register-staged kernel
]


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_strided_input_gradient_matches_oracle(shape, bf16):
    N, C, H, W, O, K, s, p = shape
    print(f"strided input gradient {shape} bf16={bf16}", flush=True)
    ho, wo = (H + 2 * p - K) // s[0] + 1, (W + 2 * p - K) // s[1] + 1
    inp = synth.random_conv_case([980, N, C, H, W, O, K, *s, p], N, C, H, W, O, K, K, 1, p, bf16=bf16)
    rng = np.random.default_rng([981, H, W, *s])
    maps = {k: rng.standard_normal((N, O, ho, wo), dtype=np.float32) for k in ("gy", "ta", "tb")}
    if bf16:
        maps = {k: synth.round_bf16(v) for k, v in maps.items()}
    d = ql.conv_desc(N, C, H, W, O, K, K, s, p, qlh.qdtype(bf16))
    w = [qlh.oihw_to_dev(inp[k], bf16) for k in ("wa", "wb", "wc")]
    m = {k: qlh.nchw_to_dev(v, bf16) for k, v in maps.items()}
    dx = torch.full((N, H, W, C), float("nan"), device=qlh.DEV, dtype=qlh.tdtype(bf16))
    ql.qlayer_conv2d_bwd_data(d, m["gy"], m["ta"], m["tb"], *w, dx)
    torch.cuda.synchronize()

    def grads(g, ta, tb, ws):  # dX = sum over terms of the transposed convolutions, in fp64
        gt = [torch.from_numpy(v.astype(np.float64)) for v in (g * tb.astype(np.float64), g * ta.astype(np.float64), g)]
        out = torch.zeros((N, C, H, W), dtype=torch.float64)
        for t in range(3):
            op = [(v + 2 * p - K) % st for v, st in ((H, s[0]), (W, s[1]))]
            out += torch.nn.functional.conv_transpose2d(gt[t], torch.from_numpy(ws[t].astype(np.float64)), stride=s,
                                                        padding=p, output_padding=op)
        return out.numpy()

    ws = [inp[k] for k in ("wa", "wb", "wc")]
    ref = grads(maps["gy"], maps["ta"], maps["tb"], ws)
    mag = grads(*(np.abs(maps[k]) for k in ("gy", "ta", "tb")), [np.abs(v) for v in ws])
    qlh.check_elementwise("dx", "dx", qlh.nhwc_to_np(dx), ref, mag, bf16, 3 * O * K * K)


# (C a multiple of 8, O of 32: K steps within one tap, scalar weight addresses)
ALIGNED = [
    (3, 136, 11, 8, 96, 3, (2, 2), 1),    # ragged maps and rows
    (2, 72, 9, 10, 64, 1, (2, 2), 0),     # three of four phases without taps
    (4, 256, 5, 5, 256, 3, (2, 2), 1),    # split-K
    (1, 104, 6, 13, 32, 3, (3, 2), 1),    # one step per tap; strides that differ
]


@pytest.mark.parametrize("cfg", [3, 2], ids=["tile128x128", "tile128x64"])
@pytest.mark.parametrize("shape", ALIGNED, ids=lambda s: "x".join(map(str, s)).replace(" ", ""))
def test_strided_channel_aligned_tiles_match_oracle(shape, cfg, monkeypatch):
    monkeypatch.setenv("QLAYER_BWD_DATA_CFG", str(cfg))
    monkeypatch.setenv("QLAYER_BWD_DATA_CA", "1")
    test_strided_input_gradient_matches_oracle(shape, True)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("C", [40, 136], ids=["64rows", "128rows"])  # (bf16: 128-row tiles with channel-aligned steps)
@pytest.mark.parametrize("neuron", [T4, T3, T2, T24], ids=lambda n: NAMES[n])
def test_strided_neuron_types_match_oracle(neuron, C, bf16):
    N, H, W, O, K, s, p = 2, 7, 9, 64, 3, 2, 1
    print(f"strided neuron {NAMES[neuron]} bf16={bf16}", flush=True)
    inp = synth.random_conv_case([982, neuron], N, C, H, W, O, K, K, s, p, bf16=bf16)
    nt = TERMS[neuron]
    w = [inp["wa"], inp["wb"] if nt >= 2 else None, inp["wc"] if nt >= 3 else None]
    b = [inp["ba"], inp["bb"] if nt >= 2 else None, inp["bc"] if nt >= 3 else None]
    ref = oracle.conv2d_bwd_neuron(neuron, inp["x"], *w, *b, inp["gy"], stride=s, pad=p)
    got = _run_conv_neuron(neuron, inp, s, p, bf16)
    e = qlh.relerr(got["dx"], ref["dx"])
    assert e <= qlh.tol(bf16, True), f"dx: normwise relative error {e:.3e}"
