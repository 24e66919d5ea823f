"""Channel counts off the 16-byte vector (8 bf16 or 4 fp32 values): the passes
copy the tensors along those channels zero-padded to whole vectors and run the
pipelined kernels on the copies.  Odd and even counts (the copy loads one or
two bf16 values at a time), one of C and O on the vector and the other off
it, both off it, against the fp64 oracle; and the route the no-allocation
weight gradient takes where the copies do not fit its scratch array."""
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

import qlh  # noqa: E402
import paper_2204_01701_amd as ql  # noqa: E402
from test_gpu_neurons import NAMES, T2, T24, T3, T4, T4I, TERMS, _run_conv_neuron  # noqa: E402

# N, C, H, W, O, K, stride, pad
SHAPES = [
    (4, 17, 9, 7, 10, 3, 1, 1),     # odd C, narrow O
    (24, 9, 6, 5, 23, 3, 2, 1),     # odd O, stride 2
    (2, 60, 9, 9, 100, 3, 1, 1),    # even counts, several tiles
    (2, 60, 1, 1, 10, 1, 1, 0),     # too little work to pay for the copies: the register-staged kernels
    (4, 16, 7, 7, 130, 1, 1, 0),    # C on the vector, O past one 128-row tile
    (5, 131, 4, 4, 64, 3, 1, 1),    # O on the vector, few pixels: split-K
] + [(3, c, 6, 5, 24, 3, 1, 1) for c in (1, 2, 3, 5, 6, 7)]  # rows below one vector (fp32: up to 3)
CASES = [(0, s) for s in SHAPES] + [(n, (2, 33, 5, 6, 33, 3, 1, 1)) for n in (T4, T4I, T3, T2, T24)]


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("neuron,shape", CASES, ids=[f"{NAMES.get(n, 'quadra')}-{'x'.join(map(str, s))}" for n, s in CASES])
def test_channels_off_the_vector_match_oracle(neuron, shape, bf16):
    N, C, H, W, O, K, s, p = shape
    print(f"off-vector channels neuron {neuron} shape {shape} bf16={bf16}", flush=True)
    inp = synth.random_conv_case([970, neuron] + list(shape), N, C, H, W, O, K, K, s, p, bf16=bf16)
    nt = TERMS[neuron]
    w = [inp["wa"], inp["wb"] if nt >= 2 else None, inp["wc"] if nt >= 3 else None]
    b = [inp["ba"], inp["bb"] if nt >= 2 else None, inp["bc"] if nt >= 3 else None]
    y, ta, tb = oracle.conv2d_fwd_neuron(neuron, inp["x"], *w, *b, stride=s, pad=p)
    ref = oracle.conv2d_bwd_neuron(neuron, inp["x"], *w, *b, inp["gy"], stride=s, pad=p)
    ref["y"] = y
    if neuron != T2:
        ref["ta"] = ta
    if nt >= 2:
        ref["tb"] = tb
    got = _run_conv_neuron(neuron, inp, s, p, bf16)
    assert sorted(got) == sorted(ref)
    for k in ref:
        e = qlh.relerr(got[k], ref[k])
        assert e <= qlh.tol(bf16, k not in ("y", "ta", "tb")), f"{k}: normwise relative error {e:.3e}"


def test_noalloc_without_room_for_the_copies():
    """G, T_a, T_b padded from 36 to 40 channels alone exceed the scratch array:
    the no-allocation entry point takes the kernel that needs no copies."""
    N, C, HW, O = 48, 8, 64, 36
    assert 3 * N * HW * HW * 40 * 2 > ql.NOALLOC_SCRATCH_BYTES
    d = ql.conv_desc(N, C, HW, HW, O, 1, 1, 1, 0, ql.QL_BF16)
    g = torch.Generator(device=qlh.DEV).manual_seed(3)
    x = torch.randn((N, HW, HW, C), generator=g, device=qlh.DEV).bfloat16()
    gy, ta, tb = (torch.randn((N, HW, HW, O), generator=g, device=qlh.DEV).bfloat16() for _ in range(3))
    dw = [torch.empty((O, 1, 1, C), device=qlh.DEV) for _ in range(3)]
    db = [torch.empty(O, device=qlh.DEV) for _ in range(3)]
    ql.qlayer_conv2d_bwd_weight_noalloc(d, x, gy, ta, tb, *dw, *db)
    torch.cuda.synchronize()
    f = [t.double().reshape(-1, t.shape[-1]) for t in (x, gy, ta, tb)]
    for t, gt in enumerate((f[1] * f[3], f[1] * f[2], f[1])):
        assert qlh.relerr(dw[t].double().cpu().numpy().reshape(O, C), (gt.T @ f[0]).cpu().numpy()) <= qlh.tol(True, True)
        assert qlh.relerr(db[t].double().cpu().numpy(), gt.sum(0).cpu().numpy()) <= qlh.tol(True, True)
