"""The narrow-layer kernels (forward, input gradient, weight gradient: at
most 16 output or input channels and a short reduction) against the fp64
oracle, with the paths on (the default for these shapes) and forced off
(the tiled kernels), fp32 and bf16: 16 channels at stride 1 and 2, 8
channels, the zero-padded 3-channel stem, a ragged last pixel block, a 1x1
filter, 16 -> 8 channels, O < 16, and the weight gradient of wider layers
(up to 64 channels) in 16-channel slices.  Normwise limits as in
test_gpu_parity."""
import pytest
import torch

import oracle
import paper_2204_01701_amd as ql
import synth

pytestmark = pytest.mark.gpu

import qlh  # noqa: E402

# (N, C, H, W, O, KH, KW, stride, pad)
SHAPES = [
    (4, 16, 12, 12, 16, 3, 3, 1, 1),    # a 16-channel CIFAR ResNet stage
    (3, 16, 11, 9, 16, 3, 3, 2, 1),     # stride 2, ragged last pixel block
    (2, 8, 10, 10, 8, 3, 3, 1, 1),      # 8 channels
    (5, 3, 9, 9, 16, 3, 3, 1, 1),       # the 3-channel stem (X zero-padded)
    (2, 16, 7, 7, 16, 1, 1, 1, 0),      # 1x1 filter
    (2, 16, 9, 9, 8, 3, 3, 1, 1),       # 16 -> 8 channels
    (1, 12, 6, 5, 12, 3, 3, 1, 1),      # 12 channels (fp32: narrow; bf16: off the vector width)
    (4, 3, 10, 10, 64, 3, 3, 1, 1),     # a 3 -> 64-channel stem: weight gradient in four 16-channel slices
    (2, 16, 9, 9, 32, 3, 3, 2, 1),      # 16 -> 32 at stride 2: two slices
    (3, 8, 7, 7, 48, 3, 3, 1, 1),       # three slices
]

KEYS_FWD = ("y", "ta", "tb")
KEYS_GRAD = ("dx", "dwa", "dwb", "dwc", "dba", "dbb", "dbc")
OFF = ("QLAYER_FWD_NARROW", "QLAYER_BWD_DATA_NARROW", "QLAYER_BWD_WEIGHT_NARROW")


@pytest.mark.parametrize("narrow", [True, False], ids=["narrow", "tiled"])
@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_narrow_paths_match_oracle(shape, bf16, narrow, monkeypatch):
    N, C, H, W, O, KH, KW, s, p = shape
    print(f"narrow={narrow} shape={shape} bf16={bf16}", flush=True)
    if not narrow:
        for k in OFF:
            monkeypatch.setenv(k, "0")
    else:
        monkeypatch.setenv("QLAYER_BWD_WEIGHT_NARROW_MAXO", "64")  # (16-channel slices in bf16 too)
    inp = synth.random_conv_case([800] + list(shape), N, C, H, W, O, KH, KW, s, p, bf16=bf16)
    got = qlh.conv_to_np(qlh.run_conv(inp, s, p, bf16))
    y, ta, tb = oracle.conv2d_fwd(inp["x"], inp["wa"], inp["wb"], inp["wc"], inp["ba"], inp["bb"], inp["bc"], s, p)
    ref = oracle.conv2d_bwd(inp["x"], inp["wa"], inp["wb"], inp["wc"], inp["ba"], inp["bb"], inp["bc"], inp["gy"], s, p)
    ref.update({"y": y, "ta": ta, "tb": tb})
    for k in KEYS_FWD + KEYS_GRAD:
        e = qlh.relerr(got[k], ref[k])
        assert e <= qlh.tol(bf16, k in KEYS_GRAD), f"{k}: normwise relative error {e:.3e}"


@pytest.mark.parametrize("shape", [(32, 16, 1024, 1024, 16, 1), (33, 8, 1024, 2048, 8, 2)],
                         ids=lambda s: "x".join(map(str, s)))
def test_maps_from_2_31_bytes_match_parts(shape):
    """The narrow kernels address maps below 2^31 bytes; a layer whose fp32 X is
    at or past that is launched in groups of images, and agrees with the same
    layer called on batches of a few images.  Either side is within the fp32
    limit of the exact result, so the two are within twice that."""
    n, c, h, w, o, s = shape
    dev, part = torch.device("cuda"), 8
    gen = torch.Generator(device=dev).manual_seed(9)
    r = lambda *sh: torch.randn(*sh, device=dev, generator=gen)  # noqa: E731
    x, ws, bs = r(n, h, w, c), [r(o, 3, 3, c) / (9 * c) ** 0.5 for _ in range(3)], [r(o) for _ in range(3)]
    assert x.numel() * 4 >= 2 ** 31

    def run(x):
        d = ql.conv_desc(x.shape[0], c, h, w, o, 3, 3, s, 1, ql.QL_F32)
        maps = [torch.empty(x.shape[0], d.ho, d.wo, o, device=dev) for _ in range(3)]
        dx, dw, db = torch.empty_like(x), [torch.empty_like(v) for v in ws], [torch.empty_like(b) for b in bs]
        ql.qlayer_conv2d_fwd(d, x, *ws, *bs, *maps)
        ql.qlayer_conv2d_bwd_data(d, maps[0], maps[1], maps[2], *ws, dx)
        ql.qlayer_conv2d_bwd_weight(d, x, maps[0], maps[1], maps[2], *dw, *db)
        return maps + [dx], dw + db

    whole, grads = run(x)
    total = None
    for i in range(0, n, part):
        got, gi = run(x[i:i + part])
        for k, (a, b) in enumerate(zip(whole, got)):
            a = a[i:i + part]
            assert float((a - b).norm() / b.norm()) <= 2 * qlh.tol(False, k == 3), (i, k)
        total = [v.double() for v in gi] if total is None else [t + v for t, v in zip(total, gi)]
    for k, (a, b) in enumerate(zip(grads, total)):
        assert float((a - b).norm() / b.norm()) <= 2 * qlh.tol(False, True), k


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape", [(5, 16, 12, 12, 16, 3, 1), (7, 16, 11, 9, 8, 3, 2), (4, 3, 9, 9, 16, 3, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_groups_of_images_match_oracle(shape, bf16, monkeypatch):
    """A layer launched in groups of two images (the limit in bytes lowered to
    that), the last group smaller, with the forward's fused epilogue and sums."""
    n, c, h, w, o, k, s = shape
    print(f"narrow groups {shape} bf16={bf16}", flush=True)
    cp = -(-c // 8) * 8 if bf16 else -(-c // 4) * 4
    ho, wo = (h + 2 - k) // s + 1, (w + 2 - k) // s + 1
    image = max(h * w * cp, ho * wo * o) * (2 if bf16 else 4)
    monkeypatch.setenv("QLAYER_NARROW_BYTES", str(2 * image + image // 2))
    inp = synth.random_conv_case([820] + list(shape), n, c, h, w, o, k, k, s, 1, bf16=bf16)
    got = qlh.conv_to_np(qlh.run_conv(inp, s, 1, bf16))
    y, ta, tb = oracle.conv2d_fwd(*(inp[v] for v in ("x", "wa", "wb", "wc", "ba", "bb", "bc")), s, 1)
    ref = oracle.conv2d_bwd(*(inp[v] for v in ("x", "wa", "wb", "wc", "ba", "bb", "bc", "gy")), s, 1)
    ref.update({"y": y, "ta": ta, "tb": tb})
    for key in KEYS_FWD + KEYS_GRAD:
        e = qlh.relerr(got[key], ref[key])
        assert e <= qlh.tol(bf16, key in KEYS_GRAD), f"{key}: normwise relative error {e:.3e}"
    d = ql.conv_desc(n, c, h, w, o, k, k, s, 1, qlh.qdtype(bf16))
    out = torch.full((n, ho, wo, o), float("nan"), device=qlh.DEV, dtype=qlh.tdtype(bf16))
    s1, s2 = (torch.full((o,), float("nan"), device=qlh.DEV) for _ in range(2))
    ql.qlayer_conv2d_fwd_ex(d, qlh.nchw_to_dev(inp["x"], bf16), *(qlh.oihw_to_dev(inp[v], bf16) for v in ("wa", "wb", "wc")),
                            *(qlh.vec_to_dev(inp[v]) for v in ("ba", "bb", "bc")), out,
                            epi=ql.epilogue(relu=True, stat_sum=s1, stat_sumsq=s2))
    torch.cuda.synchronize()
    assert qlh.relerr(qlh.nhwc_to_np(out), y.clip(min=0)) <= qlh.tol(bf16, False)
    v = out.double().reshape(-1, o)
    u = v.shape[0] * 2.0 ** -24  # an fp32 sum of that many rows
    assert torch.all((s1.double() - v.sum(0)).abs() <= u * v.abs().sum(0))
    assert torch.all((s2.double() - (v * v).sum(0)).abs() <= 2 * u * (v * v).sum(0))
