"""Which kernels a pass launches, where the choice is a rule on sizes whose wrong
side costs time only: the results are the same either way and are checked
against the oracle elsewhere."""
import pytest
import torch

import paper_2204_01701_amd as ql

pytestmark = pytest.mark.gpu

import qlh  # noqa: E402

MAPS = {ql.QL_NEURON_QUADRA: 2, ql.QL_NEURON_T3: 1, ql.QL_NEURON_T2: 0}


def launches(shape, dtype, neuron=ql.QL_NEURON_QUADRA, groups=1, passes=("fwd", "bwd_data", "bwd_weight")):
    """pass -> names of the kernels it launches."""
    n, c, hw, o, k, s = shape
    print(f"routes {shape} dtype={dtype} neuron={neuron} groups={groups}", flush=True)
    d = ql.conv_desc(n, c, hw, hw, o, k, k, s, k // 2, dtype, neuron, groups=groups)
    dt, nt = qlh.tdtype(dtype == ql.QL_BF16), ql.NEURON_TERMS[neuron]

    def new(*sh, dtype=dt):
        return torch.zeros(sh, device=qlh.DEV, dtype=dtype)

    def pad(v):
        return v + [None] * (3 - len(v))

    x, y, dx = new(n, hw, hw, c), new(n, d.ho, d.wo, o), new(n, hw, hw, c)
    w = pad([new(o, k, k, 1 if groups > 1 else c) for _ in range(nt)])
    g, ta, tb = [new(n, d.ho, d.wo, o) if i <= MAPS[neuron] else None for i in range(3)]
    dw = pad([new(*v.shape, dtype=torch.float32) for v in w if v is not None])
    f = {"fwd": lambda: ql.qlayer_conv2d_fwd(d, x, *w, None, None, None, y, ta, tb),
         "bwd_data": lambda: ql.qlayer_conv2d_bwd_data(d, g, x if neuron == ql.QL_NEURON_T2 else ta, tb, *w, dx),
         "bwd_weight": lambda: ql.qlayer_conv2d_bwd_weight(d, x, g, ta, tb, *dw)}
    out = {}
    for p in passes:
        f[p]()
        torch.cuda.synchronize()
        out[p] = qlh.kernel_names(f[p])
        if not out[p]:
            pytest.skip("the profiler records no device kernels on this runtime")
    return out


Q, T2 = ql.QL_NEURON_QUADRA, ql.QL_NEURON_T2
F32, BF16 = ql.QL_F32, ql.QL_BF16


@pytest.mark.parametrize("shape,dtype,neuron,padded", [
    # N, C, H = W, O, K, stride; the passes that copy their tensors padded to whole vectors
    ((8, 64, 6, 5, 3, 1), F32, Q, "bwd_data"),                 # fp32 weight gradient of little work
    ((64, 64, 28, 30, 3, 1), F32, Q, "bwd_data bwd_weight"),   # ... of much
    ((5, 7, 9, 140, 3, 1), F32, Q, "fwd"),                     # ... of few input channels
    ((4, 3, 9, 16, 3, 1), F32, Q, "fwd bwd_weight"),           # ... in the narrow kernel
    ((9, 32, 10, 9, 3, 1), F32, Q, "bwd_data"),                # ... in the narrow kernel, O off the vector
    ((227, 204, 60, 116, 1, 4), BF16, Q, "bwd_data"),          # a stride that skips most of X
    ((175, 25, 22, 6, 1, 1), BF16, Q, "bwd_data bwd_weight"),  # one K step onto few channels
    ((50, 60, 27, 100, 3, 1), BF16, Q, "fwd bwd_data bwd_weight"),
    ((1933, 308, 1, 10, 1, 1), F32, T2, ""),                   # one K step of one product
    ((34, 23, 13, 12, 1, 1), F32, T2, ""),
    ((316, 304, 1, 10, 1, 1), BF16, T2, "bwd_weight"),
    ((104, 48, 35, 14, 1, 2), F32, Q, "bwd_weight"),           # two K steps, large maps
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else None)
def test_passes_that_take_padded_copies(shape, dtype, neuron, padded):
    got = launches(shape, dtype, neuron)
    assert [p for p, names in got.items() if any("qconv_pad_" in n for n in names)] == padded.split()


@pytest.mark.parametrize("shape,dtype,neuron,groups,which,kernel", [
    # tiles: the template arguments after the type are rows, columns
    ((77, 400, 35, 4, 3, 1), F32, Q, 1, "bwd_data", "qconv_bwd_data_kernel<float, 128, 128"),   # many 32-row tiles
    ((32, 32, 16, 32, 3, 1), F32, Q, 1, "bwd_data", "qconv_bwd_data_kernel<float, 32, 128"),    # one, no empty rows
    ((209, 416, 2, 64, 5, 1), BF16, Q, 1, "bwd_data", "qconv_bwd_data_kernel<unsigned short, 128, 64"),  # four pixels
    ((12, 176, 22, 304, 3, 1), BF16, Q, 1, "bwd_weight", "qconv_bwd_weight16_kernel<"),  # too many steps for 64 x 64
    ((2, 256, 4, 256, 3, 1), BF16, Q, 1, "bwd_weight", "qconv_bwd_weight_kernel<64, 64"),
    ((3407, 16, 1, 848, 1, 1), F32, Q, 1, "fwd", "qconv_fwd_kernel<float, 64, 128"),     # one K step: the ramp decides
    ((2, 32, 49, 128, 1, 1), BF16, Q, 1, "fwd", "qconv_fwd_kernel<"),                    # nothing to split among waves
    ((911, 3488, 1, 320, 1, 1), BF16, Q, 1, "fwd", "qconv_fwd_kernel<"),                 # two rounds of long reductions
    ((3, 64, 8, 544, 5, 1), F32, Q, 1, "fwd", "qconv_fwd_ksplit_kernel<"),               # 102 workgroups
    ((3, 448, 9, 256, 3, 1), F32, Q, 1, "fwd", "qconv_fwd_kernel<"),                     # 64 workgroups
    # depthwise
    ((64, 256, 56, 256, 3, 1), BF16, Q, 256, "bwd_data", "qconv_dw_bwd_data_rows_kernel"),
    ((151, 352, 56, 352, 3, 1), BF16, T2, 352, "bwd_data", "qconv_dw_bwd_data_col_kernel"),
    ((151, 352, 56, 352, 3, 1), BF16, T2, 352, "fwd", "qconv_dw_fwd_col_kernel"),
    # 2^31 bytes of X: groups of images in the narrow kernels
    ((32, 16, 1024, 16, 3, 1), F32, Q, 1, "fwd", "qconv_fwd_narrow_kernel"),
    ((32, 16, 1024, 16, 3, 1), F32, Q, 1, "bwd_data", "qconv_bwd_data_narrow_kernel"),
    ((32, 16, 1024, 16, 3, 1), F32, Q, 1, "bwd_weight", "qconv_bwd_weight_narrow_kernel"),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else None)
def test_kernel_of_a_pass(shape, dtype, neuron, groups, which, kernel):
    names = launches(shape, dtype, neuron, groups, (which,))[which]
    assert any(kernel in n for n in names), names
