"""The convolution and weight-gradient kernels walk strips of columns down bands of rows:
sizes around a strip's width (16 and 32 columns), a single row or column, several bands,
and outputs that are not 16-byte aligned.  Reference: the same network in float64 on the
same bfloat16-rounded tensors, read back layer by layer."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2104_06165_amd as pm  # noqa: E402

SIZES = [(1, 1, 1), (2, 1, 15), (1, 3, 16), (2, 2, 17), (1, 5, 31), (3, 4, 32), (1, 9, 33), (1, 300, 7), (8, 70, 130)]


def bf16(t):
    return t.float().to(torch.bfloat16).double()


def layers(params):
    o = 0
    for ci, co in pm.Net.SHAPES:
        w = params[o:o + 9 * ci * co].reshape(9, ci, co)
        o += 9 * ci * co
        yield w, params[o:o + co]
        o += co


def taps(x):
    """(9, B, h, w, C): the input of each tap, zero outside the image."""
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    h, w = x.shape[1:3]
    return torch.stack([p[:, t // 3:t // 3 + h, t % 3:t % 3 + w] for t in range(9)])


@pytest.mark.parametrize("B,h,w", SIZES)
def test_strips(B, h, w):
    g = torch.Generator().manual_seed(100 * h + w)
    net = pm.Net(0, (0.3 * torch.randn(pm.Net.param_count(), generator=g)).numpy().astype(np.float32))
    params = torch.from_numpy(net.get_params()).cuda().double()
    x = torch.randn((B, h, w, 5), generator=g).cuda()
    target = torch.cat([2.0 + torch.rand((B, h, w, 1), generator=g),
                        torch.nn.functional.normalize(torch.randn((B, h, w, 3), generator=g), dim=-1)], -1)
    mask = torch.ones((B, h, w)).cuda()
    rng = torch.tensor([[1.0, 9.0]] * B).cuda()
    out = net.forward(x)
    _, grad = net.loss_grad(x, target.float().contiguous().cuda(), mask, rng, 1.0, True, True)
    acts = [net.tensor(0, l).double() for l in range(5)]
    gouts = [net.tensor(1, l).double() for l in range(5)]
    assert torch.equal(acts[0], bf16(x))
    # a sum of n products in FP32 is off by at most n 2^-24 of the sum of their magnitudes
    u = 2.0 ** -24
    o = 0
    for l, (wt, b) in enumerate(layers(params)):
        ci, co = pm.Net.SHAPES[l]
        wb = bf16(wt)
        T = taps(acts[l])
        n = 9 * 32 + 2
        y = torch.einsum("tbhwi,tio->bhwo", T.cpu(), wb.cpu()).cuda() + b
        bound = (torch.einsum("tbhwi,tio->bhwo", T.abs().cpu(), wb.abs().cpu()).cuda() + b.abs()) * n * u
        if l == 4:
            assert ((out.double() - y).abs() <= bound).all()
        else:  # stored as bfloat16: half a unit in the last place more
            y = y.clamp_min(0)
            assert ((acts[l + 1] - y).abs() <= bound + y.abs() * 2.0 ** -8).all()
        # weight and bias gradients from the stored tensors
        G = gouts[l]
        dw = torch.einsum("tbhwi,bhwo->tio", T.cpu(), G.cpu()).cuda()
        mag = torch.einsum("tbhwi,bhwo->tio", T.abs().cpu(), G.abs().cpu()).cuda()
        got = grad[o:o + 9 * ci * co].double().reshape(9, ci, co)
        k = B * h * w + 64
        assert ((got - dw).abs() <= mag * k * u).all()
        o += 9 * ci * co
        assert ((grad[o:o + co].double() - G.sum((0, 1, 2))).abs() <= G.abs().sum((0, 1, 2)) * k * u).all()
        o += co
        # data gradient into the layer below, through its ReLU
        if l:
            F = taps(gouts[l])
            flipped = wb.flip(0).transpose(1, 2).contiguous()
            gi = torch.einsum("tbhwo,toi->bhwi", F.cpu(), flipped.cpu()).cuda()
            gm = torch.einsum("tbhwo,toi->bhwi", F.abs().cpu(), flipped.abs().cpu()).cuda() * n * u
            gi = torch.where(acts[l] > 0, gi, torch.zeros_like(gi))
            # (values below bfloat16's normal range round to multiples of 2^-133)
            assert ((gouts[l - 1] - gi).abs() <= gm + gi.abs() * 2.0 ** -8 + 2.0 ** -133).all()
    net.close()


def test_unaligned_output():
    """The C entry point takes any float pointer as output."""
    net = pm.Net(0, np.load(pm.LIB_PATH.replace("libphimvs.so", "weights/proposal_net.npy")).astype(np.float32))
    x = torch.randn((1, 5, 19, 5), generator=torch.Generator().manual_seed(3)).cuda()
    ref = net.forward(x)
    raw = torch.zeros(5 * 19 * 4 + 3, device="cuda")
    for off in (1, 2, 3):
        raw.zero_()
        rc = pm.lib().phimvs_net_forward(net.h, 1, 5, 19, x.data_ptr(), ctypes.c_void_p(raw.data_ptr() + 4 * off))
        torch.cuda.synchronize()
        assert rc == 0 and torch.equal(raw[off:off + 5 * 19 * 4].reshape(5, 19, 4), ref[0])
        assert raw[:off].abs().sum() == 0 and raw[off + 5 * 19 * 4:].abs().sum() == 0
    net.close()


@pytest.mark.parametrize("B,h,w", [(2049, 2, 5), (700, 3, 97), (5000, 1, 33)])
def test_more_strips_than_waves(B, h, w):
    test_strips(B, h, w)


def test_a_row_of_more_than_2_to_the_31_elements():
    """A row of 2^26 pixels (32 channels: 2^31 elements) whose content and loss lie at its end, against
    a row of 128 with the same end: the gradients differ by the ratio of the pixel counts, a power
    of two (which bfloat16 and FP32 carry exactly), and by the order of the sums over some 40 columns,
    40 x 2^-24 of their terms; a strip read from elsewhere would change them by their own size."""
    W = 1 << 26
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GB of device memory")
    g = torch.Generator().manual_seed(26)
    net = pm.Net(0, np.load(pm.LIB_PATH.replace("libphimvs.so", "weights/proposal_net.npy")).astype(np.float32))
    end = torch.randn((64, 5), generator=g).cuda()
    tgt = torch.cat([2.0 + torch.rand((32, 1), generator=g), torch.nn.functional.normalize(torch.randn((32, 3), generator=g), dim=-1)], -1).cuda()
    grads = []
    for w in (128, W):
        x = torch.zeros((1, 1, w, 5), device="cuda")
        x[0, 0, -64:] = end
        target = torch.ones((1, 1, w, 4), device="cuda")
        target[0, 0, -32:] = tgt
        mask = torch.zeros((1, 1, w), device="cuda")
        mask[0, 0, -32:] = 1
        print(f"a row of {w} pixels", flush=True)
        _, grad = net.loss_grad(x, target, mask, torch.tensor([[1.0, 9.0]], device="cuda"), 1.0, True, True)
        grads.append(grad.double().clone() * w)
        del x, target, mask
    net.close()
    scale = grads[0].abs().max()
    assert float((grads[1] - grads[0]).abs().max()) <= float(scale) * 2.0 ** -10
    assert float(scale) > 0
