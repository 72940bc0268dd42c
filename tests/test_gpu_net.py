"""The whole-network training calls: equal bit for bit to the per-layer calls
they stand for (forward, corrected forward, backward with and without
accumulation and input gradient, Adam with the bf16 and transposed copies)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2012_03525_amd import acm, closure

pytestmark = pytest.mark.gpu

vp = closure._vp


def per_layer_forward(net, q, acts):
    L = acm.lib()
    acm.check(L.acm_cnn_pack(net.nx, net.ny, vp(q["drho"]), vp(q["u"]), vp(q["v"]), closure._f3(net.in_scale),
                             vp(acts[0]), net.stream))
    raw = torch.zeros_like(net.raw)
    for l, (ci, co) in enumerate(net.shapes):
        last = l == closure.LAYERS - 1
        acm.check(L.acm_cnn_conv(net.nx, net.ny, ci, co, closure.CONV_RAW if last else closure.CONV_RELU,
                                 vp(acts[l]), vp(net.w16[l]), vp(net.b32[l]), None, vp(raw if last else acts[l + 1]),
                                 net.stream))
    return raw


@pytest.mark.parametrize("nx,ny", [(64, 8), (128, 40), (192, 64)])
def test_whole_network_calls(nx, ny):
    L = acm.lib()
    g = torch.Generator(device="cuda").manual_seed(nx + ny)
    q = {k: torch.randn((ny, nx), generator=g, device="cuda") for k in ("drho", "u", "v")}
    net = closure.Network(nx, ny, seed=3, in_scale=(0.7, 0.5, 0.9), out_scale=(0.0, 1e-2, 2e-2))
    acts = net.new_acts()
    raw = per_layer_forward(net, q, acts)
    net.forward(q["drho"], q["u"], q["v"])
    assert torch.equal(net.raw, raw)
    for a, b in zip(net.acts, acts):
        assert torch.equal(a, b)
    # the corrected state against the in-place correction of a copy
    want = {k: t.clone() for k, t in q.items()}
    net.apply(want["drho"], want["u"], want["v"])
    out = {k: torch.full_like(t, 7.0) for k, t in q.items()}
    net.forward(q["drho"], q["u"], q["v"], out=out)
    for k in q:
        assert torch.equal(out[k], want[k]), k
    with pytest.raises(acm.AcmError):
        net.forward(q["drho"], q["u"], q["v"], out=q)
    # backward against the per-layer calls
    net.gout.copy_(torch.randn(net.gout.shape, generator=g, device="cuda"))
    zero16 = torch.zeros(16, device="cuda")
    gin, gin2 = torch.zeros((ny, nx, 16), device="cuda"), torch.zeros((ny, nx, 16), device="cuda")
    for add in (False, True):
        gw = [t.clone() for t in net.gw]
        gb = [t.clone() for t in net.gb]
        grad, wg = net.gout, (L.acm_cnn_wgrad_add if add else L.acm_cnn_wgrad)
        for l in range(closure.LAYERS - 1, -1, -1):
            ci, co = net.shapes[l]
            acm.check(wg(nx, ny, ci, co, vp(net.acts[l]), vp(grad), vp(net.wg_ws), vp(gw[l]), vp(gb[l]), net.stream))
            if l:
                nxt = torch.zeros_like(net.gacts[l - 1])
                acm.check(L.acm_cnn_conv(nx, ny, co, ci, closure.CONV_MASK, vp(grad), vp(net.wt16[l]), None,
                                         vp(net.acts[l]), vp(nxt), net.stream))
            else:
                acm.check(L.acm_cnn_conv(nx, ny, co, ci, closure.CONV_RAW, vp(grad), vp(net.wt16[0]), vp(zero16), None,
                                         vp(gin2), net.stream))
            grad = nxt
        net.backward(accumulate=add, gin=gin, zero16=zero16)
        for l in range(closure.LAYERS):
            assert torch.equal(net.gw[l], gw[l]) and torch.equal(net.gb[l], gb[l]), (add, l)
        assert torch.equal(gin, gin2)
    # Adam against one call per tensor and the transposes
    ref = {n: [t.clone() for t in getattr(net, n)] for n in ("w32", "b32", "mw", "vw", "mb", "vb", "w16", "wt16")}
    for t in (1, 2):
        for l, (ci, co) in enumerate(net.shapes):
            for p, gr, m, v, h in ((ref["w32"][l], net.gw[l], ref["mw"][l], ref["vw"][l], ref["w16"][l]),
                                   (ref["b32"][l], net.gb[l], ref["mb"][l], ref["vb"][l], None)):
                acm.check(L.acm_cnn_adam(p.numel(), vp(p), vp(gr), vp(m), vp(v), vp(h), 1e-3, 0.9, 0.999, 1e-8, t,
                                         net.stream))
            acm.check(L.acm_cnn_transpose(ci, co, vp(ref["w16"][l]), vp(ref["wt16"][l]), net.stream))
        net.adam(1e-3)
    for n, ts in ref.items():
        for a, b in zip(getattr(net, n), ts):
            assert torch.equal(a, b), n


def test_weight_gradient_bias_sum():
    """The bias gradient (a product with ones) against the FP64 sum."""
    nx, ny, co = 128, 16, 32
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((ny, nx, 32), generator=g, device="cuda").to(torch.bfloat16)
    gr = torch.randn((ny, nx, co), generator=g, device="cuda").to(torch.bfloat16)
    L = acm.lib()
    ws = torch.zeros(L.acm_cnn_wgrad_workspace(nx, ny, 32, co) // 4, device="cuda")
    dw, db = torch.zeros((9, co, 32), device="cuda"), torch.zeros(co, device="cuda")
    acm.check(L.acm_cnn_wgrad(nx, ny, 32, co, vp(x), vp(gr), vp(ws), vp(dw), vp(db),
                              ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    want = gr.double().sum((0, 1)).cpu().numpy()
    # FP32 sums of 2048 values of size 1: 2048 half-ulps of the largest partial sum
    assert np.abs(db.double().cpu().numpy() - want).max() <= 2048 * 6e-8 * np.abs(want).max() + 1e-4
    ws_, dws = x.double().cpu(), gr.double().cpu()
    t = 5  # tap (0, +1)
    ref = torch.einsum("yxo,yxi->oi", dws, torch.roll(ws_, -1, 1))
    assert torch.allclose(dw[t].double().cpu(), ref, rtol=0, atol=2048 * 6e-8 * float(ref.abs().max()) + 1e-3)
