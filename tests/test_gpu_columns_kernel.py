"""The columns-in-lanes forward kernel (lanes along the columns of Y) where it serves layers that the other kernel could
serve as well: few residuals per row and many outputs.  Every form of the forward against the CPU oracle -- outputs within
1e-5 relative, no floor -- on both sides of the sizes where the choice changes, with ragged M; the one-kernel step and the
implicit convolution bit for bit against their two calls."""
import os

import numpy as np
import pytest
import torch

from oracle import apb_oracle as o
from oracle import capi
from paper_2306_08960_amd import synth
from requant_checks import compare_codes, unpack

pytestmark = pytest.mark.gpu
THREADS = max(1, min(16, len(os.sched_getaffinity(0))))


@pytest.fixture(scope="module")
def b():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2306_08960_amd import binding
    binding.load()
    return binding


# (rows, K, columns, residuals, float output here, packed output here)
CASES = [(64, 90, 60000, 0.03, True, True), (64, 90, 59999, 0.03, False, True), (33, 70, 40001, 0.05, False, True), (20, 64, 39999, 0.05, False, False),
         (64, 200, 90000, 0.06, True, True), (64, 200, 89999, 0.06, False, True), (32, 200, 90001, 0.06, False, True),
         (128, 96, 31250, 0.03, True, False), (128, 96, 31249, 0.03, False, False), (100, 600, 40020, 0.02, True, False),
         (130, 200, 30800, 0.02, True, False), (300, 100, 13334, 0.03, True, False), (300, 100, 13333, 0.03, False, False),
         (128, 96, 31250, 0.5, False, False)]                  # (too many residuals)


@pytest.mark.parametrize("bits", [1, 2])
@pytest.mark.parametrize("N,K,M,rho,float_here,packed_here", CASES)
def test_every_form_on_both_sides_of_the_rule(b, N, K, M, rho, float_here, packed_here, bits):
    print(f"[case] columns kernel N={N} K={K} M={M} rho={rho} bits={bits}", flush=True)
    W, delta, X, step = synth.random_case(9500 + N + K + bits, N, K, M, bits, rho=rho)
    L = o.compress(W, delta)
    c = o.quantize(X, bits, step)
    F = capi.forward(L, o.pack_acts(c, bits), c, bits, step, threads=THREADS)
    layer = b.apb_compress(torch.from_numpy(W).cuda(), float(delta), alpha=float(L["alpha"]))
    assert b.apb_forward_kernel_name(layer, M, bits).startswith("k_forward_rows") != float_here
    Xd = torch.from_numpy(X).cuda()
    packed = b.apb_quantize_acts(Xd, bits, float(step))
    Y = torch.full((N, M), float("nan"), device="cuda")
    b.apb_forward(layer, packed, M, bits, float(step), Y=Y)
    got, ref = Y.cpu().numpy().astype(np.float64), F["Y"].astype(np.float64)
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref))
    assert torch.equal(b.apb_quantize_forward(layer, Xd, bits, float(step)), Y)
    Ys = torch.full((N, M), float("nan"), device="cuda")
    b.apb_quantize_forward_static(layer, Xd, bits, float(step), Ys)
    assert torch.equal(Ys, Y)
    step_out = np.float32(np.std(ref) * 0.7 + 1e-3)
    r = np.random.default_rng(N + K)
    scale, shift = r.uniform(0.5, 1.5, N).astype(np.float32), (r.standard_normal(N) * float(step_out)).astype(np.float32)
    for bits_out in (1, 2):
        want = o.requant(L["alpha"], step, F["D"], F["R"], bits_out, step_out, scale, shift)
        out = b.alloc_packed(N, M, bits_out)
        out.fill_(-1)
        b.apb_forward_requant(layer, packed, M, bits, float(step), bits_out, float(step_out), torch.from_numpy(scale).cuda(),
                              torch.from_numpy(shift).cuda(), packed_out=out)
        code, colsum = unpack(out.cpu().numpy().view(np.uint32), N, M, bits_out)
        assert np.array_equal(colsum[:M], code.sum(axis=0))
        compare_codes(code, want, L["alpha"], step, F["D"], F["R"], bits_out, step_out, scale, shift)
    layer.free()


@pytest.mark.parametrize("N,B,H,W,stride", [(64, 61, 32, 32, 1), (96, 50, 30, 29, 1), (64, 250, 31, 33, 2)])
@pytest.mark.parametrize("bits", [1, 2])
def test_convolutions(b, N, B, H, W, stride, bits):
    print(f"[case] columns kernel conv N={N} B={B} H={H} W={W} stride={stride} bits={bits}", flush=True)
    C = 32
    Wt, delta, _, step = synth.random_case(9600 + N + H + bits, N, 9 * C, 1, bits, rho=0.02)
    Xmap = np.random.default_rng(H).standard_normal((C, B * H * W)).astype(np.float32)
    if bits == 2:
        np.maximum(Xmap, 0, out=Xmap)
    layer = b.apb_compress(torch.from_numpy(Wt).cuda(), float(delta))
    P = B * o.conv_out_size(H, stride) * o.conv_out_size(W, stride)
    assert not b.apb_forward_kernel_name(layer, P, bits).startswith("k_forward_rows")
    fmap = b.apb_quantize_acts(torch.from_numpy(Xmap).cuda(), bits, float(step))
    patches = torch.from_numpy(o.im2col_codes(o.quantize(Xmap, bits, step), B, H, W, bits, stride).astype(np.float32)).cuda() * float(step)
    packed = b.apb_quantize_acts(patches, bits, float(step))
    del patches
    Y = b.apb_forward_conv3x3(layer, fmap, B, H, W, bits, float(step), stride=stride)
    assert torch.equal(Y, b.apb_forward(layer, packed, P, bits, float(step)))
    out = b.apb_forward_conv3x3_requant(layer, fmap, B, H, W, bits, float(step), 2, 1.0, stride=stride)
    assert torch.equal(out, b.apb_forward_requant(layer, packed, P, bits, float(step), 2, 1.0))
    assert torch.equal(out, b.apb_quantize_acts(Y, 2, 1.0))
    layer.free()
