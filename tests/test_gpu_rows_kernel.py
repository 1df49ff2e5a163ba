"""The matrix-core forward kernel (residuals as base-32 digits; every layer whose code table fits on chip) through
apb_forward, against the CPU oracle: every output of Y within 1e-5 relative, no floor.  Each case first checks, by the
kernel name the library reports, whether it is this kernel that runs.  Shapes: rows not a multiple of 16 (padding
tiles), K not a multiple of 128 or of 32 (padded matrix steps, partial last word), column groups with fewer than 16 valid
columns, one column, empty rows and rows of very different lengths (padding entries in the digit steps), the largest K
whose code table fits on chip, both activation widths.  Every case that runs on this kernel also runs its packed-output
form (apb_forward_requant) and compares the codes and column sums with the oracle's."""
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


def check(b, W, delta, X, bits, step, tag, expect_rows=True):
    N, K = W.shape
    M = X.shape[1]
    print(f"[case] rows kernel {tag} N={N} K={K} M={M} bits={bits}", flush=True)
    L = o.compress(W, delta)
    c = o.quantize(X, bits, step)
    F = capi.forward(L, o.pack_acts(c, bits), c, bits, step, threads=THREADS)
    layer = b.apb_compress(torch.from_numpy(W).cuda(), float(delta), alpha=float(L["alpha"]))
    name = b.apb_forward_kernel_name(layer, M, bits)
    assert name.startswith("k_forward_rows") == expect_rows, name
    packed = b.apb_quantize_acts(torch.from_numpy(X).cuda(), bits, float(step))
    Y = torch.full((N, M), float("nan"), device="cuda")
    b.apb_forward(layer, packed, M, bits, float(step), Y=Y)
    Y = Y.cpu().numpy().astype(np.float64)
    ref = F["Y"].astype(np.float64)
    bad = ~(np.abs(Y - ref) <= 1e-5 * np.abs(ref))             # (a NaN left in Y counts as bad)
    assert not bad.any(), f"{int(bad.sum())} of {bad.size} outputs off; first at {np.argwhere(bad)[0]}"
    if expect_rows:
        # the same kernel ending in the next layer's quantizer (apb_forward_requant): both output widths, with and
        # without the per-row affine map, into a buffer full of ones
        r = np.random.default_rng(N + K)
        for bits_out in (2, 1):
            step_out = np.float32(np.std(ref) * 0.7 + 1e-3)
            scale = r.uniform(0.5, 1.5, N).astype(np.float32)
            shift = (r.standard_normal(N) * float(step_out)).astype(np.float32)
            for sc, sh in ((None, None), (scale, shift)):
                want = o.requant(L["alpha"], step, F["D"], F["R"], bits_out, step_out, sc, sh)
                out = b.alloc_packed(N, M, bits_out)
                out.fill_(-1)
                b.apb_forward_requant(layer, packed, M, bits, float(step), bits_out, float(step_out),
                                      None if sc is None else torch.from_numpy(sc).cuda(),
                                      None if sh is None else torch.from_numpy(sh).cuda(), packed_out=out)
                torch.cuda.synchronize()
                code, colsum = unpack(out.cpu().numpy().view(np.uint32), N, M, bits_out)
                assert np.array_equal(colsum[:M], code.sum(axis=0))
                compare_codes(code, want, L["alpha"], step, F["D"], F["R"], bits_out, step_out, sc, sh)
    layer.free()


SHAPES = [(256, 128, 16), (257, 100, 1), (300, 97, 15), (320, 1000, 17), (513, 300, 100), (640, 4100, 70),
          (1000, 257, 1000), (256, 2304, 333),
          # a few more column tiles than fill the chip, ragged M
          (512, 300, 8310), (600, 200, 5590),
          # about one workgroup per compute unit and a few more
          (256, 128, 4340), (300, 97, 2200),
          # many rows and few columns: the tiles are shared by several workgroups
          (4100, 500, 250), (4100, 300, 120), (4100, 4100, 250)]


@pytest.mark.parametrize("bits", [1, 2])
@pytest.mark.parametrize("N,K,M", SHAPES)
def test_ragged_shapes(b, N, K, M, bits):
    W, delta, X, step = synth.random_case(9000 + N + K + M + bits, N, K, M, bits, rho=0.12)
    check(b, W, delta, X, bits, step, "ragged")


@pytest.mark.parametrize("N,K,M,bits", [(10, 500, 17000, 2), (32, 576, 25088, 1), (32, 4900, 16400, 2),    # two tiles and many columns
                                        (512, 4864, 12544, 1)])            # tables of 152 KB beside the rows' sums
def test_sizes_at_the_edges_of_the_launch_choice(b, N, K, M, bits):
    W, delta, X, step = synth.random_case(9300 + N + K + bits, N, K, M, bits, rho=0.02)
    check(b, W, delta, X, bits, step, "launch choice")


@pytest.mark.parametrize("K", [331, 683, 2049, 8192, 8193, 12001])
@pytest.mark.parametrize("bits", [1, 2])
def test_long_rows_are_summed_exactly(b, K, bits):
    # Every weight a residual (delta < 0, alpha = 0), values of 24 bits whose digits are as large as they get, or random
    # ones, and the largest codes: the digit sums of a row pass 2^24, where a float would round.  The float64 sum of the
    # reference is exact (below 2^53 units), so both sides round once and must agree to the bit.
    g = np.random.default_rng(K + bits)
    N, M, step = 40, 33, 0.5
    print(f"[case] long rows K={K} bits={bits}", flush=True)
    units = g.integers(1 << 23, 1 << 24, (N, K)) * g.choice([-1, 1], (N, K))
    units[::4] = 0xf7bdef                                        # digits 15, 15, 15, 15, 15 (of the window's lower 25 bits)
    units[1::4] = -0xf7bdef
    units[2::4] = g.choice([0xf7bdef, -0xf7bdef, 0x841ef, 1], (len(units[2::4]), K))
    W = (units.astype(np.float64) * 2.0 ** -24).astype(np.float32)
    X = (g.standard_normal((K, M)) * 2).astype(np.float32)
    X[:, :5] = 9.0                                               # all codes at their largest
    code = np.where(X >= 0, 1, -1) if bits == 1 else np.clip(np.rint(X * np.float32(1 / step)), 0, 3)
    want = (units.astype(np.float64) @ code.astype(np.float64) * (step * 2.0 ** -24)).astype(np.float32)
    layer = b.apb_compress(torch.from_numpy(W).cuda(), -1.0, alpha=0.0)
    name = b.apb_forward_kernel_name(layer, M, bits)
    assert name.startswith("k_forward_rows") and name.endswith("true>" if K > 8192 else "false>"), name
    got = b.apb_quantize_forward(layer, torch.from_numpy(X).cuda(), bits, step).cpu().numpy()
    assert np.array_equal(got, want)
    layer.free()


@pytest.mark.parametrize("N,K,M", [(100, 700, 90), (64, 300, 2100), (270, 1000, 333)])
@pytest.mark.parametrize("bits", [1, 2])
def test_residuals_of_very_different_magnitudes(b, N, K, M, bits):
    # several windows of digits; in some quads only the lowest or only the highest holds any
    g = np.random.default_rng(34 + N)
    W = (g.standard_normal((N, K)) * 0.01).astype(np.float32)
    for n in range(0, N, 2):
        cols = g.choice(K, size=n % 50, replace=False)
        mag = 2.0 ** (g.integers(-1, 18, cols.size) if n % 3 else np.full(cols.size, 17 if n % 4 else 0))
        W[n, cols] = (0.7 * mag * (1 + g.random(cols.size)) * g.choice([-1, 1], cols.size)).astype(np.float32)
    X = g.standard_normal((K, M)).astype(np.float32)
    if bits == 2:
        np.maximum(X, 0, out=X)
    step = np.float32(0.75)
    layer = b.apb_compress(torch.from_numpy(W).cuda(), 0.2)
    assert b.apb_forward_kernel_name(layer, M, bits).endswith("true>") and b.apb_layer_export_steps(layer)["windows"] == 2
    Xd = torch.from_numpy(X).cuda()
    Y = b.apb_forward(layer, b.apb_quantize_acts(Xd, bits, float(step)), M, bits, float(step))
    assert torch.equal(b.apb_quantize_forward(layer, Xd, bits, float(step)), Y)
    layer.free()
    check(b, W, np.float32(0.2), X, bits, step, "several windows")


def test_empty_rows_and_very_uneven_rows(b):
    g = np.random.default_rng(31)
    N, K, M = 384, 700, 90
    W = (g.standard_normal((N, K)) * 0.01).astype(np.float32)   # all inside the interval ...
    delta = np.float32(0.2)
    counts = g.integers(0, 61, size=N)                           # ... except planted residuals: 0 to 60 per row,
    counts[::7] = 0                                              # every seventh row none at all
    for n in range(N):
        cols = g.choice(K, size=counts[n], replace=False)
        W[n, cols] = (0.3 + g.random(counts[n])).astype(np.float32) * g.choice([-1.0, 1.0], size=counts[n]).astype(np.float32)
    for bits, step in ((1, 1.0), (2, 0.75)):
        X = g.standard_normal((K, M)).astype(np.float32)
        if bits == 2:
            np.maximum(X, 0, out=X)
        check(b, W, delta, X, bits, np.float32(step), "uneven rows")


def test_largest_k_whose_table_fits_and_the_fallback_beyond(b):
    g = np.random.default_rng(32)
    for K, expect in ((18432, True), (18464, False)):
        W, delta, X, step = synth.random_case(9100 + K, 256, K, 40, 2, rho=0.01)
        check(b, W, delta, X, 2, step, "largest K" if expect else "K beyond the table", expect_rows=expect)


def test_layers_of_few_rows_few_residuals_or_one_very_long_row(b):
    # one row carrying residuals in every column beside light rows
    g = np.random.default_rng(33)
    W = (g.standard_normal((384, 700)) * 0.01).astype(np.float32)
    W[5] = 0.5
    W[::3, :8] = -0.4
    X = np.maximum(g.standard_normal((700, 90)), 0).astype(np.float32)
    check(b, W, np.float32(0.2), X, 2, np.float32(0.75), "one very long row")
    W, delta, X, step = synth.random_case(9200, 128, 512, 64, 2, rho=0.05)
    check(b, W, delta, X, 2, step, "128 rows")
    W, delta, X, step = synth.random_case(9201, 512, 512, 64, 2, rho=0.001)       # hardly any residuals
    check(b, W, delta, X, 2, step, "0.1 % residuals")


@pytest.mark.parametrize("name", ["C3_r05_b1", "C3_r50_b1", "C3_r50_b2", "C5a", "C5b"])
def test_benchmark_layers_run_on_it(b, name):
    cfg = synth.CONFIGS[name]
    W, delta, X, step = synth.make_layer(cfg)
    check(b, W, delta, X, cfg.bits, step, name)
