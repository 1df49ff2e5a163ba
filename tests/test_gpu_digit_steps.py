"""The operands of the matrix-core forward kernel as apb_compress builds them on the GPU, byte for byte against a builder
on the host (digit_steps_host.cpp, one bit at a time) that takes the exported CSR: steps, counts, first steps, row sums
(same order of additions: same bits), and the sign words against a rearrangement in numpy."""
import ctypes
import os
import subprocess

import numpy as np
import pytest
import torch

from paper_2306_08960_amd import synth

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def b():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2306_08960_amd import binding
    binding.load()
    return binding


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("digits") / "digit_steps_host.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-shared", "-fPIC", os.path.join(HERE, "digit_steps_host.cpp"), "-o", lib],
                   check=True)
    return ctypes.CDLL(lib)


def compare(b, host, W, delta, alpha, tag):
    N, K = W.shape
    print(f"[case] digit steps {tag} N={N} K={K}", flush=True)
    layer = b.apb_compress(torch.from_numpy(W).cuda(), float(delta), alpha=alpha)
    csr = {k: v.cpu().numpy() if torch.is_tensor(v) else v for k, v in b.apb_layer_export(layer).items()}
    got = b.apb_layer_export_steps(layer)
    layer.free()
    sizes = (ctypes.c_longlong * 3)()
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)           # noqa: E731
    row_ptr, col, val = (np.ascontiguousarray(csr[k]) for k in ("row_ptr", "col_idx", "val"))
    host.digit_steps_build(N, K, ptr(row_ptr), ptr(col), ptr(val), sizes)
    assert (got["steps"], got["windows"]) == (sizes[0], sizes[1])
    if csr["nnz"]:
        assert got["unit"] == sizes[2]
    want = {k: np.empty(tuple(got[k].shape), t) for k, t in (("first", np.int32), ("count", np.uint8), ("step", np.uint8), ("valsum", np.float64))}
    host.digit_steps_copy(*(ptr(a) for a in want.values()))
    for k, a in want.items():
        g = got[k].cpu().numpy()
        if k == "valsum":
            g, a = g.view(np.uint64), a.view(np.uint64)
        bad = np.argwhere(g != a)
        assert not len(bad), f"{k}: {len(bad)} of {a.size} differ, first at {bad[0]}"
    # sign words: [tile][step][lane (i, g)] = word 4 * step + g of row 16 * tile + i, bit pairs swapped for odd g
    tiles, Kw = 2 * ((N + 31) // 32), (K + 31) // 32
    ksteps = (Kw + 3) // 4
    words = np.zeros((16 * tiles, 4 * ksteps), np.uint32)
    words[:N, :Kw] = csr["sign_words"].view(np.uint32)
    words[:, 1::2] = ((words[:, 1::2] & 0x33333333) << 2) | ((words[:, 1::2] >> 2) & 0x33333333)
    want_sign = words.reshape(tiles, 16, ksteps, 4).transpose(0, 2, 3, 1).reshape(-1)
    assert np.array_equal(got["sign"].cpu().numpy().view(np.uint32), want_sign)
    return got["windows"]


@pytest.mark.parametrize("N,K,rho", [(1, 1, 0.5), (1, 64, 0.3), (7, 31, 0.5), (16, 33, 0.2), (33, 127, 0.05), (64, 576, 0.02), (100, 517, 0.02),
                                     (130, 2049, 0.1), (512, 4608, 0.03), (40, 8192, 0.05), (40, 8193, 0.05), (34, 18432, 0.02),
                                     (256, 300, 0.0)])
def test_layers_of_trained_weights(b, host, N, K, rho):
    W, delta, _, _ = synth.random_case(9400 + N + K, N, K, 1, 2, rho=max(rho, 1e-9))
    assert compare(b, host, W, 1e9 if rho == 0.0 else delta, None, f"rho {rho}") == 1


def test_lists_of_every_length_that_the_kernel_has_code_for(b, host):
    # 0, 1, 127 .. 129, 256, 257, ... residuals in a row, alone in their pair or beside a row with other columns
    g = np.random.default_rng(41)
    lengths = [0, 1, 127, 128, 129, 256, 257, 384, 385, 512, 513, 768, 769, 1024, 1025, 1536, 1537, 2000]
    W = (g.standard_normal((16 * len(lengths), 2000)) * 0.01).astype(np.float32)
    for t, n in enumerate(lengths):
        for r in (16 * t, 16 * t + 9):
            W[r, g.choice(2000, n, replace=False)] = g.choice([-0.4, 0.7, 0.53], n)
    compare(b, host, W, 0.2, None, "list lengths")


def test_every_weight_a_residual(b, host):
    W = np.random.default_rng(42).standard_normal((35, 18432)).astype(np.float32)
    assert compare(b, host, W, -1.0, None, "dense") >= 1       # (as many steps as a quad can have)


@pytest.mark.parametrize("spread", [6, 40, 100, 240])
def test_several_windows(b, host, spread):
    g = np.random.default_rng(43 + spread)
    W = (g.standard_normal((70, 300)) * 2.0 ** g.integers(-spread // 2, spread - spread // 2 + 1, (70, 300))).astype(np.float32)
    W[5, :4] = np.float32(2.0) ** np.array([-(spread // 2) - 12, spread - spread // 2 - 10, 0, 1], np.float32)
    assert compare(b, host, W, -1.0, 0.0, f"2^{spread}") > 1


def test_zeros_denormals_infinities_and_nan(b, host):
    W = np.random.default_rng(44).standard_normal((20, 100)).astype(np.float32)
    W[0, 0], W[1, 1], W[2, 2], W[3, 3], W[4, 4] = 0.0, 1e-45, np.inf, -np.inf, 3e38
    assert compare(b, host, W, -1.0, 0.0, "extremes") > 1
