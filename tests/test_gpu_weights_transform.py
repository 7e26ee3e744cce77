"""tpla_transform_latent on bf16 weights, through the matrix-core kernel from a number of vectors on: rows and columns, ragged counts, every basis and
direction, and the same call in place (which takes the general kernel), against float64."""
import numpy as np
import pytest
import torch

import paper_2508_15881_amd as tp
from paper_2508_15881_amd import pipeline as pl
from paper_2508_15881_amd import workloads as wl
from oracle import tpla_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_c,n_outer,n_inner", [(64, 1, 1), (64, 130, 1), (192, 257, 1), (512, 129, 1), (512, 4096, 1), (64, 1, 8),
                                                 (128, 3, 40), (256, 2, 136), (512, 5, 128), (320, 1, 256),
                                                 # Hadamard bases: from here on the matrix-core kernel
                                                 (64, 3000, 1), (128, 3001, 1), (256, 4096, 1), (512, 8200, 1), (64, 3, 72), (128, 1, 384),
                                                 (256, 11, 72), (512, 12, 136)])
@pytest.mark.parametrize("mode,inverse,signed", [("dense", 0, False), ("dense", 1, False), ("hadamard", 0, True), ("hadamard", 1, True),
                                                 ("hadamard", 0, False)])
def test_weights_transform(d_c, n_outer, n_inner, mode, inverse, signed):
    if mode == "hadamard" and d_c & (d_c - 1):
        pytest.skip("a Hadamard basis needs a power of two")
    print(f"[gpu] weights transform d_c={d_c} n_outer={n_outer} n_inner={n_inner} {mode} inverse={inverse}", flush=True)
    rng = np.random.default_rng(d_c + n_outer + n_inner)
    shape = tp.TplaShape(1, 1, d_c, 1, 8, 8, 8, 64, tp.TPLA_BF16, 1.0)
    x = wl.to_storage(rng.standard_normal((n_outer, d_c, n_inner)) * 0.05, "bf16")
    signs = rng.choice(np.array([-1.0, 1.0]), size=d_c).astype(np.float32) if signed else None
    if mode == "dense":
        U = np.linalg.qr(rng.standard_normal((d_c, d_c)))[0].astype(np.float32)
        U64, code = U.astype(np.float64), tp.TPLA_U_DENSE
    else:
        U, U64, code = None, orc.hadamard_U(d_c, signs if signed else np.ones(d_c)), tp.TPLA_U_HADAMARD
    V = U64.T if inverse else U64
    x64 = wl.as_f64(x, "bf16")
    ref = np.einsum("oki,kj->oji", x64, V)
    # float sums of d_c exact products, then one rounding to bf16: half a step where the value lies, 2^(e - 8) for values from
    # 2^e on (a second rounding on the way would pass it)
    sums = d_c * 2.0 ** -24 * np.einsum("oki,kj->oji", np.abs(x64), np.abs(V))
    bound = sums + np.ldexp(1.0, np.frexp(np.abs(ref) + sums)[1] - 9)
    src = pl.to_device(x, "bf16")
    dst = torch.full_like(src, float("nan"))
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    tp.tpla_transform_latent(shape, code, inverse, dev(signs), dev(U), src, dst, n_outer, n_inner)
    torch.cuda.synchronize()
    got = wl.as_f64(pl.from_device_bits(dst), "bf16")
    assert np.all(np.abs(got - ref) <= bound)
    tp.tpla_transform_latent(shape, code, inverse, dev(signs), dev(U), src, src, n_outer, n_inner)
    torch.cuda.synchronize()
    assert np.all(np.abs(wl.as_f64(pl.from_device_bits(src), "bf16") - ref) <= bound)


@pytest.mark.parametrize("n_outer,n_inner", [(5, 1), (1, 40)])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_a_weight_that_is_not_finite(n_outer, n_inner, value):
    """An infinity stays one (its sign by the basis entry), a NaN spreads, and no other vector sees either.  The entries of
    the basis are powers of two: all low terms are zero."""
    print(f"[gpu] weights transform n_outer={n_outer} n_inner={n_inner} with {value}", flush=True)
    d_c = 64
    shape = tp.TplaShape(1, 1, d_c, 1, 8, 8, 8, 64, tp.TPLA_BF16, 1.0)
    x = np.ones((n_outer, d_c, n_inner))
    x[0, 7, n_inner // 2] = value
    U = orc.hadamard_U(d_c, np.ones(d_c))
    src = pl.to_device(wl.to_storage(x, "bf16"), "bf16")
    dst = torch.zeros_like(src)
    tp.tpla_transform_latent(shape, tp.TPLA_U_DENSE, 0, None, torch.from_numpy(U.astype(np.float32)).cuda(), src, dst, n_outer, n_inner)
    torch.cuda.synchronize()
    got = wl.as_f64(pl.from_device_bits(dst), "bf16")
    ref = np.ones_like(x)
    ref[...] = (np.ones(d_c) @ U)[None, :, None]
    ref[0, :, n_inner // 2] = value * U[7]
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.allclose(np.nan_to_num(got), np.nan_to_num(ref), rtol=2.0 ** -8, atol=1e-6)
