"""Batches whose centred input is the matrix operand itself (m = 0 or dense mode, activations of the operand's type): the kernel that
tests the 16-bit codes and reads its operands straight from the inputs, at the sizes where it can go wrong -- steps of 32 rows
(remainders, fewer than eight wavefronts' worth, one row), input lengths that are not a multiple of 8, columns that end inside a
tile, 8 and 9 tokens -- against the CPU oracle, and its rule on codes against the fp32 comparison for every code."""
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2412_07174_amd as scap
import workloads as wl
from workloads import BF16, F16, I8

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import Layer, check_against_oracle, f32_dev, gpu_sparse_fc, to_dev


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def layer_of(K, N, dt, seed, B=16):
    if dt == I8:
        W, sc = wl.quantize_i8(K, N, seed, std=0.05)
        return Layer(W, dt, sc, B=B)
    return Layer(wl.weights(K, N, seed, dt, std=0.05), dt, B=B)


def wide(layer):
    if layer.wdt == I8:
        return layer.W_host.astype(np.float64) * wl.decode(layer.scale_host, F16).astype(np.float64)[None, :]
    return wl.decode(layer.W_host, layer.wdt).astype(np.float64)


def sums_within_fp32(got, layer, D, bias, what):
    """Every result within the bound of an fp32 sum of its exact products, in any order: (terms + 2) * 2^-24 * sum |d w|, one more
    rounding for the column scale and the bias."""
    W = wide(layer)
    want = D.astype(np.float64) @ W + (0.0 if bias is None else bias.astype(np.float64)[None, :])
    bound = (np.count_nonzero(D, axis=1)[:, None] + 4) * 2.0 ** -24 * (np.abs(D) @ np.abs(W)) + 2.0 ** -22 * np.abs(want) + 1e-30
    off = np.abs(got - want)
    assert np.all(off <= bound), f"{what}: {np.max(off / bound)} times the bound"


def counts_alone(layer, X, xdt, m, tau, bias, got):
    """The counts without the lists -- each alone, both, together with y -- against those of the call with lists (checked against the
    oracle), on tickets of their own; y is the same to the bit whichever outputs are asked for."""
    B = X.shape[0]
    for nnz, union in ((True, True), (True, False), (False, True)):
        y = torch.full((B, layer.N), float("nan"), dtype=torch.float32, device="cuda")
        n = torch.full((B,), -7, dtype=torch.int32, device="cuda") if nnz else None
        u = torch.full((1,), -7, dtype=torch.int32, device="cuda") if union else None
        scap.sparse_fc(layer.W, to_dev(X, xdt), m, tau, f32_dev(bias), col_scale=layer.scale, y=y, nnz_out=n, union_nnz_out=u, workspace=layer.ws)
        torch.cuda.synchronize()
        what = f"counts alone K={layer.K} N={layer.N} B={B} tau={tau} nnz={nnz} union={union}"
        assert not nnz or np.array_equal(n.cpu().numpy(), got["nnz"]), what
        assert not union or int(u.item()) == got["union_nnz"], what
        assert np.array_equal(y.cpu().numpy().view(np.uint32), got["y"].view(np.uint32)), what


SHAPES = [
    # K, N: one row, less than a step, around one step, around eight steps, odd lengths, ragged tiles, several splits
    (1, 16), (8, 16), (31, 144), (32, 128), (33, 272), (255, 128), (256, 1040), (264, 2048), (777, 144), (1000, 4112), (4097, 528),
    (4096, 1024), (2048, 128),
]


@pytest.mark.parametrize("dt", [BF16, F16, I8])
@pytest.mark.parametrize("K,N", SHAPES)
def test_exact_operand_shapes(K, N, dt):
    layer = layer_of(K, N, dt, 9100 + K)
    xdt = F16 if dt == F16 else BF16
    bias = np.random.default_rng(K + N).standard_normal(N).astype(np.float32)
    X = wl.laplace(16, K, 9200 + K, xdt, loc=0.0, scale=0.6)
    Xf = wl.decode(X, xdt).astype(np.float64)
    for B, tau in ((5, 0.0), (8, 0.41), (9, 1.4), (16, 0.3), (16, 1e6)):
        say(f"exact operand K={K} N={N} dt={dt} B={B} tau={tau}")
        got, _ = check_against_oracle(layer, X[:B], xdt, 0.0, tau, bias, what=f"K={K} N={N} B={B} tau={tau}")
        D = np.where(np.abs(Xf[:B]) > np.float32(tau), Xf[:B], 0.0)
        sums_within_fp32(got["y"], layer, D, bias, f"K={K} N={N} B={B} tau={tau}")
        plain = torch.full((B, N), float("nan"), dtype=torch.float32, device="cuda")
        scap.sparse_fc(layer.W, to_dev(X[:B], xdt), 0.0, tau, f32_dev(bias), col_scale=layer.scale, y=plain, workspace=layer.ws)
        torch.cuda.synchronize()
        assert np.array_equal(plain.cpu().numpy().view(np.uint32), got["y"].view(np.uint32)), "y depends on the outputs requested"
        counts_alone(layer, X[:B], xdt, 0.0, tau, bias, got)
        # the general vector kernel: the same channels
        if K >= 64:
            other = gpu_sparse_fc(layer, X[:B], xdt, 0.0, tau, bias, cfg=(0, 0, 0, 64))
            assert np.array_equal(other["nnz"], got["nnz"]) and other["union_nnz"] == got["union_nnz"]
            assert all(np.array_equal(other["idx"][b], got["idx"][b]) for b in range(B))
    say(f"exact operand, dense mode K={K} N={N} dt={dt}")
    y = scap.dense_fc(layer.W, to_dev(X[:7], xdt), f32_dev(bias), col_scale=layer.scale, workspace=layer.ws)
    torch.cuda.synchronize()
    sums_within_fp32(y.cpu().numpy(), layer, Xf[:7], bias, f"dense K={K} N={N}")


@pytest.mark.parametrize("dt,xdt", [(BF16, BF16), (F16, F16), (I8, BF16), (BF16, F16), (F16, BF16), (I8, F16)])
@pytest.mark.parametrize("K,N", [(1, 16), (31, 144), (33, 272), (264, 2048), (1000, 4112), (4097, 528), (2048, 128)])
def test_centred_operand_shapes(K, N, dt, xdt):
    """m != 0, or activations of another type than the operand's: the same row steps with the centred values split into two halves
    (2^-17 of each product, fp16 2^-21)."""
    layer = layer_of(K, N, dt, 9600 + K)
    bias = np.random.default_rng(K + N).standard_normal(N).astype(np.float32)
    X = wl.laplace(16, K, 9700 + K, xdt, loc=0.1, scale=0.6)
    Xf = wl.decode(X, xdt).astype(np.float32)
    half = 2.0 ** -16 if dt != F16 else 2.0 ** -20
    W = np.abs(wide(layer))
    for B, m, tau in ((5, 0.1, 0.0), (8, -0.2, 0.41), (9, 0.1, 1.4), (16, 1.5, 0.3), (16, 0.0, 0.3)):
        say(f"centred operand K={K} N={N} dt={dt} xdt={xdt} B={B} m={m} tau={tau}")
        got, want = check_against_oracle(layer, X[:B], xdt, m, tau, bias, what=f"K={K} N={N} B={B} m={m} tau={tau}")
        D = Xf[:B] - np.float32(m)
        D = np.where(np.abs(D) > np.float32(tau), D, 0.0).astype(np.float64)
        exact = D @ wide(layer) + bias[None, :]
        bound = ((np.count_nonzero(D, axis=1)[:, None] + 4) * 2.0 ** -24 + half) * (np.abs(D) @ W) + 2.0 ** -22 * np.abs(exact) + 1e-6
        assert np.all(np.abs(got["y"] - exact) <= bound), (K, N, B, m, tau)
        counts_alone(layer, X[:B], xdt, m, tau, bias, got)
    y = scap.dense_fc(layer.W, to_dev(X[:7], xdt), f32_dev(bias), col_scale=layer.scale, workspace=layer.ws)
    torch.cuda.synchronize()
    exact = Xf[:7].astype(np.float64) @ wide(layer) + bias[None, :]
    bound = ((K + 4) * 2.0 ** -24 + half) * (np.abs(Xf[:7].astype(np.float64)) @ W) + 2.0 ** -22 * np.abs(exact) + 1e-6
    assert np.all(np.abs(y.cpu().numpy() - exact) <= bound), (K, N, "dense")


@pytest.mark.parametrize("dt", [BF16, F16])
def test_every_code_against_thresholds(dt):
    """All 65536 codes as inputs (subnormals, both zeros, infinities, NaN): kept exactly where the fp32 comparison keeps them, at
    thresholds on codes, between two codes, below the smallest and above the largest."""
    K, B = 8192, 8
    codes = np.arange(65536, dtype=np.uint16).reshape(B, K)
    val = wl.decode(codes, dt).astype(np.float32)
    layer = Layer(np.zeros((K, 16), dtype=np.uint16), dt, B=B)
    rng = np.random.default_rng(5)
    fin = np.abs(val[np.isfinite(val)])
    taus = [0.0, -0.0, float(fin.max()), float(np.nextafter(np.float32(fin.max()), np.float32(0))), 3.0e38, 1e-45, 65504.0, 65503.0, 65520.0, 6.1e-5,
            float(np.float32(2.0) ** -14), float(np.float32(2.0) ** -24)]
    for v in rng.choice(fin, 12):
        taus += [float(v), float(np.nextafter(v, np.float32(0))), float(np.nextafter(v, np.float32(3e38)))]
    for tau in taus:
        tau = float(np.float32(tau))
        say(f"codes dt={dt} tau={tau}")
        got = gpu_sparse_fc(layer, codes, dt, 0.0, tau, None)
        with np.errstate(invalid="ignore"):
            keep = np.abs(val) > np.float32(tau)
        for b in range(B):
            assert np.array_equal(got["idx"][b], np.nonzero(keep[b])[0]), (tau, b)
        assert got["union_nnz"] == int(keep.any(axis=0).sum())


def test_values_that_are_not_finite():
    """Infinities are kept and reach every column of their token, and no other token; NaN inputs are pruned, and kept in dense mode.
    What lies behind the last channel of an odd-length row (the next token's values) takes no part."""
    for K, dt in ((4096, BF16), (777, F16), (1001, BF16)):
        layer = layer_of(K, 144, dt, 9400 + K)
        X = wl.laplace(9, K, 9401 + K, dt, loc=0.0, scale=0.6)
        inf, nan = (0x7C00, 0x7E00) if dt == F16 else (0x7F80, 0x7FC0)
        X[3, 5] = inf
        X[4, 0] = nan | 0x8000
        X[6, K - 1] = nan
        X[8, 0] = nan
        say(f"not finite K={K} dt={dt}")
        check_against_oracle(layer, X, dt, 0.0, 0.3, None, what=f"not finite K={K}")
        y = scap.dense_fc(layer.W, to_dev(X, dt), None, workspace=layer.ws)
        torch.cuda.synchronize()
        bad = ~np.isfinite(y.cpu().numpy()).all(axis=1)
        assert np.array_equal(np.nonzero(bad)[0], [3, 4, 6, 8])


# 3-4 tokens on this kernel, either side of the layer sizes where it stops (3 tokens 2^25 weights; 32768 columns)
@pytest.mark.parametrize("dt", [BF16, F16, I8])
@pytest.mark.parametrize("K,N", [(33, 272), (1000, 4112), (4097, 528), (2048, 16384), (2056, 16384), (40, 32768), (40, 32784)])
def test_exact_operand_few_tokens(K, N, dt):
    layer = layer_of(K, N, dt, 9900 + K, B=4)
    xdt = F16 if dt == F16 else BF16
    X = wl.laplace(4, K, 9901 + K, xdt, loc=0.0, scale=0.6)
    if dt == F16:
        X[1, :7] = np.arange(1, 8)  # subnormal inputs count like any other
    Xf = wl.decode(X, xdt).astype(np.float64)
    for B, tau in ((3, 0.4), (4, 0.4), (4, 0.0)):
        say(f"exact operand, few tokens K={K} N={N} dt={dt} B={B} tau={tau}")
        got, _ = check_against_oracle(layer, X[:B], xdt, 0.0, tau, None, what=f"K={K} N={N} B={B} tau={tau}")
        counts_alone(layer, X[:B], xdt, 0.0, tau, None, got)
        sums_within_fp32(got["y"], layer, np.where(np.abs(Xf[:B]) > np.float32(tau), Xf[:B], 0.0), None, f"K={K} N={N} B={B} tau={tau}")


def test_subnormal_inputs_keep_their_products():
    """fp16 inputs below 2^-14 alone: the matrix instruction does not flush them."""
    layer = layer_of(512, 144, F16, 9950, B=8)
    X = (np.arange(8 * 512, dtype=np.uint16) % 1000).reshape(8, 512)
    Xf = wl.decode(X, F16).astype(np.float64)
    for B in (4, 8):
        say(f"subnormal inputs B={B}")
        y = gpu_sparse_fc(layer, X[:B], F16, 0.0, 0.0, None)["y"]
        sums_within_fp32(y, layer, Xf[:B], None, f"subnormal inputs B={B}")


@pytest.mark.parametrize("dt", [BF16, F16, I8])
@pytest.mark.parametrize("K,F,N,B", [(264, 520, 144, 5), (264, 520, 144, 2), (1001, 1032, 272, 2), (1001, 14336, 144, 2), (1001, 1032, 272, 3), (2048, 4104, 512, 4), (8, 16384, 144, 2), (8, 16392, 144, 4), (2048, 8200, 144, 2), (2056, 8200, 144, 2), (1032, 6656, 144, 2), (1001, 1032, 272, 9), (2048, 4104, 512, 16), (33, 8, 16, 8)])
def test_exact_operand_blocks(K, F, N, B, dt):
    """The block's gate|up launch on this kernel (centred inputs) against the oracle, token by token."""
    from test_gpu_swiglu import Block
    blk = Block(K, F, N, dt, seed=9500 + K, B=B)
    xdt = F16 if dt == F16 else BF16
    X = wl.laplace(B, K, 9501 + K, xdt, loc=0.0, scale=0.8)
    zs = np.abs(oracle.swiglu_block(blk.Wg, blk.Wu, blk.Wd, X[0], 0.0, 0.5, 0.0, 0.0, dt, xdt, gate_scale=blk.sg, up_scale=blk.su,
                                    down_scale=blk.sd)["z"])
    for tau_x, tau_z in ((0.0, 0.0), (0.5, float(np.median(zs))), (1.1, float(np.quantile(zs, 0.9))), (0.5, 1e9)):
        say(f"exact operand block K={K} F={F} N={N} B={B} dt={dt} tau_x={tau_x} tau_z={tau_z:.4g}")
        blk.check_batch(X, xdt, 0.0, tau_x, None, None, 0.0, tau_z, None, f"exact operand block {K} {F} {N} {B}")
        gots = blk.check_batch(X, xdt, 0.05, tau_x, None, None, 0.001, tau_z, None, f"centred operand block {K} {F} {N} {B}")
        nnz = torch.full((B,), -7, dtype=torch.int32, device="cuda")  # the counts without the lists
        y = scap.swiglu_block(blk.W_gu, blk.W_down, to_dev(X, xdt), 0.05, tau_x, None, 0.001, tau_z, None, gu_scale=blk.gu_scale,
                              down_scale=blk.down_scale, nnz_z_out=nnz, workspace=blk.ws)
        torch.cuda.synchronize()
        assert np.array_equal(nnz.cpu().numpy(), [g["idx_z"].size for g in gots])
        assert np.array_equal(y.cpu().numpy().view(np.uint32), np.stack([g["y"] for g in gots]).view(np.uint32))


def test_gated_products_below_the_operand_type():
    """Gated products so small that both halves of the operand round to 0 (fp16: below 2^-25) are kept by a threshold of 0, and counted
    and listed as such."""
    K, F, N, B = 64, 264, 144, 6
    from test_gpu_swiglu import Block
    blk = Block(K, F, N, F16, seed=9801, std=1e-4, B=B)
    X = wl.laplace(B, K, 9802, F16, loc=0.0, scale=0.01)
    gots = blk.run_batch(X, F16, 0.0, 0.0, None, None, 0.0, 0.0, None)
    for b in range(B):
        assert np.count_nonzero(np.abs(gots[b]["z"]) < 2.0 ** -26) > F // 2
        assert np.array_equal(gots[b]["idx_z"], np.nonzero(gots[b]["z"])[0])


def _large_and_small(K, N, dt, large, ones):
    """A layer whose products are 2^24 in channel `large` and 1 in the channels `ones`, with the exact sum of every column."""
    a, w = (2.0 ** 18, 64) if dt == I8 else (2.0 ** 12, 2.0 ** 12)
    xdt = F16 if dt == F16 else BF16
    W = np.zeros((K, N), dtype=np.float32)
    x = np.zeros(K, dtype=np.float32)
    W[large], x[large] = w, a
    W[ones], x[ones] = 1.0, 1.0

    def bits(v, t):
        if t == F16:
            return v.astype(np.float16).view(np.uint16)
        return (np.ascontiguousarray(v, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)

    if dt == I8:
        layer = Layer(W.astype(np.int8), dt, np.full(N, 0x3C00, dtype=np.uint16), B=16)
    else:
        layer = Layer(bits(W, dt), dt, B=16)
    return layer, xdt, bits(x, xdt), 2.0 ** 24 + len(ones)


@pytest.mark.parametrize("dt", [BF16, F16, I8])
@pytest.mark.parametrize("K,N", [(256, 144), (4096, 1024)])
def test_sums_of_wavefronts_and_splits_meet_without_a_rounding(K, N, dt):
    """2^24 and ones, each 1 in another wavefront's rows or another K split (steps of 32 rows: wavefront step % 8 of its piece; the
    first and the last step lie in different splits where there are several).  In 32 bits each 1 would be lost on 2^24 (ties to
    even); the exact sums are representable."""
    ones = [32, 64, K - 64, K - 32] if K > 256 else [32, 64, 96, 160]
    layer, xdt, x, want = _large_and_small(K, N, dt, 0, ones)
    for B in (3, 4, 5, 16):
        say(f"large and small K={K} N={N} dt={dt} B={B}")
        y = gpu_sparse_fc(layer, np.tile(x, (B, 1)), xdt, 0.0, 0.0, None)["y"]
        assert np.all(y == want), (B, y.min(), y.max(), want)


@pytest.mark.parametrize("dt", [BF16, F16])
def test_long_chains_of_a_wavefront_keep_small_products(dt):
    """One wavefront's rows alone (nine steps, 256 rows apart, of a piece of 2304): 2^24 in the first, ones in a later run of steps, which an
    accumulator that held 2^24 would lose."""
    layer, xdt, x, want = _large_and_small(4096, 144, dt, 0, [256 * st for st in (4, 5, 6, 7)])
    for B in (5, 16):
        say(f"long chain dt={dt} B={B}")
        y = gpu_sparse_fc(layer, np.tile(x, (B, 1)), xdt, 0.0, 0.0, None, cfg=(0, 2304, 0, 16))["y"]
        assert np.all(y == want), (B, y.min(), y.max(), want)


@pytest.mark.parametrize("B", [5, 16])
def test_blocks_of_more_columns_than_narrow_tiles(B):
    """int8 down launch in 16-byte lanes (256-column tiles, the sums through a tree): more than 1024 tiles of 128 columns."""
    from test_gpu_swiglu import Block
    K, F, N = 64, 72, 131104
    blk = Block(K, F, N, I8, seed=9990, std=0.05, B=B)
    X = wl.laplace(B, K, 9991, BF16, loc=0.0, scale=0.8)
    for m in (0.0, 0.05):
        say(f"int8 block of many columns B={B} m={m}")
        blk.check_batch(X, BF16, m, 0.4, None, None, 0.0, 0.01, None, f"many columns B={B} m={m}")


@pytest.mark.parametrize("m", [0.0, 0.1])
def test_longest_inputs(m):
    """2^20 channels, and a block whose gate|up launch has more of them than LDS-sized pieces could cover: a piece may be as long as the layer."""
    from test_gpu_swiglu import Block
    layer = layer_of(1 << 20, 16, F16, 9960)
    X = wl.laplace(5, 1 << 20, 9961, F16, loc=m, scale=0.6)
    say(f"longest input m={m}")
    check_against_oracle(layer, X, F16, m, 1.2, None, what=f"2^20 channels m={m}")
    blk = Block(700008, 8, 16, BF16, seed=9962, std=0.002, B=6)
    X = wl.laplace(6, 700008, 9963, BF16, loc=m, scale=0.6)
    say(f"long block m={m}")
    blk.check_batch(X, BF16, m, 1.2, None, None, 0.0, 0.05, None, f"long block m={m}")
