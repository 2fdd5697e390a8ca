"""GPU parity at the sizes where a choice of kernel, tile or hand-over changes: the edges that the general parity
tests do not visit.  Oracle, bar and helpers as there (lists and counts bit-exact, y within max-abs 1e-2, rel-L2 2e-3)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2412_07174_amd as scap
import workloads as wl
from workloads import BF16, F16, I8

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from gpu_util import Layer, assert_y_close, check_against_oracle, gpu_sparse_fc, to_dev
    from test_gpu_swiglu import B_MATRIX, Block


def _layer(K, N, wdt, seed, B=16):
    if wdt == I8:
        q, sc = wl.quantize_i8(K, N, seed)
        return Layer(q, I8, col_scale_bits=sc, B=B), BF16
    return Layer(wl.weights(K, N, seed, wdt), wdt, B=B), wdt


# tokens' lists are dealt out over the column tiles: one tile, fewer tiles than tokens, as many as lists, more
@pytest.mark.parametrize("lanes", [0, 64, 16, 1])
@pytest.mark.parametrize("K,N", [(40, 128), (1000, 128), (1000, 256), (2000, 384), (1100, 2048), (1100, 2176), (600, 2312)])
def test_lists_of_a_batch_whatever_the_number_of_tiles(K, N, lanes):
    layer, xdt = _layer(K, N, BF16, 900 + N)
    for B in (2, 5, 16):
        X = wl.laplace(B, K, 901 + K, xdt, loc=0.1, scale=0.5)
        for tau in (0.3, 1.2):
            print(f"lists K={K} N={N} B={B} lanes={lanes} tau={tau}", flush=True)
            check_against_oracle(layer, X, xdt, 0.1, tau, None, cfg=(0, 0, 0, lanes) if lanes else None, what=f"{K} {N} {B} {lanes}")


# an input length that is not a multiple of 8: the later tokens' rows start at any 2-byte boundary and the last octet is
# cut; shorter than an octet, just past chunk boundaries (64, 512), several splits
@pytest.mark.parametrize("wdt", [BF16, F16, I8])
@pytest.mark.parametrize("K,N", [(1, 144), (7, 144), (9, 4112), (65, 1040), (513, 144), (1001, 4112), (2047, 1040), (5461, 2752)])
def test_batches_over_an_odd_input_length(K, N, wdt):
    layer, xdt = _layer(K, N, wdt, 910 + K)
    for B in (2, 3, 4, 5, 9, 16):
        X = wl.laplace(B, K, 911 + K, xdt, loc=0.1, scale=0.5)
        for tau in (0.0, 0.9):
            print(f"odd K={K} N={N} wdt={wdt} B={B} tau={tau}", flush=True)
            check_against_oracle(layer, X, xdt, 0.1, tau, None, what=f"K={K} N={N} wdt={wdt} B={B} tau={tau}")
        y = scap.dense_fc(layer.W, to_dev(X, xdt), None, col_scale=layer.scale, workspace=layer.ws)
        torch.cuda.synchronize()
        want = oracle.dense_fc(layer.W_host, X, None, wdt, xdt, col_scale=layer.scale_host)
        assert_y_close(y.cpu().numpy(), want, f"dense K={K} N={N} wdt={wdt} B={B}")


def _exact(layer, X, xdt, m, tau):
    """float64 result of a layer without a fused bias (tau < 0: dense); x - m is one fp32 subtraction, as everywhere."""
    d = wl.decode(X, xdt).astype(np.float32)
    if tau >= 0:
        d = d - np.float32(m)
        d = np.where(np.abs(d) > np.float32(tau), d, np.float32(0))
    if layer.wdt == I8:
        W = layer.W_host.astype(np.float64) * wl.decode(layer.scale_host, F16).astype(np.float64)
    else:
        W = wl.decode(layer.W_host, layer.wdt).astype(np.float64)
    return d.astype(np.float64) @ W


def _rel(got, want):
    return np.linalg.norm(np.asarray(got, np.float64) - want) / np.linalg.norm(want)


# 3-4 tokens whose centred inputs need more bits than bf16 has.  Sums of K fp32 products in several chains stay within
# about 2^-23 of the result (1.3e-7 here); an operand split into two bf16 halves leaves up to 2^-17 per term, 1.8e-6 over
# random signs.  5e-7 lies between the two; 1e-5 would show a lost half (2^-9).
@pytest.mark.parametrize("K,N,bar", [(512, 256, 5e-7), (512, 512, 5e-7), (1024, 1024, 5e-7), (1000, 800, 5e-7),
                                     (513, 256, 5e-7), (2047, 1024, 5e-7), (5461, 1024, 5e-7), (520, 256, 1e-5), (4096, 1024, 1e-5)])
def test_centred_inputs_over_narrow_bf16_layers(K, N, bar):
    layer, xdt = _layer(K, N, BF16, 970 + K, B=4)
    for B in (3, 4):
        X = wl.laplace(B, K, 971 + K, xdt, loc=0.1, scale=0.5)
        print(f"centred narrow K={K} N={N} B={B}", flush=True)
        got, _ = check_against_oracle(layer, X, xdt, 0.1, 0.35, None, what=f"K={K} N={N} B={B}")
        err = _rel(got["y"], _exact(layer, X, xdt, 0.1, 0.35))
        assert err <= bar, (K, N, B, err)


# odd input lengths that the four-slot kernel does not take (more than 64 K splits; partial sums asked for), and dense
# ones: 3-4 tokens over bf16 weights stay with fp32 operands.  Bar as above.
@pytest.mark.parametrize("K,N,flags", [(100001, 128, 0), (5461, 1024, scap.CFG_PARTIAL_SUMS), (2047, 264, scap.CFG_GENERAL_KERNEL)])
def test_centred_inputs_of_odd_length_on_the_general_kernel(K, N, flags):
    layer, xdt = _layer(K, N, BF16, 980 + K, B=4)
    for B in (3, 4):
        X = wl.laplace(B, K, 981 + K, xdt, loc=0.1, scale=0.5)
        print(f"odd general K={K} N={N} B={B} flags={flags}", flush=True)
        cfg = (0, 0, 0, 0, flags) if flags else None
        got, _ = check_against_oracle(layer, X, xdt, 0.1, 0.35, None, cfg=cfg, what=f"K={K} N={N} B={B}")
        err = _rel(got["y"], _exact(layer, X, xdt, 0.1, 0.35))
        assert err <= 5e-7, (K, N, B, err)
        y = scap.dense_fc(layer.W, to_dev(X, xdt), None, workspace=layer.ws, cfg=cfg)
        torch.cuda.synchronize()
        err = _rel(y.cpu().numpy(), _exact(layer, X, xdt, 0.0, -1.0))
        assert err <= 5e-7, (K, N, B, err)


# the block over an odd hidden size; gated products that end inside a 32- or 64-channel segment
@pytest.mark.parametrize("dt", [BF16, F16, I8])
@pytest.mark.parametrize("K,F,N", [(129, 72, 144), (1001, 2088, 528), (519, 4104, 4112)])
def test_blocks_over_an_odd_hidden_size(K, F, N, dt):
    blk = Block(K, F, N, dt, 930 + K, B=16)
    xdt = F16 if dt == F16 else BF16
    rng = np.random.default_rng(931 + K)
    bg, bu, bd = (rng.standard_normal(n).astype(np.float32) * 0.1 for n in (F, F, N))
    for B in (2, 3, 4, 5, 16):
        X = wl.laplace(B, K, 932 + B, xdt, loc=0.05, scale=0.5)
        for tau_x, tau_z in ((0.0, 0.0), (0.3, 0.02), (0.8, 1e6)):
            print(f"odd block {K}->{F}->{N} dt={dt} B={B} tau_x={tau_x} tau_z={tau_z}", flush=True)
            blk.check_batch(X, xdt, 0.05, tau_x, bg, bu, 0.01, tau_z, bd, what=f"{K} {F} {N} B={B} {tau_x} {tau_z}")


# narrow layers: K splits that used to be pieces of 8-32 rows, up to the 64 splits of the fixed-point hand-over and past it
@pytest.mark.parametrize("wdt", [BF16, F16, I8])
@pytest.mark.parametrize("K,N", [(512, 512), (1024, 1024), (4096, 1024), (4099, 1040), (8200, 512), (33000, 128)])
def test_narrow_layers_of_one_to_four_tokens(K, N, wdt):
    layer, xdt = _layer(K, N, wdt, 940 + K, B=4)
    for B in (1, 2, 3, 4):
        X = wl.swiglu(B, K, 941 + K, xdt)
        print(f"narrow K={K} N={N} wdt={wdt} B={B}", flush=True)
        check_against_oracle(layer, X, xdt, 0.0, 0.4, None, what=f"K={K} N={N} wdt={wdt} B={B}")


# Long inputs and very wide layers whose best K split would give a workgroup more channels than the one-token kernel tests
# (2048): the split is taken among those it can run, so y += result, which no other kernel does, is not refused.
@pytest.mark.parametrize("K,N,wdt", [(132456, 1040, BF16), (133214, 1040, I8), (5169, 55600, BF16)])
def test_splits_stay_within_what_the_one_token_kernel_tests(K, N, wdt):
    g = torch.Generator(device="cuda").manual_seed(1020)
    if wdt == I8:
        W = torch.randint(-127, 128, (K, N), generator=g, device="cuda", dtype=torch.int8)
        scale = torch.full((N,), 2.0 ** -12, device="cuda").half()
        Wd = W.double() * scale.double()
    else:
        W, scale = (torch.randn(K, N, generator=g, device="cuda") * 0.02).bfloat16(), None
        Wd = W.double()
    x = (torch.randn(2, K, generator=g, device="cuda") + 0.1).bfloat16()
    d = x.float() - 0.1
    want = torch.where(d.abs() > 0.7, d, 0.0).double() @ Wd
    del Wd
    ws = scap.Workspace(K, N, 2)
    for B in (1, 2):
        print(f"long pieces K={K} N={N} wdt={wdt} B={B}", flush=True)
        y = scap.sparse_fc(W, x[:B].contiguous(), 0.1, 0.7, None, col_scale=scale, workspace=ws)
        torch.cuda.synchronize()
        assert float((y.double() - want[:B]).norm() / want[:B].norm()) <= 5e-7
    print(f"long pieces K={K} N={N} wdt={wdt} accumulate", flush=True)
    addend = torch.randn(1, N, generator=g, device="cuda")
    y = addend.clone()
    scap.sparse_fc(W, x[:1].contiguous(), 0.1, 0.7, None, col_scale=scale, y=y, workspace=ws, cfg=(0, 0, 0, 0, scap.CFG_ACCUMULATE))
    torch.cuda.synchronize()
    assert float((y.double() - want[:1] - addend).norm() / want[:1].norm()) <= 2e-6  # up to 256 additions in any order


def test_residual_block_with_a_very_wide_gate_up_layer():
    K, F, N = 5176, 27800, 64
    g = torch.Generator(device="cuda").manual_seed(1021)
    W_gu = (torch.randn(K, 2 * F, generator=g, device="cuda") * 0.02).bfloat16()
    W_down = (torch.randn(F, N, generator=g, device="cuda") * 0.02).bfloat16()
    x, addend = torch.randn(1, K, generator=g, device="cuda").bfloat16(), torch.randn(1, N, generator=g, device="cuda")
    ws = scap.Workspace(K, N, 1, F=F)
    print("residual block", flush=True)
    y = addend.clone()
    scap.swiglu_block(W_gu, W_down, x, 0.0, 0.5, None, 0.0, 0.0, None, y=y, workspace=ws, residual=True)
    want = scap.swiglu_block(W_gu, W_down, x, 0.0, 0.5, None, 0.0, 0.0, None, workspace=ws, cfg=(0, 0, 0, 0, scap.CFG_GENERAL_KERNEL))
    torch.cuda.synchronize()
    assert float((y - addend - want).norm() / want.norm()) <= 1e-5  # both sums of fp32 products, gated: no threshold on z


# int8 weights in 8- or 16-byte lanes: either side of the column count where the lanes change, and of the layer size
# from which 3-4 tokens go to the matrix cores
@pytest.mark.parametrize("K,N", [(300, 4096), (300, 4112), (1100, 16384), (1100, 16400), (5000, 16384)])
def test_int8_lane_widths(K, N):
    layer, xdt = _layer(K, N, I8, 950 + K, B=4)
    bf = np.random.default_rng(951 + K).standard_normal(N).astype(np.float32)
    for B in (1, 2, 3, 4):
        X = wl.laplace(B, K, 952 + K, xdt, loc=0.1, scale=0.5)
        print(f"int8 lanes K={K} N={N} B={B}", flush=True)
        check_against_oracle(layer, X, xdt, 0.1, 0.5, bf, what=f"K={K} N={N} B={B}")


# Small results keep their bits: a split's partial sums are handed over in fixed point only where that loses nothing
# against fp32.  Columns 512 and up (other slices than the first ones') are scaled by `scale`, in columns 64-127 only the
# later splits, columns 128-159 are huge; with several tokens the last one's inputs are scaled by 2^-8.  Each part by itself
# within the 5e-7 of above, as with ordinary magnitudes.
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -6, 2.0 ** -15, 2.0 ** -40])
@pytest.mark.parametrize("K,N,wdt", [(1024, 1024, BF16), (1024, 1024, F16), (1024, 1024, I8), (4096, 1032, BF16),
                                     (5461, 2744, BF16), (8193, 2048, BF16), (5461, 2752, I8), (4096, 11008, I8)])
def test_small_results_keep_their_bits(K, N, wdt, scale):
    if wdt == F16:
        scale = max(scale, 2.0 ** -6)  # smaller fp16 weights would underflow
    xdt = F16 if wdt == F16 else BF16
    if wdt == I8:
        q, sc = wl.quantize_i8(K, N, 990 + K)
        layer = Layer(q, I8, col_scale_bits=sc, B=4)
    else:
        w = wl.decode(wl.weights(K, N, 990 + K, wdt), wdt).astype(np.float32)
        w[:, 512:] *= np.float32(scale)
        w[K // 2:, 64:128] *= np.float32(scale)
        w[:, 128:160] *= np.float32(2.0 ** 14)
        layer = Layer(wl.encode(w, wdt), wdt, B=4)
    for B in (1, 2, 3, 4):
        x = wl.decode(wl.laplace(B, K, 991 + K, xdt, loc=0.1, scale=0.5), xdt).astype(np.float32)
        m, tau = 0.1, 0.35
        if wdt == I8:  # int8 weights have no small columns before their scale: all inputs small instead
            x, m, tau = x * np.float32(scale), 0.1 * scale, 0.35 * scale
        elif B > 1:
            x[-1] = 0.1 + (x[-1] - 0.1) * 2.0 ** -8
            tau = 0.35 * 2.0 ** -8
        X = wl.encode(x.astype(np.float32), xdt)
        print(f"small K={K} N={N} wdt={wdt} B={B} scale={scale}", flush=True)
        want = _exact(layer, X, xdt, m, tau)
        for cfg in (None, (0, 0, 0, 0, scap.CFG_PARTIAL_SUMS))[:2 if B <= 2 else 1]:
            got = gpu_sparse_fc(layer, X, xdt, m, tau, None, cfg=cfg)["y"]
            for b in range(B):
                for lo, hi in ((0, 64), (64, 128), (128, 160), (160, 512), (512, N)):
                    err = _rel(got[b, lo:hi], want[b, lo:hi])
                    assert err <= 5e-7, (K, N, wdt, B, b, lo, scale, cfg, err)


# the block of one to four tokens with gate and up so small that every hand-over escapes, after one with ordinary weights on
# the same workspace and before another.  z and y are products of two and three sums: three times the bar, and expf.
@pytest.mark.parametrize("dt", [BF16, I8])
def test_small_blocks_keep_their_bits(dt):
    K, F, N = 1032, 2056, 1032
    if dt == I8:
        K, F, N = 1040, 2064, 1040
    big, small = Block(K, F, N, dt, 1000, B=4), Block(K, F, N, dt, 1003, std=0.05 * (1.0 if dt == I8 else 2.0 ** -9), B=4)
    small.ws = big.ws
    m, spread = (0.05, 0.5) if dt == BF16 else (2.0 ** -14, 2.0 ** -13)
    X = wl.laplace(4, K, 1004, BF16, loc=m, scale=spread)
    for blk in (big, small, big):
        f = (lambda w, s: w.astype(np.float64) * wl.decode(s, F16).astype(np.float64) if dt == I8 else wl.decode(w, dt).astype(np.float64))
        Wg, Wu, Wd = f(blk.Wg, blk.sg), f(blk.Wu, blk.su), f(blk.Wd, blk.sd)
        for B in (1, 2, 3, 4):
            print(f"small block dt={dt} B={B} {'small' if blk is small else 'big'}", flush=True)
            d = (wl.decode(X[:B], BF16).astype(np.float32) - np.float32(m)).astype(np.float64)
            g, u = d @ Wg, d @ Wu
            z = g / (1 + np.exp(-g)) * u
            got = blk.run_batch(X[:B], BF16, m, 0.0, None, None, 0.0, 0.0, None)
            bar = 1e-5 if B_MATRIX(dt, B) else 2e-6
            for b in range(B):
                assert _rel(got[b]["z"], z[b]) <= bar, (dt, B, b, _rel(got[b]["z"], z[b]))
                assert _rel(got[b]["y"], z[b] @ Wd) <= bar, (dt, B, b, _rel(got[b]["y"], z[b] @ Wd))


# order statistics selected on the GPU: tiny samples, one value, even and odd counts, a median between two codes, between
# the signs and next to the NaNs, infinities on one side and on both, every target rank of a small sample
@pytest.mark.parametrize("dt", [F16, BF16])
def test_calibration_of_small_and_awkward_samples(dt):
    inf, nan = float("inf"), float("nan")
    samples = [[1.5], [1.5, -2.0], [0.0, -0.0], [-0.25, 0.5, 0.75], [2.0] * 100, [-1.0, -1.0, 1.0, 1.0], [1.0, inf, inf],
               [-inf, 0.25, inf], [inf, inf, inf, 1.0], [-inf, -inf, inf, inf], [nan, 1.0, 2.0], [nan, nan, 1.0],
               [nan] * 5, list(np.linspace(-3, 3, 77)), [6e-8, -6e-8, 3e-5, 0.0, 1e-7]]
    for v in samples:
        bits = wl.encode(np.array([v], dtype=np.float32), dt)
        ws = scap.Workspace(bits.shape[1], 0, 1)
        for est in (scap.MODE_ZERO, scap.MODE_MEDIAN):
            for s in (0.0, 0.01, 0.34, 0.5, 0.67, 0.99):
                print(f"calibrate dt={dt} {v[:5]} est={est} s={s}", flush=True)
                got = scap.calibrate(to_dev(bits, dt), s, est, workspace=ws)
                want = oracle.calibrate(bits, dt, s, est)
                assert np.array_equal(np.float32(got), np.float32(want), equal_nan=True), (v[:5], est, s, got, want)


# centred batches as they are planned (row steps up to 256 column tiles): workgroups of up to 512 channels and longer ones, narrow layers
@pytest.mark.parametrize("wdt", [BF16, F16, I8])
@pytest.mark.parametrize("K,N", [(64, 128), (512, 512), (4096, 1024), (4104, 1040), (8192, 2048), (5000, 8208)])
def test_staged_tile_short_and_long_workgroups(K, N, wdt):
    layer, xdt = _layer(K, N, wdt, 960 + K)
    for B in (5, 9, 16):
        X = wl.laplace(B, K, 961 + K, xdt, loc=0.1, scale=0.5)
        for tau in (0.0, 1.1):
            print(f"staged K={K} N={N} wdt={wdt} B={B} tau={tau}", flush=True)
            check_against_oracle(layer, X, xdt, 0.1, tau, None, what=f"K={K} N={N} wdt={wdt} B={B} tau={tau}")


# pieces that the caller names, the last one cut inside a step; 130 column tiles make more than 256 workgroups.  (Row steps; the pieces are
# those of the staged tile's prologues, which test_staged_tile_of_many_columns reaches)
@pytest.mark.parametrize("wdt,N", [(BF16, 144), (F16, 144), (I8, 272), (BF16, 130 * 128)])
@pytest.mark.parametrize("rows,K", [(2368, 2408), (2368, 4720), (2112, 2120), (2048, 4088), (1088, 2160), (1024, 1032), (576, 1144), (512, 1016)])
def test_staged_tile_prologues(rows, K, wdt, N):
    layer, xdt = _layer(K, N, wdt, 1010 + K)
    for B in (5, 16):
        X = wl.laplace(B, K, 1011 + K, xdt, loc=0.1, scale=0.5)
        for tau in (0.0, 1.4) if N < 1000 else (1.4,):
            print(f"prologue rows={rows} K={K} N={N} wdt={wdt} B={B} tau={tau}", flush=True)
            check_against_oracle(layer, X, xdt, 0.1, tau, None, cfg=(0, rows, 0, 16), what=f"{rows} {K} {N} {wdt} {B} {tau}")


# the same over input lengths that are not a multiple of 8, more than 256 workgroups among them
@pytest.mark.parametrize("wdt,N", [(BF16, 144), (F16, 144), (I8, 144), (I8, 130 * 128)])
@pytest.mark.parametrize("rows,K", [(2368, 2403), (2112, 2113), (1088, 2157), (1024, 1031), (576, 1141), (512, 1017), (64, 7)])
def test_staged_tile_prologues_of_odd_lengths(rows, K, wdt, N):
    layer, xdt = _layer(K, N, wdt, 1110 + K)
    for B in (5, 8, 16):
        X = wl.laplace(B, K, 1111 + K, xdt, loc=0.1, scale=0.5)
        for tau in (0.0, 1.4) if N < 1000 else (1.4,):
            print(f"odd prologue rows={rows} K={K} N={N} wdt={wdt} B={B} tau={tau}", flush=True)
            check_against_oracle(layer, X, xdt, 0.1, tau, None, cfg=(0, rows, 0, 16), what=f"{rows} {K} {N} {wdt} {B} {tau}")


# int8 layers around the choice between 16- and 8-byte lanes of the staged tile: both plans cost the same at 28672 columns (16-byte lanes), a
# tile less or more and 8-byte lanes are cheaper (3-4 tokens; 5 and more run row by row)
@pytest.mark.parametrize("K,N", [(1048, 28672), (2056, 28672), (1048, 24576), (2040, 28416), (1023, 28672), (2049, 20496)])
def test_int8_batches_of_both_lane_widths(K, N):
    layer, xdt = _layer(K, N, I8, 1210 + K)
    for B in (3, 4, 5, 16):
        X = wl.laplace(B, K, 1211 + K, xdt, loc=0.1, scale=0.5)
        print(f"int8 lanes K={K} N={N} B={B}", flush=True)
        check_against_oracle(layer, X, xdt, 0.1, 0.8, None, what=f"K={K} N={N} B={B}")


# blocks with centred inputs over int8 weights (both launches row step by row step) around the sizes where a launch's tiles fill the chip
@pytest.mark.parametrize("K,F,N", [(64, 6144, 8192), (64, 2048, 8208), (136, 4104, 1040)])
def test_int8_blocks_of_both_lane_widths(K, F, N):
    blk = Block(K, F, N, I8, 1310 + K, B=16)
    for B in (5, 16):
        X = wl.laplace(B, K, 1311 + B, BF16, loc=0.0, scale=0.5)
        print(f"int8 block lanes {K}->{F}->{N} B={B}", flush=True)
        blk.check_batch(X, BF16, 0.0, 0.3, None, None, 0.0, 0.004, None, what=f"{K} {F} {N} B={B}")


# the two-token block over int8 weights on 8-byte lanes: list segments of 32 channels, the gate|up launch in fixed point.
# The last segment cut, fewer channels than one, one tile and many; slices gated from registers and through memory (the same bits)
TWO_TOKEN_INT8 = [(256, 8, 16), (300, 72, 144), (1000, 2056, 1040), (520, 4104, 2064), (136, 16416, 528), (2000, 1032, 4112)]


@pytest.mark.parametrize("K,F,N", TWO_TOKEN_INT8)
def test_int8_blocks_of_two_tokens(K, F, N):
    blk = Block(K, F, N, I8, 1400 + K, std=0.05, B=2)
    X = wl.laplace(2, K, 1401 + K, BF16, loc=0.1, scale=0.5)
    for tau_x, tau_z in ((0.0, 0.0), (0.5, 0.02), (1e9, 0.0)):
        print(f"int8 block of two {K}->{F}->{N} tau_x={tau_x} tau_z={tau_z}", flush=True)
        args = (X, BF16, 0.1, tau_x, None, None, 0.01, tau_z, None)
        got = blk.check_batch(*args, what=f"{K} {F} {N} {tau_x} {tau_z}")
        for other in (blk.run_batch(*args), blk.run_batch(*args, cfg=(0, 0, 0, 0, scap.CFG_PARK_SLICES))):
            for b in range(2):
                assert np.array_equal(got[b]["y"].view(np.uint32), other[b]["y"].view(np.uint32)), (K, F, N, b)
                assert np.array_equal(got[b]["idx_z"], other[b]["idx_z"])


# ... with partial sums that escape the fixed point: 2^18 and more in magnitude before the column scale, i.e. large inputs over
# columns of a small scale.  "some": a few columns of a slice; "most": already 8 rows are mostly beyond the range.  Both are
# beyond what the oracle's fp32 sums are compared at, so z against double precision (the errors of 32-bit sums; no cancellation in
# silu(g) u), the lists against the z returned, y against double precision over those lists
@pytest.mark.parametrize("share", ["some", "most"])
@pytest.mark.parametrize("K,F,N", TWO_TOKEN_INT8)
def test_int8_blocks_of_two_tokens_beyond_the_fixed_point(K, F, N, share):
    up = 2.0 ** (2 if share == "some" else 10)
    blk = Block(K, F, N, I8, 1400 + K, std=0.05 / up / 64, B=2)
    X = wl.laplace(2, K, 1401 + K, BF16, loc=30.0 * up, scale=150.0 * up)
    m_x, tau_x, m_z, tau_z = np.float32(30.0 * up), np.float32(150.0 * up), np.float32(0.01), np.float32(0.02)
    d = wl.decode(X, BF16).astype(np.float32) - m_x
    d = np.where(np.abs(d) > tau_x, d, np.float32(0)).astype(np.float64)
    def beyond(rows):  # share of the partial sums of `rows` rows that lie beyond the range
        whole = K // rows * rows
        part = lambda W: np.einsum("bcr,crn->bcn", d[:, :whole].reshape(2, -1, rows), W[:whole].astype(np.float64).reshape(-1, rows, F))
        return np.mean([np.abs(part(W)) >= 2.0 ** 18 for W in (blk.Wg, blk.Wu)])
    # pieces have 24 to 80 rows here: more rows, more of them
    assert beyond(8) > 0.5 if share == "most" else beyond(24) > 0.005 and beyond(80) < 0.95, (beyond(8), beyond(24), beyond(80))
    f = lambda w, s: w.astype(np.float64) * wl.decode(s, F16).astype(np.float64)
    g, u = d @ f(blk.Wg, blk.sg), d @ f(blk.Wu, blk.su)
    z = g / (1 + np.exp(-g)) * u
    print(f"int8 block of two beyond the range {K}->{F}->{N} {share} |g| up to {np.abs(g).max():.3g}", flush=True)
    args = (X, BF16, float(m_x), float(tau_x), None, None, float(m_z), float(tau_z), None)
    got = blk.run_batch(*args)
    for b in range(2):
        assert np.isfinite(z[b]).all() and _rel(got[b]["z"], z[b]) <= 2e-6, (K, F, N, b, _rel(got[b]["z"], z[b]))
        dz = got[b]["z"] - m_z  # one fp32 subtraction
        kept = np.nonzero(np.abs(dz) > tau_z)[0]
        assert np.array_equal(got[b]["idx_z"], kept), (K, F, N, b)
        y = dz[kept].astype(np.float64) @ f(blk.Wd[kept], blk.sd)
        assert _rel(got[b]["y"], y) <= 2e-6, (K, F, N, b, _rel(got[b]["y"], y))
    for other in (blk.run_batch(*args), blk.run_batch(*args, cfg=(0, 0, 0, 0, scap.CFG_PARK_SLICES))):
        for b in range(2):
            assert np.array_equal(got[b]["y"].view(np.uint32), other[b]["y"].view(np.uint32)), (K, F, N, b)
            assert np.array_equal(got[b]["idx_z"], other[b]["idx_z"])


# the histogram estimator where the range it bins is infinite: every finite value counts in bin 0 and the estimate is the
# centre of an infinitely wide bin (lo + inf), or NaN where the lower end is -inf; a few infinities beyond the 0.1 % that the
# range leaves out change nothing about it
@pytest.mark.parametrize("dt", [F16, BF16])
def test_histogram_mode_of_a_sample_with_infinities(dt):
    inf, neg = (0x7C00, 0xFC00) if dt == F16 else (0x7F80, 0xFF80)
    base = wl.laplace(1, 4000, 1500 + dt, dt, loc=0.1, scale=0.5)
    ws = scap.Workspace(4000, 0, 1)
    for at, want in (({inf: 40}, (np.inf, np.inf)), ({neg: 40}, (np.nan, np.nan)), ({inf: 40, neg: 40}, (np.nan, np.nan)),
                     ({inf: 4000}, (np.inf, np.nan)), ({inf: 2, neg: 2}, None)):
        X, p = base.copy(), 0
        for code, n in at.items():
            X[0, p:p + n] = code
            p += n
        print(f"hist with infinities dt={dt} {at}", flush=True)
        got = scap.calibrate(to_dev(X, dt), 0.5, scap.MODE_HIST, workspace=ws)
        assert np.array_equal(got, oracle.calibrate(X, dt, 0.5, oracle.MODE_HIST), equal_nan=True), (at, got)
        assert want is None or np.array_equal(got, want, equal_nan=True), (at, got)
        assert want is not None or np.isfinite(got).all()


# the selection's groups of 64 codes: runs of 16 and of 32 codes, the last group whose counts LDS holds and the first that is
# read from memory, all of them
@pytest.mark.parametrize("groups", [1, 255, 256, 257, 511, 512, 513, 640, 1024])
def test_calibrate_selects_among_any_number_of_groups(groups):
    rng = np.random.default_rng(1600 + groups)
    for dt in (F16, BF16):
        X = np.repeat(rng.permutation(1024)[:groups].astype(np.uint16) * 64, 7)
        X = (X + rng.integers(0, 64, X.size).astype(np.uint16))[None]
        ws = scap.Workspace(X.shape[1], 0, 1)
        for est, oest in ((scap.MODE_ZERO, oracle.MODE_ZERO), (scap.MODE_MEDIAN, oracle.MODE_MEDIAN)):
            for s in (0.02, 0.5, 0.97):
                print(f"groups={groups} dt={dt} est={est} s={s}", flush=True)
                got = scap.calibrate(to_dev(X, dt), s, est, workspace=ws)
                assert np.array_equal(got, oracle.calibrate(X, dt, s, oest), equal_nan=True), (groups, dt, est, s, got)


# int8, 3-4 tokens, a call that names its rows per workgroup: up to 4096 of them in wide layers and over odd lengths, whose
# lists have room for as many; beyond that, and past 2368 where the staged tile runs, the call is refused
@pytest.mark.parametrize("K,N,rows,ok", [(1024, 8192, 4096, True), (3000, 12288, 2432, True), (4160, 17408, 4096, True),
                                         (1023, 1040, 2432, True), (2047, 4112, 4096, True), (1024, 8192, 4160, False),
                                         (1024, 8192, 64, True), (2048, 8192, 2432, False), (2048, 8192, 2368, True)])
def test_int8_rows_per_group_of_three_and_four_tokens(K, N, rows, ok):
    layer, xdt = _layer(K, N, I8, 1700 + K + rows)
    for B in (3, 4):
        X = wl.laplace(B, K, 1701 + K, xdt, loc=0.1, scale=0.5)
        print(f"int8 rows K={K} N={N} rows={rows} B={B}", flush=True)
        if ok:
            check_against_oracle(layer, X, xdt, 0.1, 0.8, None, cfg=(0, rows, 0, 0), what=f"K={K} N={N} rows={rows} B={B}")
        else:
            with pytest.raises(scap.ScapError, match="status -9"):
                gpu_sparse_fc(layer, X, xdt, 0.1, 0.8, None, cfg=(0, rows, 0, 0))


# ... and where the gate|up launch runs in 16-byte lanes (64-channel segments, partial sums): pieces of more than 512 rows that
# would be heavier in 8-byte lanes, the last segment cut, an odd input length; more columns than there are fixed-point words;
# paired with the general kernels, where the input of the down launch, or of the gate|up launch, is too long; and a down launch
# in wide lanes behind a gate|up launch in 8-byte lanes
@pytest.mark.parametrize("K,F,N", [(136, 2056, 16400), (1040, 22088, 144), (1041, 22088, 2064), (136, 32776, 528), (8, 131080, 1040), (140000, 8, 528)])
def test_int8_blocks_of_two_tokens_in_wide_lanes(K, F, N):
    blk = Block(K, F, N, I8, 1800 + K, std=0.02 if K > 2000 else 0.05, B=2)
    X = wl.laplace(2, K, 1801 + K, BF16, loc=0.1, scale=0.5)
    rng = np.random.default_rng(1802 + K)
    bg, bu, bd = (rng.standard_normal(n).astype(np.float32) * 0.05 for n in (F, F, N))
    for tau_x, tau_z in ((0.0, 0.0), (0.5, 0.02), (1e9, 0.0)):
        print(f"int8 block of two, wide lanes {K}->{F}->{N} tau_x={tau_x} tau_z={tau_z}", flush=True)
        args = (X, BF16, 0.1, tau_x, bg, bu, 0.01, tau_z, bd)
        got = blk.check_batch(*args, what=f"{K} {F} {N} {tau_x} {tau_z}")
        blk.check_batch(*args, what=f"{K} {F} {N} {tau_x} {tau_z} general kernels", cfg=(0, 0, 0, 0, scap.CFG_GENERAL_KERNEL))
        for other in (blk.run_batch(*args), blk.run_batch(*args, cfg=(0, 0, 0, 0, scap.CFG_PARK_SLICES))):
            for b in range(2):
                assert np.array_equal(got[b]["y"].view(np.uint32), other[b]["y"].view(np.uint32)), (K, F, N, b)
                assert np.array_equal(got[b]["idx_z"], other[b]["idx_z"])


# ... and where more narrow workgroups than compute units would be needed: rows that start on a cache line, or short pieces, and
# less than three times the wide ones, or not; longer pieces over other rows; 3-4 tokens on the 4-slot lists of pieces that the
# tile's LDS does not hold, and instead of more than 256 wide workgroups; odd lengths on either side
@pytest.mark.parametrize("K,N", [(64, 33280), (344, 33280), (64, 32864), (344, 32864), (1968, 16432), (1352, 32864), (2400, 49632),
                                 (1560, 39216), (343, 32864), (513, 43680), (1231, 56960), (6001, 11280)])
def test_int8_batches_of_more_tiles_than_compute_units(K, N):
    layer, xdt = _layer(K, N, I8, 1250 + K)
    for B in (3, 4, 5, 16):
        X = wl.laplace(B, K, 1251 + K, xdt, loc=0.1, scale=0.5)
        print(f"int8 lanes, many tiles K={K} N={N} B={B}", flush=True)
        check_against_oracle(layer, X, xdt, 0.1, 0.8, None, what=f"K={K} N={N} B={B}")


# three tokens where the pieces that fill the chip are longer than the kernel tests, but not than its LDS holds
def test_three_tokens_over_pieces_past_the_kernels_limit():
    K, N = 4104, 43528
    layer, xdt = _layer(K, N, BF16, 1900, B=4)
    X = wl.laplace(4, K, 1901, xdt, loc=0.1, scale=0.5)
    for B in (3, 4):
        print(f"long pieces K={K} N={N} B={B}", flush=True)
        check_against_oracle(layer, X[:B], xdt, 0.1, 0.9, None, what=f"K={K} N={N} B={B}")


# 16-bit batches in pieces of more than 1024 rows and more than 256 workgroups: up to 512 of them, more of them, pieces of more than 2048
@pytest.mark.parametrize("wdt", [BF16, F16])
@pytest.mark.parametrize("K,N,rows", [(2048, 33000, 2048), (1600, 33000, 1600), (1536, 33000, 1536), (4096, 33000, 2048), (2368, 33000, 2368)])
def test_batches_of_long_pieces_and_many_workgroups(K, N, rows, wdt):
    layer, xdt = _layer(K, N, wdt, 1950 + K)
    for B in (5, 16):
        X = wl.laplace(B, K, 1951 + K, xdt, loc=0.1, scale=0.5)
        print(f"long pieces of a batch K={K} N={N} rows={rows} wdt={wdt} B={B}", flush=True)
        check_against_oracle(layer, X, xdt, 0.1, 1.1, None, cfg=(0, rows, 0, 16), what=f"K={K} N={N} rows={rows} wdt={wdt} B={B}")


# one and two tokens over layers whose K splits lie a power of two of bytes apart: each split takes its list in a ring from a place of its
# own.  Dense, sparse with the caller's lists, few rows left per wavefront, none
@pytest.mark.parametrize("K,N,dt", [(4096, 8192, BF16), (16384, 4096, I8)])
def test_splits_that_start_their_lists_in_turn(K, N, dt):
    layer, xdt = _layer(K, N, dt, 2100 + K)
    X = wl.laplace(2, K, 2101 + K, xdt, loc=0.1, scale=0.5)
    for B in (1, 2):
        for tau in (0.0, 0.6, 2.6, 1e9):
            print(f"splits in turn K={K} N={N} B={B} tau={tau}", flush=True)
            check_against_oracle(layer, X[:B], xdt, 0.1, tau, None, what=f"K={K} N={N} B={B} tau={tau}")


# the staged tile where centred batches still run on it: more column tiles than compute units.  Each form of its prologue (1, 2, 4 or 5 chunks
# of 64 channels per wavefront, pieces on either side of 1536 rows among those of 4) at the shortest and longest piece, even and odd lengths;
# int8 weights in either lane width
@pytest.mark.parametrize("wdt,N", [(BF16, 32784), (F16, 32784), (I8, 32784)])
@pytest.mark.parametrize("rows,K", [(512, 520), (576, 584), (1088, 1096), (1600, 1608), (2112, 2120), (512, 517), (576, 583), (1088, 1091), (64, 7)])
def test_staged_tile_of_many_columns(rows, K, wdt, N):
    layer, xdt = _layer(K, N, wdt, 2200 + K)
    for B in (5, 16):
        X = wl.laplace(B, K, 2201 + K, xdt, loc=0.1, scale=0.5)
        for cfg in ((0, rows, 0, 16), None) if B == 5 else ((0, rows, 0, 16),):
            print(f"many columns rows={rows} K={K} N={N} wdt={wdt} B={B} cfg={cfg}", flush=True)
            check_against_oracle(layer, X, xdt, 0.1, 1.1, None, cfg=cfg, what=f"{rows} {K} {N} {wdt} {B} {cfg}")


# ... int8 weights in 8-byte lanes, odd length, pieces of more than four chunks: rows that start on a cache line, 5-8 tokens
def test_staged_tile_of_odd_lengths_in_long_pieces():
    rows, K, N = 2112, 2117, 32896
    layer, xdt = _layer(K, N, I8, 2250)
    X = wl.laplace(5, K, 2251, xdt, loc=0.1, scale=0.5)
    print(f"odd length in long pieces rows={rows} K={K} N={N}", flush=True)
    check_against_oracle(layer, X, xdt, 0.1, 1.1, None, cfg=(0, rows, 0, 16), what=f"{rows} {K} {N}")


# ... and the gate|up launch of blocks there, whose last arrivals leave planes of operand halves.  511 tiles of 128 columns take two rounds, so pieces are
# as long as the input: 16-bit weights in every chunk form, even and odd lengths; int8 in 16-byte lanes; then int8 in 8-byte lanes (three rounds of two
# pieces; odd lengths), with the last 256-column tile half past F, and odd lengths on the 16-slot value lists (16 tokens)
@pytest.mark.parametrize("dt,K,F", [(dt, K, 32704) for K in (264, 1000, 1088, 1600, 2120, 267, 583, 1101) for dt in (BF16, F16)] +
                                   [(I8, K, 32704) for K in (264, 504, 1000, 1600, 2120, 267, 1601)] +
                                   [(I8, 264, 16456), (I8, 2000, 24576), (I8, 3000, 24576), (I8, 1040, 22088), (I8, 1041, 22088), (I8, 1601, 22088)])
def test_centred_blocks_of_many_columns(dt, K, F):
    N, xdt = 144, F16 if dt == F16 else BF16
    blk = Block(K, F, N, dt, 2300 + K, std=0.03, B=16)
    X = wl.laplace(16, K, 2301 + K, xdt, loc=0.1, scale=0.5)
    zc = oracle.swiglu_block(blk.Wg, blk.Wu, blk.Wd, X[0], 0.1, 0.5, 0.0, 0.0, dt, xdt, gate_scale=blk.sg, up_scale=blk.su, down_scale=blk.sd, nthreads=8)["z"]
    tau_z = float(np.median(np.abs(zc)))
    for B in (5, 16):
        print(f"centred block of many columns {K}->{F} dt={dt} B={B}", flush=True)
        gots = blk.run_batch(X[:B], xdt, 0.1, 0.5, None, None, 0.0, tau_z, None)
        for b in sorted({0, B // 2, B - 1}):
            want = oracle.swiglu_block(blk.Wg, blk.Wu, blk.Wd, X[b], 0.1, 0.5, 0.0, tau_z, dt, xdt, gate_scale=blk.sg, up_scale=blk.su, down_scale=blk.sd, nthreads=8)
            blk.compare(gots[b], want, 0.0, tau_z, f"centred block of many columns {K} {F} dt={dt} B={B} token {b}", matrix_cores=True)
