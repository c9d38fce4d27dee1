"""Edges of the kernels' tilings and value ranges, against the CPU oracle."""
import numpy as np
import pytest

import oracle
import synth
from oracle import groups as og
from oracle import qat as oq

pytestmark = pytest.mark.gpu


def dev(a, gpu):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(gpu)


def host(t):
    return t.detach().cpu().numpy()


def wide_matrix(N, K, spread):
    """Complex entries over 2^-spread .. 2^spread of 1, zeros and the smallest and largest floats among them."""
    rng = np.random.default_rng((N, K, spread))
    re, im = (rng.standard_normal((N, K)) * np.exp2(rng.uniform(-spread, spread, (N, K))) for _ in range(2))
    M = (re + 1j * im).astype(np.complex64)
    flat = M.reshape(-1)
    for i, v in enumerate((0, complex(-0.0, 0.0), 2.0 ** -149, 2.0 ** -149 * 1j, 2.0 ** 120, 1 + 1j, -1 + 1j)):
        if spread > 20:
            flat[(37 * i + 11) % flat.size] = v
    return M


# ---------------------------------------------------- exact axis scales ---
# spread 60: most values lie outside the fixed-point window of their wave and
# take the limbs in LDS; leading zero rows: the window is placed late.

@pytest.mark.parametrize("spread", [0, 20, 60])
@pytest.mark.parametrize("N,K,T,zero_rows", [(5, 20, 4, 0), (33, 260, 2, 0), (64, 512, 3, 40)])
def test_quantize_value_ranges(gpu, N, K, T, zero_rows, spread):
    import paper_2512_02901_amd as f2
    M = wide_matrix(N, K, spread)
    M[:zero_rows] = 0
    codes, scales = oracle.quantize(M, T)
    c, s = f2.quantize(dev(M, gpu), T)
    np.testing.assert_array_equal(host(s).view(np.uint32), scales.view(np.uint32))
    np.testing.assert_array_equal(host(c), oracle.pack(codes))


@pytest.mark.parametrize("K,T", [(1023, 1), (1024, 2), (1025, 3), (2047, 2), (2048, 4), (2049, 2)])
def test_quantize_round_edges(gpu, K, T):
    """256 rows of 4 K entries: one byte and two (a round) for each of the full
    grid's 262144 threads, a row short of them and a row past."""
    import paper_2512_02901_amd as f2
    M = wide_matrix(256, 4 * K, 10)
    codes, scales = oracle.quantize(M, T)
    c, s = f2.quantize(dev(M, gpu), T)
    np.testing.assert_array_equal(host(s).view(np.uint32), scales.view(np.uint32))
    np.testing.assert_array_equal(host(c), oracle.pack(codes))


def test_quantize_many_values_a_lane(gpu):
    """2^28 + 2^20 entries: a lane's sums pass through a flush.  All entries
    have the same two magnitudes, so the scales are those exactly."""
    import torch
    import paper_2512_02901_amd as f2
    N, K = 32896, 8192
    M = torch.full((N, K), 0.7109375 - 0.01j, dtype=torch.complex64, device=gpu)
    M[:, ::3] = 0.02 + 0.33j
    codes, scales = f2.quantize(M, 1)
    assert scales.tolist() == [[0.7109375, float(np.float32(0.33))]]
    want = torch.zeros(K, dtype=torch.uint8, device=gpu)
    want[::3] = 1
    want = want.view(-1, 4) << torch.tensor([0, 2, 4, 6], dtype=torch.uint8, device=gpu)
    assert bool((codes[0] == want.sum(1, dtype=torch.uint8)).all())


# every lane count per group, one to four bytes a lane, the long-group kernel; ragged last groups
@pytest.mark.parametrize("G,K", [(4, 20), (8, 52), (12, 100), (32, 100), (64, 260), (128, 300), (256, 776),
                                 (512, 1156), (1020, 2044), (1024, 1028), (1028, 2200)])
@pytest.mark.parametrize("spread,off", [(1, 0), (60, 1)])
def test_quantize_grouped_edges(gpu, G, K, spread, off):
    import torch
    import paper_2512_02901_amd as f2
    N, T = 7, 3
    M = wide_matrix(N, K, spread)
    codes, scales = og.quantize_grouped(M, T, G)
    buf = torch.empty(N * K + off, dtype=torch.complex64, device=gpu)  # off = 1: 8 bytes off 16-byte alignment
    buf[off:] = dev(M, gpu).reshape(-1)
    c, s = f2.quantize_grouped(buf[off:].view(N, K), T, G)
    np.testing.assert_array_equal(host(s).view(np.uint32), scales.view(np.uint32))
    np.testing.assert_array_equal(host(c), oracle.pack(codes))


# ------------------------------------------------- training-step kernels ---
# nbytes = N K / 4 around a chunk of the two straight-through passes (2048 and
# 1024 code bytes), and one with more chunks than blocks would take at once

@pytest.mark.parametrize("N,K,T", [(1, 4, 1), (1, 4, 4), (3, 1364, 3), (1, 4096, 2), (1, 4100, 4), (2, 8192, 2),
                                   (5, 8196, 3), (2100, 2048, 2)])
def test_ste_backward_edges(gpu, N, K, T):
    import paper_2512_02901_amd as f2
    rng = np.random.default_rng(N + K + T)
    codes = rng.integers(0, 4, (T, N, K))
    scales = (0.3 * np.exp2(-np.arange(T))[:, None] * rng.uniform(0.9, 1.1, (T, 2))).astype(np.float32)
    G = (rng.standard_normal((N, K)) + 1j * rng.standard_normal((N, K))).astype(np.complex64)
    want = oq.ste_backward(codes, scales, G.astype(np.complex128))
    got = host(f2.qat_ste_backward(dev(oracle.pack(codes), gpu), dev(scales, gpu), dev(G, gpu)))
    # double sums and recursion, one rounding to float32
    assert np.linalg.norm(got - want) <= 1e-7 * np.linalg.norm(want)


@pytest.mark.parametrize("n,off", [(1, 0), (7, 0), (8, 0), (9, 0), (4099, 0), (4096, 1), (1 << 20, 0)])
def test_f32_to_bf16_edges(gpu, n, off):
    import torch
    import paper_2512_02901_amd as f2
    rng = np.random.default_rng(n)
    x = torch.from_numpy(rng.standard_normal(n + off).astype(np.float32))
    x[off] = float("inf")
    got = f2.f32_to_bf16(x.to(gpu)[off:])
    assert torch.equal(got.cpu().view(torch.int16), x[off:].to(torch.bfloat16).view(torch.int16))


@pytest.mark.parametrize("N,K,T", [(1, 4, 1), (3, 20, 2), (5, 1364, 1), (40, 2048, 2), (3, 20, 3)])
def test_realify_codes_edges(gpu, N, K, T):
    """R from the codes equals R from the float64 sums rounded once (bf16 of
    the exact sum: the sums of a few float32 scales are exact in double)."""
    import torch
    import paper_2512_02901_amd as f2
    rng = np.random.default_rng(N + K + T)
    cu, cw = rng.integers(0, 4, (2, T, N, K))
    su, sw = (0.02 * np.exp2(-np.arange(T))[None, :, None] * rng.uniform(0.9, 1.1, (2, T, 2))).astype(np.float32)
    U, W = oracle.dequantize(cu, su), oracle.dequantize(cw, sw)
    want = np.empty((N, 2, K, 2))
    want[:, 0, :, 0], want[:, 0, :, 1] = U.real + W.real, W.imag - U.imag
    want[:, 1, :, 0], want[:, 1, :, 1] = U.imag + W.imag, U.real - W.real
    R = f2.wl_realify_codes(*(dev(a, gpu) for a in (oracle.pack(cu), su, oracle.pack(cw), sw)))
    got = R.float().cpu().numpy().reshape(N, 2, K, 2).astype(np.float64)
    assert np.all(np.abs(got - want) <= np.abs(want) * 2.0 ** -8)  # half a bf16 step
    assert torch.isfinite(R).all()


# ------------------------------------------- one-launch products of a layer ---
# rows and tokens around the 16 x 16 block, K around the 256-code steps and
# the 64-code groups, fewer steps than waves and more; every T

def layer(N, K, T, gpu, seed=0):
    rng = np.random.default_rng((N, K, T, seed))
    cu, cw = rng.integers(0, 4, (2, T, N, K))
    su, sw = (0.02 * np.exp2(-np.arange(T))[None, :, None] * rng.uniform(0.9, 1.1, (2, T, 2))).astype(np.float32)
    return (cu, su, cw, sw), tuple(dev(a, gpu) for a in (oracle.pack(cu), su, oracle.pack(cw), sw)), rng


def offset_copy(t, off):
    """The same values `off` elements past an aligned address."""
    import torch
    buf = torch.empty(t.numel() + off, dtype=t.dtype, device=t.device)
    buf[off:] = t.reshape(-1)
    return buf[off:].view(t.shape)


SPLIT_SIZES = [(1, 64, 1), (15, 192, 2), (16, 256, 3), (17, 320, 16), (33, 2112, 17), (40, 5504, 33), (16, 1024, 47)]


@pytest.mark.parametrize("T", [1, 2, 3, 4])
@pytest.mark.parametrize("N,K,B", SPLIT_SIZES)
def test_int8_layer_edges(gpu, N, K, B, T):
    import paper_2512_02901_amd as f2
    (cu, su, cw, sw), d, rng = layer(N, K, T, gpu)
    q = rng.integers(-127, 128, (B, K, 2)).astype(np.int8)
    f = rng.uniform(0.001, 0.02, B).astype(np.float32)
    P = oracle.int8_accumulators(cu, cw, q)
    for off in (0, 2):  # 2 bytes off: byte loads
        dq = offset_copy(dev(q, gpu), off)
        np.testing.assert_array_equal(host(f2.int8_accumulators(d[0], d[2], dq)), P)
        y = host(f2.wl_matmul(*d, dq, dev(f, gpu)))
        want = oracle.combine_accumulators(P, su, sw, f)
        # exact integers, double sums, one rounding
        assert np.linalg.norm(y - want) <= 1e-7 * np.linalg.norm(want)


@pytest.mark.parametrize("T", [1, 2, 3, 4])
@pytest.mark.parametrize("N,K,B", [(n, k, min(b, 16)) for n, k, b in SPLIT_SIZES])
def test_bf16_layer_edges(gpu, N, K, B, T):
    import torch
    import paper_2512_02901_amd as f2
    (cu, su, cw, sw), d, rng = layer(N, K, T, gpu)
    x = synth.bf16_round_complex(rng.standard_normal((B, K)) + 1j * rng.standard_normal((B, K)))
    x[B // 2] *= 0  # a token of zeros
    xd = dev(np.stack([x.real, x.imag], -1).astype(np.float32), gpu).to(torch.bfloat16)
    want = oracle.wl_matmul(cu, su, cw, sw, x)
    for off in (0, 1):
        y = host(f2.wl_matmul(*d, offset_copy(xd, off)))
        # values within 2^14 of the largest are exact in 23 bits, the rest off by 2^-23 of it at most
        assert np.linalg.norm(y - want) <= 3e-7 * np.linalg.norm(want)
        assert not y[B // 2].any()


# either side of the lines between the one launch and the launches that it
# replaces: many rows, long K, tokens against the prefill GEMM

@pytest.mark.parametrize("dt,T,N,K,B", [
    ("bf16", 1, 24576, 64, 1), ("bf16", 1, 24592, 64, 1), ("bf16", 4, 5600, 64, 16), ("bf16", 4, 5616, 64, 16),
    ("bf16", 2, 16, 16384, 1), ("bf16", 2, 272, 16448, 1), ("bf16", 3, 32, 33024, 2), ("bf16", 2, 30, 32768, 2),
    ("i8", 1, 16384, 64, 3), ("i8", 1, 16400, 64, 3), ("i8", 4, 33, 5504, 4), ("i8", 4, 33, 5696, 4),
    ("i8", 4, 4112, 64, 2), ("i8", 4, 32, 8256, 16), ("i8", 3, 17, 16128, 1), ("i8", 3, 17, 16384, 1),
    ("i8", 2, 272, 16640, 4), ("i8", 2, 16, 16640, 4), ("i8", 3, 16384, 64, 32), ("i8", 2, 8192, 64, 17),
    ("i8", 4, 4096, 256, 33), ("i8", 2, 7680, 320, 48), ("i8", 3, 7680, 320, 48),
    # one block a CU and a few more, short and long rows
    ("bf16", 3, 4112, 2048, 1), ("bf16", 3, 4112, 4096, 1), ("bf16", 4, 4112, 8192, 2), ("i8", 3, 4112, 5504, 2),
    ("i8", 3, 4112, 8192, 4)])
def test_layer_launch_lines(gpu, dt, T, N, K, B):
    import torch
    import paper_2512_02901_amd as f2
    (cu, su, cw, sw), d, rng = layer(N, K, T, gpu)
    if dt == "i8":
        q = rng.integers(-127, 128, (B, K, 2)).astype(np.int8)
        f = rng.uniform(0.001, 0.02, B).astype(np.float32)
        y = host(f2.wl_matmul(*d, dev(q, gpu), dev(f, gpu)))
        want = oracle.wl_matmul_int8(cu, su, cw, sw, q, f)
        tol = 1e-6  # exact integers; the GEMM combines its axis sums in float32
    else:
        x = synth.bf16_round_complex(rng.standard_normal((B, K)) + 1j * rng.standard_normal((B, K)))
        xd = dev(np.stack([x.real, x.imag], -1).astype(np.float32), gpu).to(torch.bfloat16)
        y = host(f2.wl_matmul(*d, xd))
        want = oracle.wl_matmul(cu, su, cw, sw, x)
        tol = 3e-7  # 23 bits of the token's largest magnitude
    assert np.linalg.norm(y - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("B,K,off", [(1, 4, 0), (3, 2048, 0), (2, 8192, 0), (2, 8196, 0), (5, 1500, 1), (2, 6, 0),
                                     (3, 252, 0), (2, 256, 0), (3, 260, 0), (2, 512, 0), (3, 516, 0), (2, 1024, 0),
                                     (3, 1028, 0)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_act_quant_edges(gpu, B, K, off, dt):
    """Around the eight-value groups, the widths of the thread blocks and the
    most that one keeps in registers; misaligned tokens and odd widths go one
    value at a time."""
    import torch
    import paper_2512_02901_amd as f2
    rng = np.random.default_rng(K)
    x = synth.bf16_round_complex(rng.standard_normal((B, K)) + 1j * rng.standard_normal((B, K)))
    x[B - 1, 1:] = 0
    q, f = oracle.quantize_act_int8(x)
    xd = dev(x, gpu) if dt == "f32" else dev(np.stack([x.real, x.imag], -1).astype(np.float32), gpu).to(torch.bfloat16)
    gq, gf = f2.quantize_act_int8(offset_copy(xd, off))
    np.testing.assert_array_equal(host(gq), q)
    np.testing.assert_array_equal(host(gf), f)


# --------------------------------------- float activations, vector units ---
# rows around the four of a block, every token group, K around the 1024 codes
# that a block's lanes take at once

@pytest.mark.parametrize("T", [1, 2, 3, 4])
@pytest.mark.parametrize("N,K,B", [(1, 4, 1), (3, 20, 2), (4, 1024, 3), (5, 1028, 4), (9, 1500, 5), (2, 2100, 7), (6, 100, 16)])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_float_layer_edges(gpu, N, K, B, T, dt):
    import torch
    import paper_2512_02901_amd as f2
    if dt == "bf16" and K % 64 == 0:
        pytest.skip("the matrix cores take it")
    (cu, su, cw, sw), d, rng = layer(N, K, T, gpu)
    x = (rng.standard_normal((B, K)) + 1j * rng.standard_normal((B, K))).astype(np.complex64)
    if dt == "bf16":
        x = synth.bf16_round_complex(x)
    xd = dev(x, gpu) if dt == "f32" else dev(np.stack([x.real, x.imag], -1).astype(np.float32), gpu).to(torch.bfloat16)
    want = oracle.wl_matmul(cu, su, cw, sw, x)
    # float32 sums of up to 4 K / 256 products a lane, then a tree: each term
    # rounded at most 4 K / 256 + 10 times, against the 2-norm of the terms
    R = np.abs(oracle.dequantize(cu, su)) + np.abs(oracle.dequantize(cw, sw))
    bound = 2.0 ** -24 * (K / 64 + 14) * np.linalg.norm(np.abs(x) @ R.T)
    for off in (0, 1):
        y = host(f2.wl_matmul(*d, offset_copy(xd, off)))
        assert np.linalg.norm(y - want) <= bound
        np.testing.assert_array_equal(y, host(f2.wl_matmul(*d, offset_copy(xd, off))))


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_float_layer_not_finite(gpu, bad):
    """An infinite real part reaches only the component that its code's axis
    feeds (T = 1: one code of U and one of W); an undefined one likewise."""
    import paper_2512_02901_amd as f2
    N, K = 7, 20
    (cu, su, cw, sw), d, rng = layer(N, K, 1, gpu)
    x = (rng.standard_normal((2, K)) + 1j * rng.standard_normal((2, K))).astype(np.complex64)
    x.real[1, 13] = bad
    y = host(f2.wl_matmul(*d, dev(x, gpu)))
    odd_u, odd_w = cu[0, :, 13] & 1 == 1, cw[0, :, 13] & 1 == 1
    assert np.isfinite(y[0]).all()
    # Re x feeds Re y through the real axis (even codes), Im y through the imaginary one
    np.testing.assert_array_equal(np.isfinite(y[1].real), odd_u & odd_w)
    np.testing.assert_array_equal(np.isfinite(y[1].imag), ~odd_u & ~odd_w)


@pytest.mark.parametrize("dt,B", [("bf16", 1), ("bf16", 3), ("i8", 16), ("i8", 40), ("group", 1), ("group", 4)])
def test_outputs_over_tokens(gpu, dt, B):
    """Outputs written over the tokens' own memory: such calls read every token
    before they write (the one-launch kernels, which do not, leave them to the
    launches that do)."""
    import torch
    import paper_2512_02901_amd as f2
    N, K, T = 512, 1024, 2
    rng = np.random.default_rng((95, B))
    cu, cw = (dev(rng.integers(0, 256, (T, N, K // 4)).astype(np.uint8), gpu) for _ in range(2))
    su, sw = (dev(rng.uniform(0.01, 0.02, (T, 2)).astype(np.float32), gpu) for _ in range(2))
    x = torch.from_numpy(rng.standard_normal((B, K, 2)).astype(np.float32)).to(gpu).to(torch.bfloat16)
    xs = None
    if dt == "i8":
        x, xs = f2.quantize_act_int8(x)
    if dt == "group":
        cu, cw = f2.repack_tiled_fp4(cu), f2.repack_tiled_fp4(cw)

    def product(tokens, y):
        if dt == "group":
            f2.WlGroup([(cu, su, cw, sw, tokens, None, y)], T=T, B=B, layout=f2.LAYOUT_TILED_FP4).run()
        else:
            f2.wl_matmul(cu, su, cw, sw, tokens, xs, out=y)
        return host(y)

    want = product(x, torch.empty((B, N), dtype=torch.complex64, device=gpu))
    raw = torch.empty(8 * B * N, dtype=torch.uint8, device=gpu)  # as many bytes as bf16 tokens take
    mem = raw.view(torch.complex64).view(B, N)
    tokens = raw[:x.numel() * x.element_size()].view(x.dtype).view(x.shape)
    tokens.copy_(x)
    got = product(tokens, mem)
    assert np.linalg.norm(got - want) <= 1e-6 * np.linalg.norm(want)


@pytest.mark.parametrize("B", [1, 16])
def test_outputs_over_token_factors(gpu, B):
    """Outputs written over the int8 tokens' factors: read before as well, up to
    16 tokens."""
    import torch
    import paper_2512_02901_amd as f2
    N, K, T = 512, 1024, 2
    rng = np.random.default_rng((96, B))
    w = []
    for _ in range(2):
        w += [dev(rng.integers(0, 256, (T, N, K // 4)).astype(np.uint8), gpu),
              dev(rng.uniform(0.01, 0.02, (T, 2)).astype(np.float32), gpu)]
    q, xs = f2.quantize_act_int8(dev((rng.standard_normal((B, K)) + 1j * rng.standard_normal((B, K))).astype(np.complex64), gpu))
    want = host(f2.wl_matmul(*w, q, xs))
    for first in (0, 2 * B * N - B):  # the factors at the start and at the end of the outputs
        y = torch.empty((B, N), dtype=torch.complex64, device=gpu)
        factors = torch.view_as_real(y).view(-1)[first:first + B]
        factors.copy_(xs)
        got = host(f2.wl_matmul(*w, q, factors, out=y))
        assert np.linalg.norm(got - want) <= 1e-6 * np.linalg.norm(want)


@pytest.mark.parametrize("T", [1, 2, 3, 4])
@pytest.mark.parametrize("B", [2, 5])
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_float_layer_infinity_values(gpu, dt, B, T):
    """One infinite activation: every other token of its block keeps the values
    of a finite call, and its own token's outputs are those plus the terms
    +-s infinity that the codes of that column give (opposite ones: undefined)."""
    import torch
    import paper_2512_02901_amd as f2
    N, K, col = 7, 20, 13
    (cu, su, cw, sw), d, rng = layer(N, K, T, gpu)
    x = synth.bf16_round_complex(rng.standard_normal((B, K)) + 1j * rng.standard_normal((B, K))).astype(np.complex64)
    bad = B - 2
    x.real[bad, col] = 0
    want = oracle.wl_matmul(cu, su, cw, sw, x)
    R = np.abs(oracle.dequantize(cu, su)) + np.abs(oracle.dequantize(cw, sw))
    bound = 2.0 ** -24 * (K / 64 + 14) * (np.abs(x) @ R.T)
    # Re x enters Re y through codes +-1 and Im y through +-i, of both matrices
    inf = np.zeros((N, 2))
    with np.errstate(invalid="ignore"):
        for c in (cu, cw):
            for t in range(T):
                k = c[t, :, col].astype(int)
                inf[np.arange(N), k & 1] += np.where(k & 2, -np.inf, np.inf)
    x.real[bad, col] = np.inf
    xd = dev(x, gpu) if dt == "f32" else dev(np.stack([x.real, x.imag], -1).astype(np.float32), gpu).to(torch.bfloat16)
    y = host(f2.wl_matmul(*d, xd))
    for b in range(B):
        for part, (g, w) in enumerate(((y[b].real, want[b].real), (y[b].imag, want[b].imag))):
            e = inf[:, part] if b == bad else np.zeros(N)
            fin = e == 0
            assert (np.abs(g - w)[fin] <= bound[b][fin]).all()
            np.testing.assert_array_equal(g[~fin], e[~fin])


def one_launch_calls(gpu, seed):
    """(name, inputs, call) of the one-launch routes and the table kernel; a call
    writes the same outputs each time."""
    import torch
    import paper_2512_02901_amd as f2
    g = torch.Generator(device=gpu)
    g.manual_seed(seed)

    def weights(T, N, K):
        return [t for _ in range(2) for t in
                (torch.randint(0, 256, (T, N, K // 4), generator=g, device=gpu, dtype=torch.uint8),
                 0.01 + 0.01 * torch.rand((T, 2), generator=g, device=gpu))]

    def out(B, N):
        return torch.empty((B, N), dtype=torch.complex64, device=gpu)

    def layer_call(T, N, K, x, xs=None):
        w, y = weights(T, N, K), out(x.shape[0], N)
        dt = f2.ACT_I8 if xs is not None else f2.ACT_BF16 if x.dtype == torch.bfloat16 else f2.ACT_F32
        ws = torch.empty(max(1, f2.wl_matmul_workspace_bytes(N, K, T, x.shape[0], dt)), dtype=torch.uint8, device=gpu)
        return lambda: f2.wl_matmul(*w, x, xs, out=y, workspace=ws)

    def bf16(B, K):
        return torch.randn((B, K, 2), generator=g, device=gpu).to(torch.bfloat16)

    calls = []
    x = bf16(3, 1024)
    calls.append(("bf16", x, layer_call(2, 272, 1024, x)))
    q, xs = f2.quantize_act_int8(bf16(40, 1024))
    calls.append(("int8", xs, layer_call(2, 272, 1024, q, xs)))
    z = torch.view_as_complex(torch.randn((3, 500, 2), generator=g, device=gpu))
    calls.append(("table", z, layer_call(3, 130, 500, z)))
    t = bf16(4, 1024)
    layers = []
    for N in (272, 512):
        cu, su, cw, sw = weights(2, N, 1024)
        layers.append((f2.repack_tiled_fp4(cu), su, f2.repack_tiled_fp4(cw), sw, t, None, out(4, N)))
    plan = f2.WlGroup(layers, T=2, B=4, layout=f2.LAYOUT_TILED_FP4)

    def run():
        plan.run()
        return torch.cat([l[6] for l in layers], 1)
    calls.append(("group", t, run))
    return calls


def test_one_launch_under_capture(gpu):
    """A captured call, replayed with other tokens in the same memory and eager
    work between the replays, gives what the eager call gives."""
    import torch
    for name, x, call in one_launch_calls(gpu, 31):
        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            y = call()
        for i in range(3):
            x.copy_(x.roll(1, -1) if name == "int8" else x.roll(7 + i, 1))
            want = call().clone()
            y.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, want), (name, i)


def test_one_launch_from_two_threads(gpu):
    """Two threads, each on a stream of its own with its own operands."""
    import threading
    import torch
    calls = [one_launch_calls(gpu, 41), one_launch_calls(gpu, 42)]
    want = [[call().clone() for _, _, call in c] for c in calls]
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream(gpu)) as _:
                for _ in range(20):
                    for (name, _, call), w in zip(calls[i], want[i]):
                        if not torch.equal(call(), w):
                            wrong.append((i, name))
        except Exception as e:  # an assertion in a thread would be lost
            wrong.append((i, repr(e)))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong


@pytest.mark.parametrize("N,K,T,B", [(256, 260, 1, 4), (130, 1500, 2, 3), (67, 5508, 3, 16), (33, 16388, 4, 5), (5, 12, 2, 1)])
def test_bf16_layer_rounded_once(gpu, N, K, T, B):
    """bf16 tokens off the matrix cores: 8-bit significands times sums of scales,
    in double, so the output's rounding to float32 is the error (2^-24 a value)."""
    import torch
    import paper_2512_02901_amd as f2
    (cu, su, cw, sw), d, rng = layer(N, K, T, gpu)
    x = synth.bf16_round_complex(rng.standard_normal((B, K)) + 1j * rng.standard_normal((B, K)))
    xd = dev(np.stack([x.real, x.imag], -1).astype(np.float32), gpu).to(torch.bfloat16)
    want = x.astype(np.complex128) @ oracle.dequantize(cu, su).astype(np.complex128).T
    want += np.conj(x).astype(np.complex128) @ oracle.dequantize(cw, sw).astype(np.complex128).T
    y = host(f2.wl_matmul(*d, xd)).astype(np.complex128)
    for g, w in ((y.real, want.real), (y.imag, want.imag)):
        assert (np.abs(g - w) <= 2.0 ** -24 * np.abs(w) + 2.0 ** -46 * np.abs(want).max()).all()
