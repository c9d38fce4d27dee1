"""Performance cases of the widely-linear layer library: single layers from the
smallest to LLaMA-2-7B's, grouped decode of whole stacks, prefill, one decoder
block, the offline quantiser and a training step, each through the public
entry points of ``paper_2512_02901_amd``.

A case is a dict of plain values; ``kind`` selects the path:

layer     wl_matmul on one layer (codes as the quantiser writes them), into an
          output and a workspace that the caller keeps.  With ``act`` "i8" the
          pass starts from bf16 activations and quantises them first.
group     WlGroup.run over ``blocks`` decoder blocks' projections (``parts``:
          "all" seven, "qkv" or "gate_up") in the fp4 tiled layout; the outputs
          of all layers of one width share a buffer [layers, B, N].
block     WlBlock.decode of one token at position ``ctx`` - 1.
quantize  to_widely_linear, quantize (or quantize_grouped) of U and W and, for
          per-tensor scales, their repacking for decode.
qat       one training step of a layer: quantise both masters, the three
          products in the real form, the straight-through gradients.

N and K are complex dimensions (the real layer is 2N x 2K).
"""
import math

import torch

import paper_2512_02901_amd as f2

MAX_COST = 2 * 5504 * 2048 * 2048  # stages * N * K * tokens of the largest listed prefill


def listed():
    return [
        # a 256 x 256 layer, one float32 token: launch and host latency only
        dict(name="layer_256_f32", kind="layer", T=2, N=128, K=128, B=1, act="f32"),
        # one attention projection for one decode token, plain call
        dict(name="layer_q_bf16_b1", kind="layer", T=2, N=2048, K=2048, B=1, act="bf16"),
        # the down projection for a decode batch with int8 activations
        dict(name="layer_down_i8_b16", kind="layer", T=2, N=2048, K=5504, B=16, act="i8"),
        # a width that no power of two divides (3000 real inputs), float32 tokens, three stages
        dict(name="layer_odd_f32_b5", kind="layer", T=3, N=1001, K=1500, B=5, act="f32"),
        # a short prompt (or a large decode batch) through the down projection
        dict(name="prefill_down_77", kind="layer", T=2, N=2048, K=5504, B=77, act="i8"),
        # a 2048-token prompt through the gate projection
        dict(name="prefill_gate_2048", kind="layer", T=2, N=5504, K=2048, B=2048, act="i8"),
        # every projection of LLaMA-2-7B for one decode token
        dict(name="stack_b1", kind="group", parts="all", blocks=32, n=2048, n_ff=5504, T=2, B=1, G=0),
        # the same for the largest decode batch
        dict(name="stack_b16", kind="group", parts="all", blocks=32, n=2048, n_ff=5504, T=2, B=16, G=0),
        # q, k, v of one decoder block with per-group scales, a small decode batch
        dict(name="qkv_group256_b4", kind="group", parts="qkv", blocks=1, n=2048, n_ff=5504, T=2, B=4, G=256),
        # one decode token through one decoder block after 2047 others
        dict(name="block_ctx2048", kind="block", n=2048, n_ff=5504, heads=32, ctx=2048, T=2),
        # offline conversion of one attention projection
        dict(name="quantize_q", kind="quantize", N=2048, K=2048, T=2, G=0),
        # one training step of an attention projection, 4096 tokens
        dict(name="qat_q_4096", kind="qat", N=2048, K=2048, T=2, tokens=4096),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _stages(rng, most=4):
    return min(most, rng.choice((1, 2, 2, 2, 3, 4)))


def draw(rng):
    kind = rng.choice(("layer", "layer", "layer", "prefill", "prefill", "prefill", "group", "group", "block",
                       "quantize", "qat"))
    if kind in ("layer", "prefill"):
        step = rng.choice((4, 64, 64))
        N = rng.choice((2048, 5504, _log(rng, 64, 5504), _log(rng, 64, 5504)))
        K = rng.choice((2048, 5504, 0, 0)) or -(-_log(rng, 64, 5504) // step) * step
        T = _stages(rng)
        if kind == "layer":
            return dict(kind="layer", T=T, N=N, K=K, B=_log(rng, 1, 16), act=rng.choice(("f32", "bf16", "bf16", "i8")))
        top = max(17, min(2048, MAX_COST // (T * N * K)))
        return dict(kind="layer", T=T, N=N, K=K, B=_log(rng, 17, top), act="i8")
    if kind == "group":
        T = _stages(rng)
        parts = rng.choice(("all", "qkv", "gate_up"))
        G = rng.choice((0, 0, 256, 512, 1024))
        most = 16 if T <= 2 else 8 if T == 3 else 4
        return dict(kind="group", parts=parts, blocks=_log(rng, 1, 16 if G else 32 * 2 // max(T, 2)),
                    n=64 * _log(rng, 8, 32), n_ff=64 * _log(rng, 16, 86), T=T, B=_log(rng, 1, most), G=G)
    if kind == "block":
        heads = rng.choice((8, 16, 32))
        return dict(kind="block", n=64 * heads, n_ff=64 * _log(rng, 16, 86), heads=heads, ctx=_log(rng, 1, 4096),
                    T=_stages(rng))
    if kind == "quantize":
        return dict(kind="quantize", N=_log(rng, 64, 2752), K=4 * _log(rng, 16, 512), T=_stages(rng),
                    G=rng.choice((0, 0, 64, 256)))
    return dict(kind="qat", N=8 * _log(rng, 16, 256), K=8 * _log(rng, 16, 256), T=_stages(rng),
                tokens=_log(rng, 128, 4096))


# ---------------------------------------------------------------- inputs ---

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _codes(g, T, N, K):
    return torch.randint(0, 256, (T, N, K // 4), generator=g, device="cuda", dtype=torch.uint8)


def _scales(g, shape):
    """Axis scales of a residual recursion (each stage about 0.55 of the one
    before); shape [T, ..., 2]."""
    s = 0.016 * (0.9 + 0.2 * torch.rand(shape, generator=g, device="cuda"))
    decay = 0.55 ** torch.arange(shape[0], device="cuda", dtype=torch.float32)
    return (s * decay.view(-1, *[1] * (len(shape) - 1))).contiguous()


def _weights(g, T, N, K, G=0):
    sshape = (T, 2) if G == 0 else (T, N, -(-K // G), 2)
    cu, cw = _codes(g, T, N, K), _codes(g, T, N, K)
    return cu, _scales(g, sshape), cw, _scales(g, sshape)


def _tokens(g, B, K, channels=0.01, gain=8.0):
    """[B, K, 2] float32 activations: N(0, 1), with about 1 % of the channels 8 times as large."""
    x = torch.randn((B, K, 2), generator=g, device="cuda")
    big = torch.rand((1, K, 1), generator=g, device="cuda") < channels
    return torch.where(big, x * gain, x)


def _layer_inputs(c, seed):
    g = _gen(seed)
    w = _weights(g, c["T"], c["N"], c["K"])
    x = _tokens(g, c["B"], c["K"])
    x = torch.view_as_complex(x).contiguous() if c["act"] == "f32" else x.to(torch.bfloat16)
    return w, x


def _group_shapes(c):
    n, f = c["n"], c["n_ff"]
    parts = {"all": [(n, n)] * 4 + [(f, n)] * 2 + [(n, f)], "qkv": [(n, n)] * 3, "gate_up": [(f, n)] * 2}[c["parts"]]
    return parts * c["blocks"]


def _group_inputs(c, seed):
    """(N, weights, bf16 tokens) layer by layer."""
    g = _gen(seed)
    for N, K in _group_shapes(c):
        yield N, _weights(g, c["T"], N, K, c["G"]), _tokens(g, c["B"], K).to(torch.bfloat16)


def _block_inputs(c, seed):
    g = _gen(seed)
    n, f, H = c["n"], c["n_ff"], c["heads"]
    shapes = {"q": (n, n), "k": (n, n), "v": (n, n), "o": (n, n), "gate": (f, n), "up": (f, n), "down": (n, f)}
    w = {name: _weights(g, c["T"], N, K) for name, (N, K) in shapes.items()}
    norms = [1.0 + 0.1 * torch.randn(2 * n, generator=g, device="cuda") for _ in range(2)]
    x = torch.view_as_complex(torch.randn((1, n, 2), generator=g, device="cuda"))
    caches = [torch.view_as_complex(torch.randn((H, c["ctx"], n // H, 2), generator=g, device="cuda"))
              for _ in range(2)]
    return w, norms, x, caches


def _master(g, N, K):
    """Complex master weights with the tails of a trained matrix (Student-t,
    4 degrees of freedom, standard deviation 0.02 / sqrt(2) a component)."""
    z = torch.randn((N, K, 2), generator=g, device="cuda")
    v = sum(torch.randn((N, K, 2), generator=g, device="cuda") ** 2 for _ in range(4))
    return torch.view_as_complex(z * torch.rsqrt(v / 4) * 0.01)


def _quantize_input(c, seed):
    g = _gen(seed)
    z = torch.randn((2 * c["N"], 2 * c["K"]), generator=g, device="cuda")
    v = sum(torch.randn(z.shape, generator=g, device="cuda") ** 2 for _ in range(4))
    A = z * torch.rsqrt(v / 4) * (0.02 / math.sqrt(2.0))
    big = torch.rand((1, z.shape[1]), generator=g, device="cuda") < 0.01
    return torch.where(big, A * 10.0, A).contiguous()


def _qat_inputs(c, seed):
    g = _gen(seed)
    Mu, Mw = _master(g, c["N"], c["K"]), _master(g, c["N"], c["K"])
    X = torch.randn((c["tokens"], 2 * c["K"]), generator=g, device="cuda").to(torch.bfloat16)
    GY = torch.randn((c["tokens"], 2 * c["N"]), generator=g, device="cuda") * 1e-3
    return Mu, Mw, X, GY


# ------------------------------------------------------------ the passes ---

_DTYPE = {"f32": f2.ACT_F32, "bf16": f2.ACT_BF16, "i8": f2.ACT_I8}


def prepare(case, seed):
    c = case
    if c["kind"] == "layer":
        w, x = _layer_inputs(c, seed)
        y = torch.empty((c["B"], c["N"]), dtype=torch.complex64, device="cuda")
        need = f2.wl_matmul_workspace_bytes(c["N"], c["K"], c["T"], c["B"], _DTYPE[c["act"]])
        return dict(kind="layer", act=c["act"], w=w, x=x, y=y,
                    ws=torch.empty(max(1, need), dtype=torch.uint8, device="cuda"))
    if c["kind"] == "group":
        widths = [N for N, _ in _group_shapes(c)]
        y = {str(N): torch.empty((widths.count(N), c["B"], N), dtype=torch.complex64, device="cuda") for N in widths}
        layers, rows = [], {N: iter(t) for N, t in y.items()}
        for N, (cu, su, cw, sw), x in _group_inputs(c, seed):
            layers.append((f2.repack_tiled_fp4(cu), su, f2.repack_tiled_fp4(cw), sw, x, None, next(rows[str(N)])))
        plan = f2.WlGroup(layers, T=c["T"], B=c["B"], layout=f2.LAYOUT_TILED_FP4, group_size=c["G"])
        return dict(kind="group", plan=plan, y=y)
    if c["kind"] == "block":
        w, norms, x, (k, v) = _block_inputs(c, seed)
        w = {name: (f2.repack_tiled_fp4(cu), su, f2.repack_tiled_fp4(cw), sw) for name, (cu, su, cw, sw) in w.items()}
        blk = f2.WlBlock(w, norms[0], norms[1], c["n"], c["n_ff"], c["heads"], c["T"], c["ctx"])
        return dict(kind="block", blk=blk, x=x, k=k, v=v, pos=c["ctx"] - 1, out=torch.empty_like(x))
    if c["kind"] == "quantize":
        return dict(kind="quantize", A=_quantize_input(c, seed), T=c["T"], G=c["G"])
    Mu, Mw, X, GY = _qat_inputs(c, seed)
    N, K, M = c["N"], c["K"], c["tokens"]
    st = dict(kind="qat", T=c["T"], N=N, K=K, Mu=Mu, Mw=Mw, X=X, GY=GY,
              R=torch.empty((2 * N, 2 * K), dtype=torch.bfloat16, device="cuda"),
              GYb=torch.empty((M, 2 * N), dtype=torch.bfloat16, device="cuda"),
              Y=torch.empty((M, 2 * N), device="cuda"), GX=torch.empty((M, 2 * K), device="cuda"),
              GR=torch.empty((2 * N, 2 * K), device="cuda"),
              GU=torch.empty((N, K), dtype=torch.complex64, device="cuda"),
              GW=torch.empty((N, K), dtype=torch.complex64, device="cuda"),
              ws=torch.empty(f2.load().fairy2i_gemm_bf16_workspace_bytes(), dtype=torch.uint8, device="cuda"))
    # a training program tunes its three products once, before the first step
    st["R"].zero_()
    st["GYb"].zero_()
    f2.gemm_bf16(X, st["R"], transB=True, out=st["Y"], workspace=st["ws"], tune=True)
    f2.gemm_bf16(st["GYb"], st["R"], out=st["GX"], workspace=st["ws"], tune=True)
    f2.gemm_bf16(st["GYb"], X, transA=True, out=st["GR"], workspace=st["ws"], tune=True)
    return st


def run(state):
    s = state
    if s["kind"] == "layer":
        x, xs = f2.quantize_act_int8(s["x"]) if s["act"] == "i8" else (s["x"], None)
        return f2.wl_matmul(*s["w"], x, xs, out=s["y"], workspace=s["ws"])
    if s["kind"] == "group":
        s["plan"].run()
        return s["y"]
    if s["kind"] == "block":
        out = s["blk"].decode(s["x"], s["k"], s["v"], s["pos"], out=s["out"])
        return {"out": out, "k": s["k"], "v": s["v"]}
    if s["kind"] == "quantize":
        U, W = f2.to_widely_linear(s["A"])
        if s["G"]:
            (cu, su), (cw, sw) = (f2.quantize_grouped(M, s["T"], s["G"]) for M in (U, W))
            return {"codes": [cu, cw], "scales": [su, sw]}
        (cu, su), (cw, sw) = (f2.quantize(M, s["T"]) for M in (U, W))
        return {"codes": [cu, cw], "scales": [su, sw], "tiled": [f2.repack_tiled_fp4(cu), f2.repack_tiled_fp4(cw)]}
    (cu, su), (cw, sw) = (f2.quantize(M, s["T"]) for M in (s["Mu"], s["Mw"]))
    R = f2.wl_realify_codes(cu, su, cw, sw, out=s["R"])
    Y = f2.gemm_bf16(s["X"], R, transB=True, out=s["Y"], workspace=s["ws"])
    GYb = f2.f32_to_bf16(s["GY"], out=s["GYb"])
    GX = f2.gemm_bf16(GYb, R, out=s["GX"], workspace=s["ws"])
    GR = f2.gemm_bf16(GYb, s["X"], transA=True, out=s["GR"], workspace=s["ws"])
    GU, GW = f2.wl_unrealify_grad(GR, s["N"], s["K"], out=(s["GU"], s["GW"]))
    return {"Y": Y, "GX": GX, "GMu": f2.qat_ste_backward(cu, su, GU), "GMw": f2.qat_ste_backward(cw, sw, GW)}


def work(case):
    """Each input read once, each output written once; operations: one signed
    add (two operations) per code and real activation component, and the real
    products' multiply-adds in training."""
    c = case
    if c["kind"] == "layer":
        T, N, K, B = c["T"], c["N"], c["K"], c["B"]
        return {"bytes": T * N * K // 2 + 16 * T + B * K * (8 if c["act"] == "f32" else 4) + 8 * B * N,
                "flops": 8 * T * N * K * B}
    if c["kind"] == "group":
        T, B, G = c["T"], c["B"], c["G"]
        b = f = 0
        for N, K in _group_shapes(c):
            b += T * N * K // 2 + 16 * T * (N * -(-K // G) if G else 1) + 4 * B * K + 8 * B * N
            f += 8 * T * N * K * B
        return {"bytes": b, "flops": f}
    if c["kind"] == "block":
        n, ff, T = c["n"], c["n_ff"], c["T"]
        nk = 4 * n * n + 3 * n * ff
        return {"bytes": T * nk // 2 + 16 * n * c["ctx"] + 32 * n, "flops": 8 * T * nk + 8 * n * c["ctx"]}
    N, K, T = c["N"], c["K"], c["T"]
    if c["kind"] == "quantize":
        sb = 16 * T * (N * -(-K // c["G"]) if c["G"] else 1)
        tiled = 0 if c["G"] else T * N * K // 2
        return {"bytes": 16 * N * K + T * N * K // 2 + tiled + sb, "flops": 16 * T * N * K}
    M = c["tokens"]
    return {"bytes": 32 * N * K + 4 * M * K + 8 * M * N + 8 * M * N + 8 * M * K, "flops": 24 * M * N * K}


def tolerance(case):
    """What another order of the same sums gives, about four times over."""
    c = case
    if c["kind"] == "quantize":
        return "exact"
    if c["kind"] == "layer":
        # exact integer sums, or float32 sums of the tokens' own values
        return {"rel": 5e-7 if c["act"] == "i8" else 1e-6, "max": 2e-5}
    if c["kind"] == "group":
        # above four tokens (two at T = 4) one digit pair a value: small
        # products beside a large one may lose their low bits
        one_band = c["B"] > (4 if c["T"] < 4 else 2)
        return {"rel": 1e-4 if one_band else 1e-6, "max": 2e-3 if one_band else 2e-5}
    if c["kind"] == "block":
        # a value next to a bf16 tie may round either way at the layers' inputs
        return {"rel": 4e-3, "max": 4e-2}
    # bf16 operands, float32 sums
    return {"rel": 1e-5, "max": 4e-4}


# --------------------------------------------------- the same in 64 bits ---

def _unpack(codes):
    """uint8 [..., K/4] -> int64 codes [..., K]."""
    shifts = torch.tensor([0, 2, 4, 6], device=codes.device, dtype=torch.uint8)
    return ((codes.unsqueeze(-1) >> shifts) & 3).flatten(-2).long()


def _dense(codes, scales, G=0):
    """The dequantised matrix, complex128 [N, K]."""
    T, N, KB = codes.shape
    out = torch.zeros((N, 4 * KB), dtype=torch.complex128, device=codes.device)
    unit = torch.tensor([1, 1j, -1, -1j], dtype=torch.complex128, device=codes.device)
    for t in range(T):
        k = _unpack(codes[t])
        s = scales[t].double()
        if G:
            s = s.repeat_interleave(G, dim=1)[:, : 4 * KB]
            mag = torch.where(k % 2 == 0, s[..., 0], s[..., 1])
        else:
            mag = torch.where(k % 2 == 0, s[0], s[1])
        out += unit[k] * mag
    return out


def _apply(w, x, G=0):
    """y = U x + W conj(x) for tokens x complex128 [B, K]."""
    cu, su, cw, sw = w
    return x @ _dense(cu, su, G).T + x.conj() @ _dense(cw, sw, G).T


def _complex(x):
    return torch.view_as_complex(x.double().contiguous())


def _rounded(x):
    """complex128 -> its components rounded to bf16, complex128."""
    return torch.view_as_complex(torch.view_as_real(x).to(torch.bfloat16).double())


def _int8(x):
    """The library's int8 activations, by their definition in float32: (q, factor)."""
    g = x.float().abs().amax(dim=(1, 2))
    top = torch.full_like(g, 127.0)  # a tensor: torch divides by and into a scalar through a reciprocal
    inv = torch.where(g > 0, top / g, torch.zeros_like(g))
    q = torch.clamp(torch.round(x.float() * inv.view(-1, 1, 1)), -127, 127)
    return _complex(q), (g / top).double()


def _project(r):
    """Codes of the nearest codeword by angle, ties counter-clockwise."""
    re, im = r.real, r.imag
    k = torch.zeros(r.shape, dtype=torch.long, device=r.device)
    k[(im > 0) & (re <= im) & (re > -im)] = 1
    k[(re < 0) & (im <= -re) & (im > re)] = 2
    k[(im < 0) & (re >= im) & (re < -im)] = 3
    return k


def _axis_means(r, k, G):
    """Per-tensor [2] or per-group [N, groups, 2] axis scales, rounded to float32."""
    out = []
    for on, v in ((k % 2 == 0, r.real), (k % 2 == 1, r.imag)):
        v = torch.where(on, v.abs(), torch.zeros_like(v))
        if G:
            pad = -v.shape[1] % G
            v = torch.nn.functional.pad(v, (0, pad)).view(v.shape[0], -1, G)
            n = torch.nn.functional.pad(on.double(), (0, pad)).view(v.shape).sum(-1)
            out.append(torch.where(n > 0, v.sum(-1) / n.clamp(min=1), torch.zeros_like(n)))
        else:
            n = on.sum()
            out.append(v.sum() / n.clamp(min=1))
    return torch.stack(out, dim=-1).float()


def _phase_quant(M, T, G=0):
    """T residual stages in 64 bits: (codes [T, N, K], scales, the sum of the stages)."""
    r = M.to(torch.complex128)
    unit = torch.tensor([1, 1j, -1, -1j], dtype=torch.complex128, device=r.device)
    codes, scales, total = [], [], torch.zeros_like(r)
    for _ in range(T):
        k = _project(r)
        s = _axis_means(r, k, G)
        wide = s.double().repeat_interleave(G, dim=1)[:, : r.shape[1]] if G else s.double()
        q = unit[k] * torch.where(k % 2 == 0, wide[..., 0], wide[..., 1])
        codes.append(k)
        scales.append(s)
        total += q
        r = r - q
    return torch.stack(codes), torch.stack(scales), total


def _straight_through(codes, scales, g):
    H = torch.zeros_like(g)
    for t in reversed(range(codes.shape[0])):
        k = codes[t]
        b_re = (k == 0).double() - (k == 2).double()
        b_im = (k == 1).double() - (k == 3).double()
        gq = g - H
        d_re = (gq.real * b_re).sum() / (k % 2 == 0).sum().clamp(min=1)
        d_im = (gq.imag * b_im).sum() / (k % 2 == 1).sum().clamp(min=1)
        s = scales[t].double()
        H = H + torch.complex(s[0] * gq.real + b_re * d_re, s[1] * gq.imag + b_im * d_im)
    return H


def _block_exact(c, seed):
    w, (g1, g2), x, (kc, vc) = _block_inputs(c, seed)
    n, H, pos = c["n"], c["heads"], c["ctx"] - 1
    dc = n // H
    x = x.to(torch.complex128)

    def norm(a, gain):
        r = torch.rsqrt(torch.view_as_real(a).square().sum() / (2 * n) + 1e-5)
        return _rounded(torch.complex(a.real * r * gain[:n].double(), a.imag * r * gain[n:].double()))

    z = norm(x, g1)
    turn = pos * 10000.0 ** (-torch.arange(dc, device="cuda", dtype=torch.float64) / dc)
    turn = torch.polar(torch.ones_like(turn), turn)
    q = _apply(w["q"], z).view(H, dc) * turn
    kc, vc = kc.to(torch.complex128), vc.to(torch.complex128)
    kc[:, pos] = _apply(w["k"], z).view(H, dc) * turn
    vc[:, pos] = _apply(w["v"], z).view(H, dc)
    p = torch.softmax((q.conj().unsqueeze(1) * kc).sum(-1).real / math.sqrt(2 * dc), dim=1)
    o = _rounded((p.unsqueeze(-1) * vc).sum(1).reshape(1, n))
    h = x + _apply(w["o"], o)
    z2 = norm(h, g2)
    g, u = _apply(w["gate"], z2), _apply(w["up"], z2)
    act = _rounded(torch.complex(torch.nn.functional.silu(g.real) * u.real, torch.nn.functional.silu(g.imag) * u.imag))
    return {"out": h + _apply(w["down"], act), "k": kc, "v": vc}


def exact(case, seed):
    c = case
    if c["kind"] == "layer":
        w, x = _layer_inputs(c, seed)
        if c["act"] == "i8":
            q, factor = _int8(x)
            return _apply(w, q) * factor.view(-1, 1)
        return _apply(w, x.to(torch.complex128) if c["act"] == "f32" else _complex(x))
    if c["kind"] == "group":
        y = {}
        for N, w, x in _group_inputs(c, seed):
            y.setdefault(str(N), []).append(_apply(w, _complex(x), c["G"]))
        return {N: torch.stack(t) for N, t in y.items()}
    if c["kind"] == "block":
        return _block_exact(c, seed)
    if c["kind"] == "quantize":
        A = _quantize_input(c, seed).double()
        N, K = c["N"], c["K"]
        r11, r12, r21, r22 = A[:N, :K], A[:N, K:], A[N:, :K], A[N:, K:]
        pair = [torch.complex((r11 + r22) / 2, (r21 - r12) / 2), torch.complex((r11 - r22) / 2, (r12 + r21) / 2)]
        scales = [_phase_quant(M.to(torch.complex64), c["T"], c["G"])[1].double() for M in pair]
        return {"codes": [None, None], "scales": scales, **({} if c["G"] else {"tiled": [None, None]})}
    Mu, Mw, X, GY = _qat_inputs(c, seed)
    (ku, su, U), (kw, sw, W) = (_phase_quant(M, c["T"]) for M in (Mu, Mw))
    x = torch.view_as_complex(X.double().view(c["tokens"], -1, 2))
    gy = torch.view_as_complex(GY.double().view(c["tokens"], -1, 2))
    Y = x @ U.T + x.conj() @ W.T
    GX = gy @ U.conj() + gy.conj() @ W
    GU, GW = gy.T @ x.conj(), gy.T @ x
    flat = (torch.view_as_real(a).flatten(1) for a in (Y, GX))
    return {"Y": next(flat), "GX": next(flat), "GMu": _straight_through(ku, su, GU),
            "GMw": _straight_through(kw, sw, GW)}
