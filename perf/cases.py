"""What is measured: the layer steps, the attention products and the weight update as a training or serving program
calls them through paper_2207_08822_amd.fxp, from one-tile layers to the 8192^3 product, aligned and ragged.

Every result of the library is defined bit for bit (the random stream belongs to the element, the sums are integers and
the inverse mapping rounds once), so every case is compared exactly.
"""
import math

import torch

from paper_2207_08822_amd import fxp, synth

# ViT-B tokens of one image; ResNet and ViT sizes below are those of the layers in synth.WORKLOADS and around them
TOKENS = 197


def listed():
    return [
        # the smallest training step (bench workload c1): launches and latency
        dict(name="linear_small", kind="linear", M=256, K=256, N=256),
        # serving: one image through one ViT-B projection, forward only, rounding to nearest, no workspace
        dict(name="linear_serve", kind="serve", M=TOKENS, K=768, N=768),
        # an ordinary large training step: the first MLP layer of ViT-B at batch 64 (c3)
        dict(name="linear_vit", kind="linear", M=64 * TOKENS, K=768, N=3072),
        # the qkv layer of the same block in the middle of a training run: last step's scales at hand as guesses,
        # six of the eight bits of the low-bit ablation
        dict(name="linear_guess", kind="linear", M=64 * TOKENS, K=768, N=2304, guess=True, bits=6),
        # the classifier head over a last, partial batch of seven images: odd rows, 1000 outputs
        dict(name="linear_ragged", kind="linear", M=7 * TOKENS, K=768, N=1000),
        # the largest step (c5)
        dict(name="linear_square", kind="linear", M=8192, K=8192, N=8192),
        # the 3x3 convolution of ResNet-18's second stage (c2conv), forward and both gradients
        dict(name="conv_3x3", kind="conv", N=32, H=28, W=28, C=128, Cout=128, KH=3, KW=3, stride=1, pad=1, need_dX=True),
        # ResNet-18's stem: 7x7, stride 2, three channels; the image needs no gradient
        dict(name="conv_stem", kind="conv", N=32, H=224, W=224, C=3, Cout=64, KH=7, KW=7, stride=2, pad=3, need_dX=False),
        # the downsampling convolution at the head of ResNet-18's third stage
        dict(name="conv_stride", kind="conv", N=32, H=28, W=28, C=128, Cout=256, KH=3, KW=3, stride=2, pad=1, need_dX=True),
        # both attention products of a ViT-B block, batch 64 x 12 heads, tokens padded to 208 (vitb_attn)
        dict(name="attn_padded", kind="attn", batch=768, S=208, real=TOKENS, d=64),
        # the same products as the model has them, 197 tokens unpadded, batch 8
        dict(name="attn_ragged", kind="attn", batch=96, S=TOKENS, real=TOKENS, d=64),
        # the int16 update of ResNet-18's 62 parameter tensors (sgd16_multi)
        dict(name="sgd_resnet18", kind="sgd", width=64, classes=1000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, step=1):
    return max(lo, _log_int(rng, lo, hi) // step * step)


def _options(rng, case):
    """The options a training run really varies: the width of the ablation, now and then."""
    if rng.random() < 0.25:
        case["bits"] = rng.randint(4, 7)
    return case


def draw(rng):
    what = rng.choice(["small", "serve", "vit", "guess", "ragged", "square", "conv", "stem", "stride", "padded", "unpadded",
                       "sgd"])
    if what == "small":
        step = rng.choice([1, 4, 16, 64])
        return _options(rng, dict(kind="linear", M=_size(rng, 32, 512, step), K=_size(rng, 64, 512, step), N=_size(rng, 64, 512, step)))
    if what == "serve":
        return dict(kind="serve", M=_log_int(rng, 1, 512), K=_size(rng, 256, 3072, rng.choice([16, 64, 128])),
                    N=_size(rng, 256, 3072, rng.choice([4, 16, 128])))
    if what in ("vit", "guess"):
        width, wide = rng.choice([(384, 1536), (768, 2304), (768, 3072), (768, 768), (1024, 1024)])
        if rng.random() < 0.5:
            width, wide = wide, width
        case = dict(kind="linear", M=TOKENS * 16 * rng.randint(1, 4), K=width, N=wide)
        if what == "guess":
            case["guess"] = True
        return _options(rng, case)
    if what == "ragged":
        return _options(rng, dict(kind="linear", M=_size(rng, 197, 4096), K=_size(rng, 256, 3072, rng.choice([1, 4, 64])),
                                  N=_size(rng, 64, 3072, rng.choice([1, 2, 8]))))
    if what == "square":
        step = rng.choice([16, 64, 256])
        return dict(kind="linear", M=_size(rng, 1024, 8192, step), K=_size(rng, 1024, 8192, step), N=_size(rng, 1024, 8192, step))
    if what == "conv":
        c, hw = rng.choice([(64, 56), (128, 28), (256, 14), (512, 7)])
        k = rng.choice([1, 3, 3])
        return _options(rng, dict(kind="conv", N=rng.randint(4, 64), H=hw, W=hw, C=c, Cout=c * rng.choice([1, 1, 2]), KH=k, KW=k, stride=1,
                                  pad=k // 2, need_dX=True))
    if what == "stem":
        k = rng.choice([3, 7])
        hw = rng.randint(64, 224)
        return dict(kind="conv", N=rng.randint(4, 32), H=hw, W=hw, C=rng.choice([1, 3, 4]), Cout=rng.choice([32, 64, 96]), KH=k, KW=k,
                    stride=2, pad=k // 2, need_dX=False)
    if what == "stride":
        c, hw = rng.choice([(64, 56), (128, 28), (256, 14), (48, 57)])
        k = rng.choice([1, 3, 3])
        return _options(rng, dict(kind="conv", N=rng.randint(4, 48), H=hw, W=hw, C=c, Cout=2 * c, KH=k, KW=k, stride=2, pad=k // 2,
                                  need_dX=True))
    if what == "padded":
        s = 16 * rng.randint(4, 16)
        return _options(rng, dict(kind="attn", batch=12 * rng.randint(2, 48), S=s, real=s - rng.randint(0, 15), d=64))
    if what == "unpadded":
        s = rng.randint(50, 257)
        return dict(kind="attn", batch=12 * rng.randint(1, 16), S=s, real=s, d=rng.choice([32, 64, 80]))
    return dict(kind="sgd", width=rng.choice([16, 24, 32, 48, 64]), classes=rng.choice([10, 100, 1000]))


def _normal(gen, shape, sigma):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(sigma)


def _laplace(gen, shape, b, outliers):
    """Laplace values, a share of them a thousand times larger: the gradients of the paper's ViT runs."""
    u = torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32).sub_(0.5)
    out = torch.log1p(u.abs().mul_(-2.0).clamp_(min=-1.0 + 1e-7)).mul_(torch.sign(u.sub_(1e-9))).mul_(-b)
    if outliers:
        out[torch.rand(shape, generator=gen, device="cuda") < outliers] *= 1000.0
    return out


def _parameter_sizes(width, classes):
    """Parameter tensors of a ResNet-18 of another stage width and class count (64 and 1000: the ResNet-18)."""
    if (width, classes) == (64, 1000):
        return synth.resnet18_parameter_sizes()
    sizes, cin = [width * 3 * 7 * 7, width, width], width
    for cout in (width, 2 * width, 4 * width, 8 * width):
        for block in range(2):
            c = cin if block == 0 else cout
            sizes += [cout * c * 9, cout, cout, cout * cout * 9, cout, cout]
            if c != cout:
                sizes += [cout * c, cout, cout]
        cin = cout
    return sizes + [classes * 8 * width, classes]


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    st = dict(kind=kind, seed=seed, bits=case.get("bits", 8))
    if kind in ("linear", "serve"):
        M, K, N = case["M"], case["K"], case["N"]
        st["X"] = _normal(gen, (M, K), 1.0)
        st["W"] = _normal(gen, (K, N), 0.02 if M < 8192 or K != N else 1.0)
        if kind == "linear":
            st["dY"] = _laplace(gen, (M, N), 1e-5, 1e-3) if M * N < 1 << 26 else _normal(gen, (M, N), 1.0)
        st["buf"] = fxp.LayerBuffers(M, K, N)
        st["guess"] = case.get("guess", False)
    elif kind == "conv":
        g = [case[k] for k in ("N", "H", "W", "C", "Cout", "KH", "KW", "stride", "pad")]
        n, h, w, c, cout, kh, kw = g[:7]
        st["buf"] = fxp.ConvBuffers(*g)
        st["X"] = _normal(gen, (n, h, w, c), 1.0)
        if c >= 16:                                        # behind a rectifier; the image itself is not
            st["X"].clamp_(min=0.0)
        st["W"] = _normal(gen, (cout, kh, kw, c), math.sqrt(2.0 / (kh * kw * c)))
        st["dY"] = _normal(gen, (n, st["buf"].Ho, st["buf"].Wo, cout), 1e-3)
        st["need_dX"] = case["need_dX"]
    elif kind == "attn":
        b, s, real, d = case["batch"], case["S"], case["real"], case["d"]
        q, k, v = (_normal(gen, (b, s, d), 1.0) for _ in range(3))
        for t in (q, k, v):
            t[:, real:, :] = 0.0
        p = torch.zeros((b, s, s), device="cuda")
        # softmax of products of normal rows: the scores of unit-variance heads are N(0,1) themselves
        p[:, :real, :real] = torch.softmax(_normal(gen, (b, real, real), 1.0), dim=2)
        st.update(Q=q, K=k, V=v, P=p, dS=_normal(gen, (b, s, s), 1e-3), dO=_normal(gen, (b, s, d), 1e-3))
        st["scores"] = fxp.BmmBuffers(b, s, d, s, transB=True)
        st["context"] = fxp.BmmBuffers(b, s, s, d)
    else:
        sizes = _parameter_sizes(case["width"], case["classes"])
        total, at = sum((n + 3) // 4 * 4 for n in sizes), 0
        flat = [_normal(gen, (total,), 1.0) for _ in range(3)]
        lists = ([], [], [])
        for n in sizes:
            sigma = math.sqrt(2.0 / max(n, 64)) * 8.0
            for f, out, scale in zip(flat, lists, (sigma, sigma * 2e-2, sigma * 1e-1)):
                out.append(f[at:at + n].mul_(scale))
            at += (n + 3) // 4 * 4
        st["w"], st["v"] = flat[0], flat[2]                # the parameters of a model are views of two vectors
        st["buf"] = fxp.SgdMultiBuffers(*lists)
    return st


def run(st):
    kind, seed, bits = st["kind"], st["seed"], st["bits"]
    if kind == "linear":
        buf = st["buf"]
        y = fxp.linear_fwd(st["X"], st["W"], buf, seed=seed, step=1, bits=bits, guess=st["guess"])
        dx, dw = fxp.linear_bwd(st["dY"], buf, seed=seed, step=1, bits=bits, guess=st["guess"])
        return y, dx, dw, buf.e
    if kind == "serve":
        buf = st["buf"]
        return fxp.linear_fwd_static(st["X"], st["W"], buf, rounding=fxp.NEAREST, bits=bits), buf.e[:2]
    if kind == "conv":
        buf = st["buf"]
        y = fxp.conv2d_fwd(st["X"], st["W"], buf, seed=seed, step=1, bits=bits)
        dx, dw = fxp.conv2d_bwd(st["dY"], buf, seed=seed, step=1, bits=bits, need_dX=st["need_dX"])
        return (y, dw, buf.e) if dx is None else (y, dx, dw, buf.e)
    if kind == "attn":
        scores, context = st["scores"], st["context"]
        s = fxp.bmm_fwd(st["Q"], st["K"], scores, seed=seed, step=1, bits=bits)
        o = fxp.bmm_fwd(st["P"], st["V"], context, seed=seed, step=2, bits=bits)
        dp, dv = fxp.bmm_bwd(st["dO"], context, seed=seed, step=2, bits=bits)
        dq, dk = fxp.bmm_bwd(st["dS"], scores, seed=seed, step=1, bits=bits)
        return s, o, dp, dv, dq, dk
    fxp.sgd16_step_multi(st["buf"], lr=0.1, momentum=0.9, weight_decay=5e-4, seed=seed, step=1)
    return dict(w=st["w"], v=st["v"])


def work(case):
    """fp32 inputs read and fp32 outputs written once, the int8 copies a call leaves with its caller written once; two
    operations per product term (per element and line for the update)."""
    kind = case["kind"]
    if kind in ("linear", "serve"):
        M, K, N = case["M"], case["K"], case["N"]
        fwd = 6 * (M * K + K * N) + 4 * M * N
        if kind == "serve":
            return dict(bytes=fwd, flops=2 * M * N * K)
        return dict(bytes=fwd + 6 * M * N + 4 * (M * K + K * N), flops=6 * M * N * K)
    if kind == "conv":
        n, h, w, c, cout = (case[k] for k in ("N", "H", "W", "C", "Cout"))
        ho = (h + 2 * case["pad"] - case["KH"]) // case["stride"] + 1
        wo = (w + 2 * case["pad"] - case["KW"]) // case["stride"] + 1
        x, y, k = n * h * w * c, n * ho * wo * cout, case["KH"] * case["KW"] * c
        grads = 1 + (1 if case["need_dX"] else 0)
        return dict(bytes=5 * x + 6 * k * cout + 4 * y + 6 * y + 4 * k * cout + (4 * x if case["need_dX"] else 0),
                    flops=2 * (1 + grads) * n * ho * wo * cout * k)
    if kind == "attn":
        b, s, d = case["batch"], case["S"], case["d"]
        narrow, square = b * s * d, b * s * s
        return dict(bytes=6 * (4 * narrow + 2 * square) + 4 * (4 * narrow + 2 * square), flops=12 * b * s * s * d)
    n = sum(_parameter_sizes(case["width"], case["classes"]))
    return dict(bytes=20 * n, flops=12 * n)


def tolerance(case):
    return "exact"
