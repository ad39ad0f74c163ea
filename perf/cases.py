"""Timed cases of the three pipeline stages: denoising steps, prompt encoding, latent decoding.

A case names a stage and its sizes in plain values:

  stage "diffuse"  `model` (a key of synth.CONFIGS), `blocks` / `single` (how many of the model's
                   equal blocks are built), `reqs` (requests "FxHxW+C", latent extent and condition
                   tokens, comma separated), `steps`, `update` ("euler" / "ddim"), and `call`:
                   "sample" (all steps in one call) or "step" (one call of one step, with the
                   model output returned as well).
  stage "encode"   `model` (synth.ENCODERS), `lens` (prompt lengths, comma separated).
  stage "decode"   `model` (synth.DECODERS or synth.VIDEO_DECODERS), `n` (images, or latent frames
                   of one video), `h`, `w` (latent size).

Blocks of one model are equal in cost and run one after the other, so the widest models are built
with a few of their blocks: the work per block, its shapes and its traffic are those of the model.
"""
import math

import numpy as np
import torch

import synth
from paper_2510_02838_amd import binding, decoder, encoder


def listed():
    return [
        # Smallest model and image: about a hundred launches of a few microseconds each, so this is
        # the latency of the host path and of single launches.
        dict(name="tiny_4steps", stage="diffuse", model="tiny", blocks=2, single=0, reqs="1x16x16+16", steps=4, update="euler", call="sample"),
        # One 256x256 image, one step per call, as a serving loop that mixes requests at every step
        # does: few rows against 4 GB of weights.
        dict(name="sd3_256_step", stage="diffuse", model="sd3", blocks=24, single=0, reqs="1x32x32+154", steps=1, update="euler", call="step"),
        # The benchmark's headline request, 1024x1024 (4250 tokens), heads of 64.
        dict(name="sd3_1024", stage="diffuse", model="sd3", blocks=24, single=0, reqs="1x128x128+154", steps=2, update="euler", call="sample"),
        # Eight requests of four resolutions in one packed batch (18384 tokens), with the other update rule.
        dict(name="hetero8", stage="diffuse", model="sd3", blocks=24, single=0,
             reqs="1x32x32+154,1x32x32+154,1x64x64+154,1x64x64+154,1x96x96+154,1x128x128+154,1x128x128+154,1x128x128+154",
             steps=1, update="ddim", call="sample"),
        # Rotary two-stream and single-stream blocks at the benchmark size (4608 tokens, heads of 128) ...
        dict(name="flux_1024", stage="diffuse", model="flux", blocks=4, single=8, reqs="1x128x128+512", steps=2, update="euler", call="sample"),
        # ... and two odd-sized requests of the same model (1080x720 and 520x776, short prompts).
        dict(name="flux_ragged", stage="diffuse", model="flux", blocks=4, single=8, reqs="1x90x134+77,1x64x98+333", steps=1, update="euler", call="step"),
        # Video denoiser at its benchmark size: 32760 tokens, self- and cross-attention.
        dict(name="wan_32k", stage="diffuse", model="wan", blocks=3, single=0, reqs="21x60x104+512", steps=1, update="euler", call="sample"),
        # One short prompt through the text encoder: every weight is read for 32 rows.
        dict(name="encode_32", stage="encode", model="t5_xxl", lens="32"),
        # A queue of prompts of the lengths that the paper's pipelines meet (30-500 tokens).
        dict(name="encode_batch", stage="encode", model="t5_xxl", lens="500,431,350,287,256,201,160,128,97,77,77,64,51,42,33,30"),
        # One 256x256 image: the smallest decode in ordinary use.
        dict(name="decode_256", stage="decode", model="ae_kl", n=1, h=32, w=32),
        # One 1024x1024 image.
        dict(name="decode_1024", stage="decode", model="ae_kl", n=1, h=128, w=128),
        # A 17-frame 384x256 video from five latent frames.
        dict(name="decode_video", stage="decode", model="vae3d", n=5, h=32, w=48),
    ]


LARGEST_FLOPS = 1.3e14     # of the listed cases (wan_32k)


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any stage and model, sizes over the whole range (logarithmic), odd ones among them."""
    while True:
        kind = rng.choice(["tiny", "sd3", "sd3", "sd3", "flux", "flux", "wan", "encode", "encode", "decode", "decode", "video"])
        if kind in ("tiny", "sd3", "flux", "wan"):
            n_req = {"tiny": 4, "sd3": 8, "flux": 3, "wan": 2}[kind]
            n_req = _logint(rng, 1, n_req)
            same = rng.random() < 0.3                      # batches of one shape are common too
            reqs = []
            for _ in range(n_req):
                lo, hi = {"tiny": (8, 64), "sd3": (16, 160), "flux": (16, 160), "wan": (16, 104)}[kind]
                f = _logint(rng, 1, 21) if kind == "wan" else 1
                reqs.append(f"{f}x{2 * _logint(rng, lo // 2, hi // 2)}x{2 * _logint(rng, lo // 2, hi // 2)}+{_logint(rng, 16, 512)}")
            if same:
                reqs = reqs[:1] * n_req
            step = rng.random() < 0.4
            case = dict(stage="diffuse", model=kind, blocks={"tiny": 2, "sd3": 24, "flux": 4, "wan": 3}[kind],
                        single=8 if kind == "flux" else 0, reqs=",".join(reqs), steps=1 if step else rng.choice([1, 2, 4]),
                        update=rng.choice(["euler", "ddim"]), call="step" if step else "sample")
        elif kind == "encode":
            lens = [_logint(rng, 16, 512) for _ in range(_logint(rng, 1, 32))]
            case = dict(stage="encode", model="t5_xxl", lens=",".join(map(str, lens)))
        elif kind == "decode":                             # latent pixels in whole groups of 64 (of 256 for a batch)
            n = _logint(rng, 1, 4)
            q = 8 if n == 1 else 16
            case = dict(stage="decode", model="ae_kl", n=n, h=q * _logint(rng, 1, 128 // q), w=q * _logint(rng, 1, 160 // q))
        else:
            case = dict(stage="decode", model="vae3d", n=_logint(rng, 1, 9), h=16 * rng.randint(1, 3), w=16 * rng.randint(1, 4))
        if work(case)["flops"] <= LARGEST_FLOPS:
            return case


# ---- sizes ---------------------------------------------------------------------------------------

def _reqs(case):
    out = []
    for r in case["reqs"].split(","):
        dims, cond = r.split("+")
        out.append(tuple(int(v) for v in dims.split("x")) + (int(cond),))
    return out


def _lens(case):
    return [int(v) for v in case["lens"].split(",")]


def _arch(case):
    if case["stage"] == "encode":
        return synth.ENCODERS[case["model"]]
    if case["stage"] == "decode":
        return {**synth.DECODERS, **synth.VIDEO_DECODERS}[case["model"]]
    return dict(synth.CONFIGS[case["model"]]["arch"], n_blocks=case["blocks"], n_single=case["single"])


def _diffuse_work(case):
    a = _arch(case)
    d, ff, pt, ph, pw = a["hidden"], a["mlp_hidden"], *a["patch"]
    pdim = a["latent_ch"] * pt * ph * pw
    reqs, T = _reqs(case), case["steps"]
    img = [(f // pt) * (h // ph) * (w // pw) for f, h, w, _ in reqs]
    txt = [c for *_, c in reqs]
    Ni, Nt, R = sum(img), sum(txt), T * len(reqs)
    lat = sum(a["latent_ch"] * f * h * w for f, h, w, _ in reqs)
    stream = 4 * d * d + 2 * d * ff                        # qkv, projection, MLP
    once = Nt * a["cond_dim"] * d + R * (256 * d + d * d)  # multiply-adds of one call, and weights of one call
    w_once = a["cond_dim"] * d + 256 * d + d * d
    step = 2 * Ni * pdim * d
    w_step = 2 * pdim * d
    if a["family"] in ("J", "F"):
        joint = [i + t for i, t in zip(img, txt)]
        mod = a["n_blocks"] * 12 * d * d + a["n_single"] * 3 * d * d + 2 * d * d
        step += a["n_blocks"] * (Ni + Nt) * stream + a["n_single"] * (Ni + Nt) * stream
        step += (a["n_blocks"] + a["n_single"]) * 2 * sum(n * n for n in joint) * d
        w_step += a["n_blocks"] * 2 * stream + a["n_single"] * stream
    else:
        mod = 8 * d * d
        once += a["n_blocks"] * Nt * 2 * d * d
        w_once += a["n_blocks"] * 2 * d * d
        step += a["n_blocks"] * (Ni * (stream + 2 * d * d) + 2 * sum(n * n for n in img) * d + 2 * sum(i * t for i, t in zip(img, txt)) * d)
        w_step += a["n_blocks"] * (stream + 2 * d * d)
    # every weight matrix once (bf16), condition, noise in, latent out (and the model output of a step call)
    moved = 2 * (w_once + mod + w_step) + 2 * Nt * a["cond_dim"] + 4 * lat * (3 if case["call"] == "step" else 2)
    return {"bytes": moved, "flops": 2 * (once + R * mod + T * step)}


def _encode_work(case):
    a, lens = _arch(case), _lens(case)
    d, hd, ff, n = a["d_model"], a["n_heads"] * a["head_dim"], a["d_ff"], sum(lens)
    layer = 4 * d * hd + 3 * d * ff
    macs = a["n_layers"] * (n * layer + 2 * sum(v * v for v in lens) * hd)
    return {"bytes": 2 * a["n_layers"] * layer + n * (4 + 4 * d + 2 * d), "flops": 2 * macs}


def _decode_work(case):
    a = _arch(case)
    ch, video = a["channels"], "t_up" in a
    taps, n, h, w = (27 if video else 9), case["n"], case["h"], case["w"]
    total = {"macs": 0, "weights": 0}

    def conv(pixels, cin, cout, k):
        total["macs"] += pixels * k * cin * cout
        total["weights"] += k * cin * cout

    def res(pixels, cin, cout):
        conv(pixels, cin, cout, taps)
        conv(pixels, cout, cout, taps)
        if cin != cout:
            conv(pixels, cin, cout, 1)

    px = n * h * w
    moved = 4 * a["latent_ch"] * px
    conv(px, a["latent_ch"], ch[0], taps)
    res(px, ch[0], ch[0])
    res(px, ch[0], ch[0])
    for _ in range(4):
        conv(px, ch[0], ch[0], 1)
    total["macs"] += n * 2 * (h * w) ** 2 * ch[0]
    prev = ch[0]
    for level, c in enumerate(ch):
        for r in range(a["n_res"]):
            res(px, prev if r == 0 else c, c)
        prev = c
        if level != len(ch) - 1:
            n = 2 * n - 1 if video and level < a["t_up"] else n
            h, w = 2 * h, 2 * w
            px = n * h * w
            conv(px, c, c, taps)
    conv(px, prev, a["out_ch"], taps)
    return {"bytes": moved + 2 * total["weights"] + 4 * a["out_ch"] * px, "flops": 2 * total["macs"]}


def work(case):
    return {"diffuse": _diffuse_work, "encode": _encode_work, "decode": _decode_work}[case["stage"]](case)


# ---- inputs and the pass -------------------------------------------------------------------------

def prepare(case, seed):
    a = _arch(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["stage"] == "diffuse":
        reqs = _reqs(case)
        m = binding.DiT(a)
        m.ensure_workspace(reqs, case["steps"])
        m.init_weights(seed, 0.02)
        lat = sum(a["latent_ch"] * f * h * w for f, h, w, _ in reqs)
        noise = torch.randn(lat, generator=gen, device="cuda")
        cond = torch.randn((sum(r[3] for r in reqs), a["cond_dim"]), generator=gen, device="cuda").to(torch.bfloat16)
        rows = []
        for f, h, w, _ in reqs:                            # larger requests stay longer at high noise
            shift = min(3.0, max(1.0, math.sqrt(h * w) / 42.0))
            rows.append(synth.default_sigmas(case["steps"] + (case["update"] == "ddim"), shift))
        # the whole way down to zero noise (ddim starts one level later: it needs sigma below 1)
        sig = np.ascontiguousarray(np.stack(rows)[:, -case["steps"] - 1:])
        return dict(case=case, m=m, reqs=reqs, noise=noise, x=torch.empty_like(noise), v=torch.empty_like(noise), cond=cond,
                    sigmas=sig, kind={"euler": 0, "ddim": 1}[case["update"]])
    if case["stage"] == "encode":
        lens = _lens(case)
        m = encoder.Encoder(a)
        m.ensure_workspace(lens)
        # attention scores are not divided by sqrt(head size): at this deviation their own is about 2, as in a
        # trained encoder (0.02 makes the softmax one-hot and the output depend on the last bit of every sum)
        m.init_weights(seed, 0.008)
        tokens = torch.randint(0, a["vocab"], (sum(lens),), generator=gen, device="cuda", dtype=torch.int32)
        return dict(case=case, m=m, lens=lens, tokens=tokens,
                    out=torch.empty((sum(lens), a["d_model"]), dtype=torch.bfloat16, device="cuda"))
    n, h, w = case["n"], case["h"], case["w"]
    m = decoder.Decoder(a)
    m.ensure_workspace(h, w, n)
    m.init_weights(seed, 0.02)
    up, frames = m.up_factor(), (m.frames_out(n) if "t_up" in a else n)
    latent = torch.randn(n * a["latent_ch"] * h * w, generator=gen, device="cuda")
    image = torch.empty((frames, h * up, w * up, a["out_ch"]), dtype=torch.float32, device="cuda")
    return dict(case=case, m=m, latent=latent, image=image)


def run(state):
    case, m = state["case"], state["m"]
    if case["stage"] == "diffuse":
        x = state["x"]
        x.copy_(state["noise"])                            # the call updates the latent in place
        if case["call"] == "step":
            m.denoise_step(state["reqs"], x, state["cond"], state["sigmas"][:, 0], state["sigmas"][:, 1], state["kind"], state["v"])
            return x, state["v"]
        m.sample(state["reqs"], x, state["cond"], state["sigmas"], state["kind"])
        return x
    if case["stage"] == "encode":
        m.forward(state["lens"], state["tokens"], out_bf16=state["out"])
        return state["out"]
    m.forward(case["h"], case["w"], state["latent"], state["image"], n=case["n"])
    return state["image"]


def tolerance(case):
    """Relative 2-norm errors between two correct evaluations in bf16 (fp32 sums and streams): about four
    times what the same inputs give with other roundings on the way (the q/k norm and the value transpose
    as separate kernels with bf16 between: 6e-7, 5e-4, 4e-3, 4e-3) or with the products summed in another
    order (a prompt or an image alone and in a larger batch, a video alone and as the start of a longer one:
    1.3e-2, 8e-3, 5e-3)."""
    rel = {"tiny": 1e-5, "sd3": 2e-3, "flux": 1.5e-2, "wan": 1.5e-2, "t5_xxl": 4e-2, "ae_kl": 2.5e-2, "vae3d": 2e-2}
    return {"rel": rel[case["model"]]}
