"""The work that stands for this library in use: what a quantized video Diffusion Transformer has it
do in one denoising step, through the tensor helpers of the binding.

Three kinds of case:

* ``linear``: one quantized linear (quantize the activations, integer GEMM, epilogue).  ``scheme``
  picks the activation quantizer: ``token`` (one scale per token), ``rot`` (the same on rotated
  activations), ``asym`` (unsigned codes with a zero point) or ``tensor`` (one scale per input).
* ``block``: the four linears of one STDiT block, the second MLP linear fed with the first one's
  output, each with its own weight bit-width.
* ``decide``: the reductions behind one step's cache, bit-width and pruning decisions: the latent
  delta and the inter-frame gradient norm of Eq. (5), the variation over earlier steps of Eq. (11)
  and the similarity of two layers' features of Eq. (9).

Weights, their scales, biases, workspaces and output buffers are made once and kept, as a serving
program keeps them; activations and latents are drawn on the GPU from the seed with the
distributions of the library's synthetic inputs (normal with 1 % outlier columns twenty times as
large, or post-GELU; weights of standard deviation 0.02).
"""
import math

import torch

from paper_2503_06545_amd import binding as qc

HIDDEN, MLP = 1152, 4608
DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "bf16": 2}

# the largest linear a case may hold: the second MLP linear of the 512 x 512 video with both halves
# of the classifier-free guidance
MOST_MACS = 131072 * HIDDEN * MLP


def _linear(name=None, M=256, K=HIDDEN, N=HIDDEN, bits=8, act_bits=8, scheme="token", rot=0, x="bf16",
            out="bf16", epi="none", bias=True, post_gelu=False):
    case = {"kind": "linear", "M": M, "K": K, "N": N, "bits": bits, "act_bits": act_bits, "scheme": scheme,
            "rot": rot, "x": x, "out": out, "epi": epi, "bias": bias, "post_gelu": post_gelu}
    return dict(case, name=name) if name else case


def _block(name=None, M=4096, qkv=8, proj=8, fc1=8, fc2=8):
    case = {"kind": "block", "M": M, "qkv": qkv, "proj": proj, "fc1": fc1, "fc2": fc2}
    return dict(case, name=name) if name else case


def _decide(name=None, frames=16, inner=4096, earlier=3, tokens=4096):
    case = {"kind": "decide", "frames": frames, "inner": inner, "earlier": earlier, "tokens": tokens}
    return dict(case, name=name) if name else case


def listed():
    return [
        # one conditioning vector per guidance half through the linear that makes a block's six
        # modulation vectors: the fewest tokens there are, all of it weight traffic and latency
        _linear("modulation_2_tokens", M=2, N=6 * HIDDEN),
        # the tiny configuration: a few hundred tokens (a short video, a text conditioning)
        _linear("tiny_256_f32", M=256, x="f32", out="f32"),
        # nothing a multiple of anything: ragged tokens, reduction and channels
        _linear("ragged_k1000", M=4099, K=1000, N=1301, bits=4, out="f32"),
        # QKV of a 256 x 256 video
        _linear("qkv_256", M=16384, N=3 * HIDDEN),
        # first MLP linear with GELU, 512 x 512 video
        _linear("fc1_gelu_512", M=65536, N=MLP, epi="gelu_tanh"),
        # second MLP linear with 4-bit weights, 512 x 512 video
        _linear("fc2_w4_512", M=65536, K=MLP, bits=4, post_gelu=True),
        # the W4A6 operating point on rotated activations, attention output projection
        _linear("proj_rot_w4a6_512", M=65536, bits=4, act_bits=6, scheme="rot", rot=128),
        # the asymmetric quantizer on post-GELU inputs, a short 51-frame video
        _linear("fc2_asym_ragged", M=51 * 193, K=MLP, act_bits=8, scheme="asym", post_gelu=True),
        # one scale for the whole layer input, both guidance halves of a 256 x 256 video
        _linear("qkv_tensor_256_cfg", M=32768, N=3 * HIDDEN, scheme="tensor"),
        # one whole block at 512 x 512 with both guidance halves: the largest
        _block("block_512_cfg", M=131072, qkv=8, proj=4, fc1=8, fc2=8),
        # the decisions of a step on the latents of a small video: latency
        _decide("decide_256", frames=16, inner=4 * 32 * 32, earlier=3, tokens=1024),
        # the same on the latent shape of the benchmark and the features of a 512 x 512 video
        _decide("decide_512", frames=16, inner=4 * 16 * 64 * 64, earlier=4, tokens=65536),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear"] * 7 + ["block"] * 1 + ["decide"] * 3)
    if kind == "block":
        return _block(M=_log_uniform(rng, 64, 65536), qkv=rng.choice([8, 8, 4]), proj=rng.choice([8, 8, 4]),
                      fc1=rng.choice([8, 8, 4]), fc2=rng.choice([8, 8, 4]))
    if kind == "decide":
        return _decide(frames=rng.randint(2, 51), inner=4 * _log_uniform(rng, 200, 16384) + rng.choice([0, 0, 0, 1]),
                       earlier=rng.randint(1, qc.QC_MAX_PREV), tokens=_log_uniform(rng, 64, 65536))
    scheme = rng.choice(["token"] * 4 + ["rot", "asym", "tensor"])
    # widths of the transformer half of the time, any others otherwise, one in four of those odd
    K = rng.choice([HIDDEN, HIDDEN, HIDDEN, MLP]) if rng.random() < 0.6 else 16 * _log_uniform(rng, 8, 288)
    N = rng.choice([HIDDEN, 3 * HIDDEN, MLP]) if rng.random() < 0.6 else _log_uniform(rng, 32, MLP)
    if scheme in ("token", "tensor") and K not in (HIDDEN, MLP) and rng.random() < 0.4:
        K += rng.choice([2, 4, 8, 10])
    rot = 0
    if scheme == "rot":
        K = K // 128 * 128 if K >= 128 else 128
        rot = rng.choice([16, 32, 64, 128])
    M = min(_log_uniform(rng, 1, 131072), max(1, MOST_MACS // (K * N)))
    post_gelu = K == MLP or scheme == "asym"
    return _linear(M=M, K=K, N=N, bits=rng.choice([8, 8, 4]), act_bits=rng.choice([8, 8, 8, 6, 4]), scheme=scheme,
                   rot=rot, x=rng.choice(["bf16", "bf16", "bf16", "f32"]), out=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                   epi=rng.choice(["none", "none", "gelu_tanh", "gelu_erf"]), bias=rng.random() < 0.8, post_gelu=post_gelu)


# ---- inputs --------------------------------------------------------------------------------------

def _activations(g, M, K, dtype, post_gelu):
    x = torch.randn(M, K, generator=g, device="cuda")
    if post_gelu:
        x = torch.nn.functional.gelu(x, approximate="tanh")
    else:
        cols = torch.randperm(K, generator=g, device="cuda")[:max(1, round(0.01 * K))]
        x[:, cols] *= 20.0
    return x.to(dtype)


def _weights(g, N, K, bits, rot=0):
    pw = qc.pack_weight_t(torch.randn(N, K, generator=g, device="cuda") * 0.02, bits, rot)
    return pw, torch.randn(N, generator=g, device="cuda") * 0.01


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    state = {"case": case}
    if case["kind"] == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        pw, bias = _weights(g, N, K, case["bits"], case["rot"])
        make_workspace = {"asym": qc.qlinear_asym_workspace_t, "tensor": qc.qlinear_tensor_workspace_t}.get(
            case["scheme"], qc.qlinear_workspace_t)
        state.update(X=_activations(g, M, K, DTYPE[case["x"]], case["post_gelu"]), pw=pw,
                     bias=bias if case["bias"] else None, workspace=make_workspace(M, K, N),
                     Y=torch.empty(M, N, dtype=DTYPE[case["out"]], device="cuda"))
        if case["scheme"] == "asym":
            state["row_sums"] = qc.weight_row_sums_t(pw)
        return state
    if case["kind"] == "block":
        M = case["M"]
        state["workspace"] = qc.qlinear_workspace_t(M, MLP, HIDDEN)
        for name, K, N in (("qkv", HIDDEN, 3 * HIDDEN), ("proj", HIDDEN, HIDDEN), ("fc1", HIDDEN, MLP), ("fc2", MLP, HIDDEN)):
            pw, bias = _weights(g, N, K, case[name])
            state[name] = {"pw": pw, "bias": bias, "Y": torch.empty(M, N, dtype=torch.bfloat16, device="cuda")}
            if name != "fc2":  # which reads what fc1 wrote
                state[name]["X"] = _activations(g, M, K, torch.bfloat16, False)
        return state
    frames, inner, earlier = case["frames"], case["inner"], case["earlier"]
    n, f = frames * inner, case["tokens"] * HIDDEN
    prev = torch.randn(frames, inner, generator=g, device="cuda")
    state["earlier"] = [prev + 0.01 * (i + 1) * torch.randn(frames, inner, generator=g, device="cuda") if i else prev
                        for i in range(earlier)]
    state["cur"] = prev + 0.01 * torch.randn(frames, inner, generator=g, device="cuda")
    a = torch.randn(case["tokens"], HIDDEN, generator=g, device="cuda")
    state["layers"] = (a.bfloat16(), (a + 0.5 * torch.randn(case["tokens"], HIDDEN, generator=g, device="cuda")).bfloat16())
    sizes = (qc.qc_latent_delta_workspace_bytes(n), qc.qc_frame_gradient_norm_workspace_bytes(frames, inner),
             qc.qc_cumulative_variation_workspace_bytes(n, earlier), qc.qc_layer_similarity_workspace_bytes(f))
    state["workspace"] = [torch.empty(s, dtype=torch.uint8, device="cuda") for s in sizes]
    state["out"] = [torch.empty(s, device="cuda") for s in (3, 2, earlier + 1, 4)]
    return state


# ---- one pass ------------------------------------------------------------------------------------

def run(state):
    case = state["case"]
    if case["kind"] == "linear":
        args = dict(bias=state["bias"], epi=case["epi"], out=case["out"], workspace=state["workspace"], Y=state["Y"],
                    act_bits=case["act_bits"])
        if case["scheme"] == "asym":
            return qc.qlinear_asym_t(state["X"], state["pw"], state["row_sums"], **args)
        if case["scheme"] == "tensor":
            return qc.qlinear_tensor_t(state["X"], state["pw"], **args)
        return qc.qlinear_t(state["X"], state["pw"], rot_block=case["rot"], **args)
    if case["kind"] == "block":
        outs = {}
        for name, epi in (("qkv", "none"), ("proj", "none"), ("fc1", "gelu_tanh"), ("fc2", "none")):
            s = state[name]
            X = outs["fc1"] if name == "fc2" else s["X"]
            outs[name] = qc.qlinear_t(X, s["pw"], bias=s["bias"], epi=epi, workspace=state["workspace"], Y=s["Y"])
        return outs
    ws, out = state["workspace"], state["out"]
    return {"delta": qc.latent_delta_t(state["cur"], state["earlier"][0], workspace=ws[0], out3=out[0]),
            "gradient": qc.frame_gradient_norm_t(state["cur"], workspace=ws[1], out2=out[1]),
            "variation": qc.cumulative_variation_t(state["cur"], state["earlier"], workspace=ws[2], out=out[2]),
            "similarity": qc.layer_similarity_t(*state["layers"], workspace=ws[3], out4=out[3])}


# ---- what a pass cannot do without ---------------------------------------------------------------

def _linear_work(M, K, N, bits, x="bf16", out="bf16"):
    return {"bytes": M * K * SIZE[x] + N * K * bits / 8 + M * N * SIZE[out] + 8 * N, "flops": 2.0 * M * N * K}


def work(case):
    if case["kind"] == "linear":
        return _linear_work(case["M"], case["K"], case["N"], case["bits"], case["x"], case["out"])
    if case["kind"] == "block":
        M = case["M"]
        parts = [_linear_work(M, HIDDEN, 3 * HIDDEN, case["qkv"]), _linear_work(M, HIDDEN, HIDDEN, case["proj"]),
                 _linear_work(M, HIDDEN, MLP, case["fc1"]), _linear_work(M, MLP, HIDDEN, case["fc2"])]
        return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}
    # every tensor once: the current latent and the earlier ones, both layers' features
    n, f = case["frames"] * case["inner"], case["tokens"] * HIDDEN
    return {"bytes": 4.0 * n * (1 + case["earlier"]) + 2.0 * 2 * f, "flops": n * (7.0 + 3 * case["earlier"]) + 6.0 * f}


def tolerance(case):
    # Four times what the outputs were measured to be off the same integers carried through the
    # scales, the bias, the activation and the sums in 64 bits: reductions 3e-8 (their last
    # rounding to 32 bits), 32-bit outputs 9e-8 (largest 3.1e-7, with GELU), bf16 outputs 1.66e-3
    # (largest 3.9e-3, half a unit in the last place).
    if case["kind"] == "decide":
        return {"rel": 2.5e-7, "max": 2.5e-7}
    if case["kind"] == "linear" and case["out"] == "f32":
        return {"rel": 4e-7, "max": 1.3e-6}
    return {"rel": 6.6e-3, "max": 1.6e-2}
