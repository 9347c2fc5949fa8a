"""What is measured: the calls a user of this library makes, over the range they are made in.

Two programs use the library.  A converter takes fp32 weights through qg_quantize, qg_pack and (for
batch-1 serving) qg_to_narrow, and now and then reads a blob back with qg_unpack.  A server keeps
packed weights, activation and output buffers and workspaces, and calls the matrix-vector products
(single, grouped per decoder block, gated pair) for every generated token and qg_gemm_small for a
prompt of a few tokens.  Shapes are those of the benchmark's decoder layer sets (4096 / 11008,
5120 / 13824, 8192 / 22016), its 512 x 512 smallest problem, and ragged sizes in between.
"""
import math

import torch

from paper_2307_03738_amd import binding as qg

CELL = {4: 8, 2: 16, 3: 32}           # codes a group has to be a whole number of
STEP = {4: 128, 2: 256, 3: 256}       # the narrow layout's K granule


def listed():
    return [
        # latency of the smallest single product (the benchmark's smallest problem)
        {"name": "matvec_512", "kind": "matvec", "N": 512, "K": 512, "bits": 4, "group": 64},
        # one product whose outputs and inputs are no multiple of anything the kernels tile by
        {"name": "matvec_ragged", "kind": "matvec", "N": 5003, "K": 4160, "bits": 3, "group": 32},
        # one token through the seven linear layers of a block, the three benchmark sets; the
        # last one on the layout a server keeps that also runs prompts
        {"name": "block_7b_b4", "kind": "block_narrow", "hidden": 4096, "inner": 11008, "bits": 4, "group": 128},
        {"name": "block_13b_b3", "kind": "block_narrow", "hidden": 5120, "inner": 13824, "bits": 3, "group": 64},
        {"name": "block_65b_b2_wide", "kind": "block", "hidden": 8192, "inner": 22016, "bits": 2, "group": 32},
        # the gated MLP input of a block in one call
        {"name": "gated_7b_b4", "kind": "gated", "N": 11008, "K": 4096, "bits": 4, "group": 128},
        # a prompt of 16, 37 and 128 tokens through single layers, every width
        {"name": "prompt16_7b_up_b4", "kind": "prompt", "N": 11008, "K": 4096, "bits": 4, "group": 128, "M": 16},
        {"name": "prompt37_13b_up_b3", "kind": "prompt", "N": 13824, "K": 5120, "bits": 3, "group": 64, "M": 37},
        {"name": "prompt128_7b_down_b4", "kind": "prompt", "N": 4096, "K": 11008, "bits": 4, "group": 128, "M": 128},
        {"name": "prompt128_65b_up_b2", "kind": "prompt", "N": 22016, "K": 8192, "bits": 2, "group": 32, "M": 128},
        # the converter: fp32 weights to the blob a batch-1 server loads, and a blob read back
        {"name": "convert_13b_b3", "kind": "convert", "N": 13824, "K": 5120, "bits": 3, "group": 64},
        {"name": "unpack_7b_b4", "kind": "unpack", "N": 11008, "K": 4096, "bits": 4, "group": 128},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["matvec", "block_narrow", "block", "gated", "prompt", "prompt", "convert", "unpack"])
    bits = rng.choice([4, 4, 3, 2])
    group = rng.choice([32, 64, 128])
    case = {"kind": kind, "bits": bits, "group": group}
    if kind in ("block", "block_narrow"):
        hidden = max(2, round(_log_uniform(rng, 512, 8192) / 256)) * 256
        case["hidden"] = hidden
        case["inner"] = max(2, round(hidden * rng.uniform(2.0, 22016 / 8192) / 256)) * 256
        return case
    # K is a whole number of groups (always), of steps for the narrow layout, and in between
    # anything; N is anything, odd ones among them (the gated pair takes multiples of 64)
    most = 13824 * 5120 if kind in ("convert", "unpack") else 22016 * 8192
    grain = STEP[bits] if kind == "convert" else group
    K = max(1, round(_log_uniform(rng, 512, 22016) / grain)) * grain
    N = round(_log_uniform(rng, 512, min(22016, most // K)))
    if kind == "gated":
        N = max(1, min(N, most // K // 2) // 64) * 64
    if kind in ("matvec", "prompt") and rng.random() < 0.2:
        case["group"] = K if K % (STEP[bits]) == 0 else group          # one group per output
    case["N"], case["K"] = N, K
    if kind == "prompt":
        case["M"] = round(_log_uniform(rng, 2, 128))
    return case


def _shapes(case):
    if "hidden" in case:
        h, i = case["hidden"], case["inner"]
        return [(h, h)] * 4 + [(i, h)] * 2 + [(h, i)]
    n = 2 * case["N"] if case["kind"] == "gated" else case["N"]
    return [(n, case["K"])]


# Zero-mean Gaussian weights; at 4 bits one entry in a thousand is 20 times larger, as in the
# benchmark's 4-bit set.  Activations are standard normal.
def _weights(case, gen, N, K):
    W = torch.randn((N, K), generator=gen, device="cuda") * 0.02
    if case["bits"] == 4:
        W = torch.where(torch.rand((N, K), generator=gen, device="cuda") < 0.001, W * 20.0, W)
    return W


def _draws(case, seed):
    """(W, activations) per matrix, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    for N, K in _shapes(case):
        W = _weights(case, gen, N, K)
        yield W, torch.randn((case.get("M", 1), K), generator=gen, device="cuda")


def prepare(case, seed):
    kind, bits, group = case["kind"], case["bits"], case["group"]
    if kind == "convert":
        (W, _), = _draws(case, seed)
        return {"case": case, "W": W}
    problems = []
    for W, x in _draws(case, seed):
        N, K = W.shape
        blob = qg.qg_pack(*qg.qg_quantize(W, bits, group), bits, group)
        if kind == "block_narrow":
            blob = qg.qg_to_narrow(blob, N, K, bits, group)
        M = x.shape[0]
        problems.append({"packed": blob, "N": N, "K": K, "bits": bits, "group": group,
                         "x": x if kind == "prompt" else x[0].clone(),
                         "y": torch.empty((M, N) if kind == "prompt" else N, device="cuda")})
        del W
    state = {"case": case, "problems": problems}
    p = problems[0]
    if kind == "block":
        state["launch"] = qg.GroupedGemv(problems)
    elif kind == "block_narrow":
        state["launch"] = qg.GroupedGemvNarrow(problems)
    elif kind in ("matvec", "gated", "prompt"):
        state["workspace"] = qg.new_workspace(qg.qg_workspace_bytes(p["N"], p["K"], bits, group, case.get("M", 1)))
    if kind == "gated":
        state["h"] = torch.empty(case["N"], device="cuda")
    return state


def run(state):
    case = state["case"]
    kind, bits, group = case["kind"], case["bits"], case["group"]
    if kind == "convert":
        N, K = case["N"], case["K"]
        q, s, z = qg.qg_quantize(state["W"], bits, group)
        blob = qg.qg_pack(q, s, z, bits, group)
        return [q, s, z, blob, qg.qg_to_narrow(blob, N, K, bits, group)]
    p = state["problems"][0]
    if kind in ("block", "block_narrow"):
        state["launch"].launch()
        return [p["y"] for p in state["problems"]]
    if kind == "matvec":
        return qg.qg_gemv(p["packed"], p["N"], p["K"], bits, group, p["x"], p["y"], state["workspace"])
    if kind == "gated":
        return qg.qg_gemv_swiglu(p["packed"], case["N"], p["K"], bits, group, p["x"], state["h"], state["workspace"])
    if kind == "prompt":
        return qg.qg_gemm_small(p["packed"], p["N"], p["K"], bits, group, p["x"], p["y"], state["workspace"])
    return list(qg.qg_unpack(p["packed"], p["N"], p["K"], bits, group))


def _stored_bytes(case, N, K):
    """Codes, fp32 scales and b-bit zero-points."""
    return N * K * case["bits"] / 8 + N * (K // case["group"]) * (4 + case["bits"] / 8)


def work(case):
    M = case.get("M", 1)
    nbytes = flops = 0.0
    for N, K in _shapes(case):
        stored = _stored_bytes(case, N, K)
        plain = N * K + N * (K // case["group"]) * 5                  # a byte per code and zero-point
        if case["kind"] == "convert":
            nbytes += 4 * N * K + plain + 2 * stored                  # W read; codes, blob, narrow blob written
        elif case["kind"] == "unpack":
            nbytes += stored + plain
        else:
            outputs = case["N"] if case["kind"] == "gated" else N
            nbytes += stored + 4 * M * (K + outputs)
            flops += 2.0 * M * N * K
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] in ("convert", "unpack"):
        return "exact"
    if case["kind"] == "prompt":
        # bf16 activations (in some 4-bit forms bf16 weights too), fp32 sums: 1.7e-3 seen, 2.4e-3 with both
        return {"rel": 8e-3, "max": 5e-2}
    # fp32 sums of exact products: 1.3e-7 ... 1e-6 seen
    return {"rel": 4e-6, "max": 4e-5}


def _dequantized(W, bits, group):
    """s (q - z) in 64 bits: min-max round-to-nearest per group, every step rounded to fp32 (a 64-bit
    quotient of 32-bit numbers rounds to the correctly rounded 32-bit one)."""
    N, K = W.shape
    w = W.view(N, K // group, group)
    qmax = (1 << bits) - 1
    lo = w.amin(2).clamp(max=0.0)
    hi = w.amax(2).clamp(min=0.0)
    span = hi - lo
    s = (span.double() / qmax).float()
    s = torch.where(span == 0, torch.ones_like(s), s)
    z = torch.where(span == 0, torch.zeros_like(s), (-lo.double() / s.double()).float().round().clamp(0, qmax))
    q = ((w.double() / s.double().unsqueeze(2)).float().round() + z.unsqueeze(2)).clamp(0, qmax)
    return ((q - z.unsqueeze(2)).double() * s.double().unsqueeze(2)).view(N, K)


def exact(case, seed):
    if case["kind"] in ("convert", "unpack"):
        return None
    outs = []
    for W, x in _draws(case, seed):
        What = _dequantized(W, case["bits"], case["group"])
        outs.append(x.double() @ What.t())
        del W, What
    if case["kind"] == "prompt":
        return outs[0]
    outs = [y[0] for y in outs]
    if case["kind"] == "gated":
        g, u = outs[0][:case["N"]], outs[0][case["N"]:]
        return g / (1.0 + torch.exp(-g)) * u
    return outs[0] if case["kind"] == "matvec" else outs
