"""Performance cases: what a program that uses this package has the GPU do, through its public entry points.

Four kinds of call:

  step     one next-scale step through some of a model's blocks (StepRunner.run_step): entropy, selection, pruned block
           and cache merge per block, every call issued one by one.  The bulk of the work at the later scales.
  image    all scales of one batch of images (ImageRunner).  "graphs": planned buffers and one HIP graph per scale, as a
           serving loop replays them; otherwise eager calls whose keep counts come from the layer-linkage controller,
           every image with its own.  The early scales are a long row of small, latency-bound launches.
  tokens   token entropies and their per-image means from stored logits (Nova.entropy), as the activation rule asks for
           at every dense scale.
  head     the same straight from the prediction head (Nova.head_entropy), the logits never stored.

Inputs are drawn on the device with the distributions of the repository's workloads: logits N(0, s^2) with one s per
token, log-uniform in [0.1, 10]; activations, prior keys / values and residual caches N(0, 1); weights N(0, 0.02^2).
"""
import math

import torch

from paper_2602_01345_amd import Nova, pack_k_cache, pack_v_cache
from paper_2602_01345_amd.binding import BlockVariant
from paper_2602_01345_amd.image import ImageRunner
from paper_2602_01345_amd.step import BlockState, StepRunner

_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
_SIZES = {"f32": 4, "bf16": 2}
_GRIDS = {256: (1, 2, 3, 4, 5, 6, 8, 10, 13, 16), 512: (1, 2, 3, 4, 6, 9, 13, 18, 24, 32),
          1024: (1, 2, 4, 6, 8, 12, 16, 20, 24, 32, 40, 48, 64)}
_TEXT = 77                     # condition tokens of the text-conditioned blocks
_NOVA = None


def _nova():
    global _NOVA
    if _NOVA is None:
        _NOVA = Nova(0)
    return _NOVA


# ---- the cases ------------------------------------------------------------------------------------------------------
def _step(name, dtype, B, C, heads, blocks, V, grid, prev, kv_len, hi, lo, variant=False):
    return {"name": name, "kind": "step", "dtype": dtype, "B": B, "C": C, "heads": heads, "blocks": blocks, "V": V,
            "grid": grid, "prev": prev, "kv_len": kv_len, "keep_hi": hi, "keep_lo": lo, "variant": variant}


def listed():
    return [
        # one small fp32 block, one image: the least that can be asked for; launches and host time
        _step("step-tiny-f32", "f32", 1, 64, 4, 1, 512, 16, 13, 424, 0.5, 0.5),
        # last scale of 256-pixel images, a small model at full depth, eight images
        _step("step-256px-b8", "bf16", 8, 1024, 16, 16, 4096, 16, 13, 424, 0.8, 0.4),
        # the scale before the last of a wide 256-pixel model (13 x 13, every size odd), sixteen images
        _step("step-256px-b16-wide", "bf16", 16, 1920, 30, 8, 4096, 13, 10, 255, 0.7, 0.3),
        # last scale of 512-pixel images, eight images, half of the tokens kept
        _step("step-512px-b8", "bf16", 8, 2304, 36, 6, 4096, 32, 24, 1216, 0.5, 0.5),
        # last scale of 1024-pixel images, two images: the largest step, every fourth of 32 blocks
        _step("step-1024px-b2", "bf16", 2, 2048, 16, 8, 4096, 64, 48, 6425, 0.6, 0.2),
        # first pruned scale of one 1024-pixel image, text-conditioned blocks: modulation, gates, unit-length queries
        # and keys, tanh GELU, cross-attention
        _step("step-1024px-b1-text", "bf16", 1, 2048, 16, 8, 4096, 32, 24, 1497, 0.6, 0.2, True),
        # one image, all scales, the serving loop of a small model: a graph per scale, nothing but small launches
        {"name": "image-256px-b1-graphs", "kind": "image", "B": 1, "C": 1024, "heads": 16, "blocks": 16, "V": 4096,
         "pixels": 256, "scales": 10, "pruned": 2, "keep_hi": 0.8, "keep_lo": 0.4, "graphs": True, "interp": 0},
        # the first ten scales of two 1024-pixel images (up to 32 x 32): dense scales of a wide model, the last pruned
        {"name": "image-1024px-b2-graphs", "kind": "image", "B": 2, "C": 2048, "heads": 16, "blocks": 8, "V": 4096,
         "pixels": 1024, "scales": 10, "pruned": 1, "keep_hi": 0.6, "keep_lo": 0.2, "graphs": True, "interp": 0},
        # eight images, eager calls, keep counts from the controller (each image its own), bicubic cache interpolation
        {"name": "image-256px-b8-controller", "kind": "image", "B": 8, "C": 1024, "heads": 16, "blocks": 8, "V": 4096,
         "pixels": 256, "scales": 10, "pruned": 2, "keep_hi": 0.7, "keep_lo": 0.7, "graphs": False, "interp": 2},
        # entropies of a dense scale: a few rows of a small scale, and fp32 logits of a large, odd codebook
        {"name": "tokens-small-bf16", "kind": "tokens", "dtype": "bf16", "B": 8, "N": 100, "V": 4096},
        {"name": "tokens-f32-20000", "kind": "tokens", "dtype": "f32", "B": 2, "N": 1024, "V": 20000},
        # entropies from the head at the largest scale
        {"name": "head-1024px-b2", "kind": "head", "B": 2, "N": 4096, "C": 2048, "V": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / 5e14


def draw(rng):
    """One more case of the same ranges; never dearer than the largest listed one."""
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(("step", "step", "step", "image", "image", "tokens", "head"))
        if kind == "step":
            pixels = rng.choice((256, 512, 1024))
            grids = _GRIDS[pixels]
            t = rng.randrange(len(grids) - 4, len(grids))
            dtype = "f32" if rng.random() < 0.1 else "bf16"
            dh = rng.choice((64, 128))
            C = 16 * rng.randint(2, 12) if dtype == "f32" else dh * _log_int(rng, 512 // dh, 2304 // dh)
            hi = rng.uniform(0.3, 0.95)
            case = {"kind": "step", "dtype": dtype, "B": _log_int(rng, 1, 16), "C": C,
                    "heads": C // 16 if dtype == "f32" else C // dh, "blocks": rng.randint(1, 8),
                    "V": rng.choice((512, 1024, 4096, 8192)), "grid": grids[t], "prev": grids[t - 1],
                    "kv_len": sum(g * g for g in grids[:t]), "keep_hi": hi, "keep_lo": rng.uniform(0.1, hi),
                    "variant": dtype == "bf16" and rng.random() < 0.3}
            if dtype == "f32" and case["grid"] > 16:
                continue
        elif kind == "image":
            pixels = rng.choice((256, 512, 1024))
            dh = rng.choice((64, 128))
            C = dh * _log_int(rng, 512 // dh, 2304 // dh)
            pruned = rng.randint(1, 3)
            hi = rng.uniform(0.4, 0.9)
            graphs = rng.random() < 0.6
            case = {"kind": "image", "B": _log_int(rng, 1, 8), "C": C, "heads": C // dh, "blocks": rng.randint(2, 8),
                    "V": rng.choice((512, 1024, 4096)), "pixels": pixels, "scales": rng.randint(6, 10), "pruned": pruned,
                    "keep_hi": hi, "keep_lo": rng.uniform(0.2, hi) if graphs else hi, "graphs": graphs,
                    "interp": rng.randint(0, 2)}
        elif kind == "tokens":
            case = {"kind": "tokens", "dtype": rng.choice(("f32", "bf16")), "B": _log_int(rng, 1, 16),
                    "N": rng.choice((1, 4, 9, 16, 25, 36, 64, 100, 169, 256, 576, 1024, 2304, 4096)),
                    "V": rng.choice((512, 1024, 4096, 8192, 16384, 32768, _log_int(rng, 500, 32000), _log_int(rng, 500, 32000)))}
        else:
            case = {"kind": "head", "B": _log_int(rng, 1, 16), "N": rng.choice((36, 100, 169, 256, 576, 1024, 2304, 4096)),
                    "C": 64 * _log_int(rng, 8, 36), "V": rng.choice((512, 1000, 4096, 4096, 8192, 16384))}
        if _cost(case) <= most:
            return case


# ---- sizes ----------------------------------------------------------------------------------------------------------
def _keep(case, j, N):
    hi, lo, L = case["keep_hi"], case["keep_lo"], case["blocks"]
    r = hi if L == 1 else hi + (lo - hi) * j / (L - 1)
    return max(0, min(N, int(math.ceil(r * N - 1e-9))))


def _image_scales(case):
    grids = _GRIDS[case["pixels"]][:case["scales"]]
    return grids, len(grids) - case["pruned"]          # scales from this index on are pruned


def _block_work(e, B, N, C, V, Nprev, P, k, pruned, variant, cache):
    """Bytes and flops of one block call sequence: entropy and selection (pruned scales), block, merge."""
    M = B * k
    w = 12 * C * C * e                                                        # the four projections' weights
    flops = 24.0 * M * C * C + 4.0 * M * (P + k) * C
    b = w + (B * N + M) * C * e                                               # x and the block's output
    b += (2 * B * P * C + 2 * M * C) * e                                      # prior keys / values read, new ones written
    b += (B * N * (2 if cache else 1) + (B * Nprev if k < N else 0)) * C * e  # out, new cache, prior cache
    if pruned:
        b += B * N * (V * e + 4 + 1) + 4 * M
    if variant:
        b += (2 * C * C + 6 * B * C + 2 * B * _TEXT * C) * e
        flops += 4.0 * M * C * C + 4.0 * M * _TEXT * C
    return b, flops


def work(case):
    if case["kind"] == "tokens":
        rows, e = case["B"] * case["N"], _SIZES[case["dtype"]]
        return {"bytes": rows * (case["V"] * e + 4.0) + 4 * case["B"], "flops": 0}
    if case["kind"] == "head":
        rows, C, V = case["B"] * case["N"], case["C"], case["V"]
        return {"bytes": 2.0 * (rows * C + V * C + V) + 4 * rows, "flops": 2.0 * rows * C * V}
    b = f = 0.0
    B, C, V = case["B"], case["C"], case["V"]
    if case["kind"] == "step":
        N, e = case["grid"] ** 2, _SIZES[case["dtype"]]
        for j in range(case["blocks"]):
            bb, ff = _block_work(e, B, N, C, V, case["prev"] ** 2, case["kv_len"], _keep(case, j, N), True,
                                 case["variant"], True)
            b, f = b + bb, f + ff
        return {"bytes": b, "flops": f}
    grids, first = _image_scales(case)
    kv = [0] * case["blocks"]
    for t, g in enumerate(grids):
        for j in range(case["blocks"]):
            N = g * g
            k = _keep(case, j, N) if t >= first else N
            bb, ff = _block_work(2, B, N, C, V, grids[max(t - 1, 0)] ** 2, kv[j], k, t >= first, False, t >= first - 1)
            b, f, kv[j] = b + bb, f + ff, kv[j] + k
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times the difference that another order of the sums makes (other tile shapes, K slices and key runs
    forced on the same inputs; entropies and the fp32 block against 64-bit arithmetic)."""
    if case["kind"] == "tokens":
        return {"rel": 1e-6, "max": 1e-5}              # seen: 6e-8, 1.7e-7 (exponentials of other widths sum in other orders)
    if case["kind"] == "head":
        return {"rel": 1e-6, "max": 1e-5}              # seen: 2.3e-7, 2.2e-6
    if case["kind"] == "step" and case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 1e-5}              # seen: 7e-8, 5e-7
    # bf16: rounding flips that travel on from block to block; largest in the residual caches (output minus input)
    if case["kind"] == "step":
        return {"rel": 2.5e-2, "max": 0.5}             # seen: 7e-3, 0.12
    return {"rel": 3e-2, "max": 0.5}                   # seen: 1.3e-2, 0.13 (all scales in a row)


# ---- inputs ---------------------------------------------------------------------------------------------------------
class _Draw:
    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dtype = dtype

    def normal(self, shape, std=1.0, dtype=None):
        t = torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)
        return (t.mul_(std) if std != 1.0 else t).to(dtype or self.dtype)

    def logits(self, B, N, V):
        s = torch.empty((B, N, 1), device="cuda").uniform_(math.log(0.1), math.log(10.0), generator=self.g).exp_()
        return torch.randn((B, N, V), generator=self.g, device="cuda").mul_(s).to(self.dtype)

    def weights(self, C):
        F = 4 * C
        shapes = {"w_qkv": (3 * C, C), "b_qkv": (3 * C,), "w_o": (C, C), "b_o": (C,),
                  "w_fc1": (F, C), "b_fc1": (F,), "w_fc2": (C, F), "b_fc2": (C,)}
        return {n: self.normal(s, 0.02) for n, s in shapes.items()}

    def variant(self, B, C, heads):
        ada = self.normal((B, 6, C), 0.2, torch.float32)
        ada[:, 2] += 1.0
        ada[:, 5] += 1.0
        cross = {"w_cq": self.normal((C, C), 0.02), "b_cq": self.normal((C,), 0.02), "w_co": self.normal((C, C), 0.02),
                 "b_co": self.normal((C,), 0.02), "k_text": pack_k_cache(self.normal((B, _TEXT, C)), heads, 128),
                 "v_text": pack_v_cache(self.normal((B, _TEXT, C)), heads, 128), "text_len": _TEXT}
        scale = torch.empty(heads, device="cuda").uniform_(4.0, 16.0, generator=self.g)
        return BlockVariant(gelu_tanh=True, qk_scale=scale, ada=ada.to(self.dtype), cross=cross)


def _prepare_step(case, seed):
    B, C, heads, L, N, P = case["B"], case["C"], case["heads"], case["blocks"], case["grid"] ** 2, case["kv_len"]
    dtype = _DTYPES[case["dtype"]]
    d = _Draw(seed, dtype)
    cap = (P + N + 63) // 64 * 64
    runner = StepRunner(_nova(), B=B, grid=case["grid"], prev_grid=case["prev"], C=C, heads=heads, kv_len=P,
                        kv_capacity=cap, dtype=dtype)
    dh = C // heads
    k_all = torch.zeros((L, B, heads, cap, dh), dtype=dtype, device="cuda")
    v_all = torch.zeros((L, B, heads, dh, cap), dtype=dtype, device="cuda")
    for j in range(L):
        keys = d.normal((B, heads, P, dh), dtype=torch.float32)
        if case["variant"]:                            # the cache of a unit-length-key model holds unit-length rows
            keys = torch.nn.functional.normalize(keys, dim=-1)
        k_all[j, :, :, :P] = keys.to(dtype)
        v_all[j, :, :, :, :P] = d.normal((B, heads, dh, P))
        runner.add_block(BlockState(k=_keep(case, j, N), logits=d.logits(B, N, case["V"]), weights=d.weights(C),
                                    k_cache=k_all[j], v_cache=v_all[j], cache_prev=d.normal((B, case["prev"] ** 2, C)),
                                    variant=d.variant(B, C, heads) if case["variant"] else None))
    return {"kind": "step", "runner": runner, "x": d.normal((B, N, C)), "k_all": k_all, "v_all": v_all}


def _prepare_image(case, seed):
    B, C, L = case["B"], case["C"], case["blocks"]
    d = _Draw(seed, torch.bfloat16)
    grids, first = _image_scales(case)
    runner = ImageRunner(_nova(), B=B, C=C, heads=case["heads"], grids=grids, dtype=torch.bfloat16,
                         weights=[d.weights(C) for _ in range(L)], interp=case["interp"])
    xs = [d.normal((B, g * g, C)) for g in grids]
    logits = {t: [d.logits(B, grids[t] ** 2, case["V"]) for _ in range(L)] for t in range(first, len(grids))}
    st = {"kind": "image", "runner": runner, "xs": xs, "first": first}
    if case["graphs"]:
        tables = {t: [_keep(case, j, grids[t] ** 2) for j in range(L)] for t in logits}
        st["plans"] = runner.plan_image(tables, logits, first_cache_scale=first - 1)
        for plan, x in zip(st["plans"], xs):
            plan.x.copy_(x)
            runner.capture(plan)
        return st
    # reduction ratio of every image: around 1 - keep, each image its own
    st["logits"] = logits
    ratio = torch.empty(B, device="cuda").uniform_(-0.1, 0.1, generator=d.g) + (1.0 - case["keep_hi"])
    st["ratio"] = ratio.clamp_(0.05, 0.9)
    return st


def prepare(case, seed):
    if case["kind"] == "step":
        return _prepare_step(case, seed)
    if case["kind"] == "image":
        return _prepare_image(case, seed)
    B, N, V = case["B"], case["N"], case["V"]
    st = {"kind": case["kind"], "entropy": torch.empty((B, N), dtype=torch.float32, device="cuda"),
          "mean": torch.empty((B,), dtype=torch.float32, device="cuda")}
    if case["kind"] == "tokens":
        st["logits"] = _Draw(seed, _DTYPES[case["dtype"]]).logits(B, N, V)
        return st
    d = _Draw(seed, torch.bfloat16)
    # hidden states of unit variance and a head whose logits spread over a few nats
    st["hidden"], st["w"], st["b"] = d.normal((B, N, case["C"])), d.normal((V, case["C"]), 0.05), d.normal((V,), 0.02)
    st["ws"] = torch.empty(max(_nova().head_entropy_workspace_bytes(N, B, V), 256), dtype=torch.uint8, device="cuda")
    return st


def run(state):
    kind = state["kind"]
    if kind == "tokens":
        _nova().entropy(state["logits"], state["entropy"], state["mean"])
        return [state["entropy"], state["mean"]]
    if kind == "head":
        _nova().head_entropy(state["hidden"], state["w"], state["b"], state["entropy"], state["ws"], state["mean"])
        return [state["entropy"], state["mean"]]
    r = state["runner"]
    if kind == "step":
        out = r.run_step(state["x"])
        return {"out": out, "k": state["k_all"], "v": state["v_all"], "cache": [b.cache_new for b in r.blocks],
                "kept": [b.kept_idx for b in r.blocks]}
    if "plans" in state:
        outs = []
        for plan, x in zip(state["plans"], state["xs"]):
            plan.x.copy_(x)
            outs.append(r.launch(plan))
        return {"out": outs, "k": r.k_cache, "v": r.v_cache, "cache": state["plans"][-1].cache_new}
    r.reset()
    outs, counts = [], []
    for t, x in enumerate(state["xs"]):
        pruned = t >= state["first"]
        res = r.run_scale(t, x, logits=state["logits"][t] if pruned else None, ratio_t=state["ratio"] if pruned else None,
                          keep_cache=t >= state["first"] - 1)
        outs.append(res.out)
        if pruned:
            counts.extend(res.k)
    return {"out": outs, "k": r.k_cache, "v": r.v_cache, "cache": res.block_cache, "counts": counts}
