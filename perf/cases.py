"""The work that users of this library have it do, as timed cases.

A case is one call, or one short sequence of calls, through the public Python
entry points (``paper_2407_02068_amd.lpv`` and ``encoder``) at the sizes of the
DeiT family (192 / 384 / 768 channels, 197 tokens per image): inference of the
pruned linear layers in each element type, the dense layer beside them, the
backward of finetuning, attention, pruning and packing a weight, the delta
curve of the sparsity allocation, and a whole 12-block encoder.

Inputs are synthetic (X ~ N(0, 1), W and bias ~ N(0, 0.02), gradients ~
N(0, 1)), drawn on the GPU from the seed alone.
"""
import math

import torch

from paper_2407_02068_amd import encoder, lpv

TOKENS = 197  # 224 x 224 image, 16 x 16 patches, plus the class token
DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}


def listed():
    return [
        # one image through the first MLP layer of the smallest model, in fp32
        # with the finest blocks: the smallest call, all latency
        _linear("tiny_fc1_f32_b1", TOKENS, 768, 192, 16, 16, 50, "f32"),
        # one image through the largest model's first MLP layer: single-image
        # serving, too few token tiles to fill the chip
        _linear("b_fc1_gelu_b1", TOKENS, 3072, 768, 32, 32, 50, "bf16", gelu=True),
        # DeiT-S first MLP layer with its activation at batch 64: an ordinary
        # inference batch
        _linear("s_fc1_gelu_b64", 64 * TOKENS, 1536, 384, 32, 32, 50, "bf16", gelu=True),
        # DeiT-B first MLP layer at batch 256, half of the blocks kept: the
        # throughput workload of the benchmark
        _linear("b_fc1_b256", 256 * TOKENS, 3072, 768, 32, 32, 50, "bf16"),
        # DeiT-B second MLP layer (long reduction, few outputs) in fp16 with
        # tall blocks and a high sparsity at batch 128
        _linear("b_fc2_f16_b128", 128 * TOKENS, 768, 3072, 64, 32, 70, "f16"),
        # an unpruned layer next to pruned ones: the qkv projection at batch 32
        {"name": "b_qkv_dense_b32", "kind": "dense", "M": 32 * TOKENS, "N": 2304, "K": 768,
         "dtype": "bf16", "gelu": False},
        # finetuning the pruned model: the backward of DeiT-B fc1, micro-batch 64
        _backward("b_fc1_backward_b64", 64 * TOKENS, 3072, 768, 32, 32, 50, "bf16"),
        # the same for the smallest model in fp32 with 16 x 16 blocks
        _backward("tiny_fc1_backward_f32_b16", 16 * TOKENS, 768, 192, 16, 16, 50, "f32"),
        # the attention between the pruned layers of DeiT-B at batch 64
        {"name": "b_attention_b64", "kind": "attention", "n_seq": 64, "T": TOKENS, "H": 12,
         "dtype": "bf16"},
        # pruning one layer: Taylor scores and top-k mask, the packed weight,
        # and its transpose for the input gradient of finetuning
        {"name": "b_fc1_prune", "kind": "prune", "N": 3072, "K": 768, "b_r": 32, "b_c": 32,
         "sparsity": 50, "dtype": "bf16"},
        # the delta curve of one layer from 64 calibration samples, one of many
        # such calls of the sparsity allocation
        {"name": "b_fc1_delta_64", "kind": "delta", "N": 3072, "K": 768, "b_r": 32, "b_c": 32,
         "n_samples": 64, "n_points": 21, "dtype": "bf16"},
        # a whole pruned DeiT-B encoder at batch 8, captured once and replayed:
        # the serving loop
        {"name": "b_encoder_b8", "kind": "encoder", "batch": 8, "T": TOKENS, "H": 12, "blocks": 12,
         "b": 32, "dtype": "bf16"},
    ]


def _linear(name, M, N, K, b_r, b_c, sparsity, dtype, gelu=False):
    return {"name": name, "kind": "linear", "M": M, "N": N, "K": K, "b_r": b_r, "b_c": b_c,
            "sparsity": sparsity, "dtype": dtype, "gelu": gelu, "skew": False}


def _backward(name, M, N, K, b_r, b_c, sparsity, dtype):
    return {"name": name, "kind": "backward", "M": M, "N": N, "K": K, "b_r": b_r, "b_c": b_c,
            "sparsity": sparsity, "dtype": dtype}


# ---------------------------------------------------------------- drawn cases

# (output, input) widths of the layers of an encoder block, in channels D
LAYERS = ((3, 1), (1, 1), (4, 1), (1, 4))
# the largest listed pass: kept multiply-adds x 2, and bytes of X and Y
MOST_FLOPS = 119e9
MOST_BYTES = 390e6


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over the logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _tokens(rng, lo, hi, N, K, density, dtype):
    """Token rows: whole images or any count from one 7 x 7 window up, within the
    largest listed cost."""
    hi = min(hi, MOST_FLOPS / (2 * N * K * density), MOST_BYTES / ((N + K) * SIZE[dtype]))
    M = _spread(rng, lo, max(lo, int(hi)))
    if rng.random() < 0.5 and M >= TOKENS:
        M = M // TOKENS * TOKENS
    return M


def draw(rng):
    kind = rng.choice(["linear"] * 5 + ["dense"] * 2 + ["backward"] * 2 +
                      ["attention", "prune", "delta", "encoder"])
    dtype = rng.choice(["bf16", "bf16", "f16"])
    D = rng.choice([192, 384, 768])
    n, k = rng.choice(LAYERS)
    b_r, b_c = rng.choice([16, 32, 64]), rng.choice([16, 32, 64])
    if rng.random() < 0.5:
        b_c = b_r
    sparsity = rng.randint(30, 90)
    if kind == "attention":
        T = rng.choice([49, TOKENS, TOKENS, rng.randint(16, 512)])
        H = D // 64
        return {"kind": kind, "n_seq": _spread(rng, 1, 64 * 12 * TOKENS // (H * T)), "T": T, "H": H,
                "dtype": dtype}
    if kind == "encoder":
        return {"kind": kind, "batch": _spread(rng, 1, 8), "T": TOKENS, "H": D // 64, "blocks": 12,
                "b": rng.choice([16, 32, 64]), "dtype": "bf16"}
    if rng.random() < 0.2:
        dtype, D = "f32", min(D, 384)
    N, K = n * D, k * D
    if kind == "prune":
        return {"kind": kind, "N": N, "K": K, "b_r": b_r, "b_c": b_c, "sparsity": sparsity,
                "dtype": dtype}
    if kind == "delta":
        most = int(min(64, 64 * 3072 * 768 * 2 / (N * K * SIZE[dtype])))
        return {"kind": kind, "N": N, "K": K, "b_r": b_r, "b_c": b_c,
                "n_samples": rng.randint(8, max(8, most)), "n_points": rng.choice([11, 21, 41]),
                "dtype": dtype}
    # fp32 layers are the small models'
    top = 256 * TOKENS if dtype != "f32" else 64 * TOKENS
    if kind == "dense":
        return {"kind": kind, "M": _tokens(rng, 49, top // 2, N, K, 1.0, dtype), "N": N, "K": K,
                "dtype": dtype, "gelu": rng.random() < 0.3}
    density = 1 - sparsity / 100
    if kind == "backward":
        return {"kind": kind, "M": _tokens(rng, 49, top // 4, N, K, 2 * density, dtype), "N": N,
                "K": K, "b_r": b_r, "b_c": b_c, "sparsity": sparsity, "dtype": dtype}
    return {"kind": kind, "M": _tokens(rng, 49, top, N, K, density, dtype), "N": N, "K": K,
            "b_r": b_r, "b_c": b_c, "sparsity": sparsity, "dtype": dtype,
            "gelu": rng.random() < 0.3, "skew": rng.random() < 0.3}


# ---------------------------------------------------------------- inputs

class _Inputs:
    """Seeded tensors on the GPU."""

    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = DTYPE[dtype]

    def normal(self, *shape, std=1.0):
        t = torch.randn(shape, generator=self.g, device="cuda")
        return (t if std == 1.0 else t * std).to(self.dtype)

    def mask(self, R, C, sparsity, skew=False):
        """The given share of the blocks dropped at random; skew: some block
        rows keep most of their blocks and others few."""
        s = torch.rand((R, C), generator=self.g, device="cuda")
        if skew:
            s = s + torch.randn((R, 1), generator=self.g, device="cuda") * 0.5
        keep = ((100 - sparsity) * R * C + 99) // 100
        m = torch.zeros(R * C, dtype=torch.uint8, device="cuda")
        m[s.reshape(-1).topk(keep).indices] = 1
        return m.reshape(R, C)


def _parts(case, seed):
    """The plain tensors of a case (the handles and plans are built from them)."""
    r = _Inputs(seed, case["dtype"])
    kind = case["kind"]
    if kind == "attention":
        return {"qkv": r.normal(case["n_seq"] * case["T"], 3 * 64 * case["H"])}
    if kind == "encoder":
        D, b = 64 * case["H"], case["b"]
        layers = []
        for _ in range(case["blocks"]):
            for j, (n, k) in enumerate(LAYERS):
                N, K = n * D, k * D
                s = int(torch.randint(30, 81, (1,), generator=r.g, device="cuda"))
                layers.append((r.normal(N, K, std=0.02), r.mask(N // b, K // b, s, skew=True),
                               r.normal(N, std=0.02), j == 2))
        return {"layers": layers, "gamma": 1 + r.normal(D, std=0.1), "beta": r.normal(D, std=0.1),
                "x0": r.normal(case["batch"] * case["T"], D)}
    N, K = case["N"], case["K"]
    p = {"W": r.normal(N, K, std=0.02)}
    if kind in ("linear", "backward"):
        p["mask"] = r.mask(N // case["b_r"], K // case["b_c"], case["sparsity"],
                           case.get("skew", False))
    if kind in ("linear", "dense"):
        p["X"], p["bias"] = r.normal(case["M"], K), r.normal(N, std=0.02)
    elif kind == "backward":
        p["X"], p["G"] = r.normal(case["M"], K), r.normal(case["M"], N)
    elif kind == "prune":
        p["G"] = r.normal(N, K)
    elif kind == "delta":
        p["grad"], p["samples"] = r.normal(N, K), r.normal(case["n_samples"], N, K)
    return p


def _points(case):
    n = case["n_points"]
    return [100 * i // (n - 1) for i in range(n)]


def prepare(case, seed):
    p = _parts(case, seed)
    kind = case["kind"]
    s = {"kind": kind, "epi": "gelu" if case.get("gelu") else None}
    if kind == "attention":
        s.update(p, out=torch.empty(case["n_seq"] * case["T"], 64 * case["H"],
                                    dtype=p["qkv"].dtype, device="cuda"),
                 n_seq=case["n_seq"], T=case["T"], H=case["H"])
    elif kind == "encoder":
        lins = [encoder.Linear("%d" % i, W, mask, bias, case["b"], case["b"], gelu)
                for i, (W, mask, bias, gelu) in enumerate(p["layers"])]
        s["chain"] = encoder.EncoderChain(lins, case["batch"], case["T"], case["H"], p["gamma"],
                                          p["beta"])
        s["x0"] = p["x0"]
        s["graph"], s["out"] = s["chain"].capture(s["x0"])
    elif kind == "prune":
        s.update(p, b_r=case["b_r"], b_c=case["b_c"], sparsity=case["sparsity"])
    elif kind == "delta":
        s.update(p, b_r=case["b_r"], b_c=case["b_c"], pcts=_points(case))
        s["out"] = torch.empty(case["n_points"], dtype=torch.float64, device="cuda")
        s["workspace"] = torch.empty(
            lpv.delta_curve_workspace_size(case["N"], case["K"], case["b_r"], case["b_c"],
                                           case["n_samples"], case["n_points"]),
            dtype=torch.uint8, device="cuda")
    elif kind == "backward":
        h = lpv.bsr_pack(p["W"], p["mask"], case["b_r"], case["b_c"])
        s.update(h=h, ht=lpv.bsr_transpose(h), X=p["X"], G=p["G"])
        s["dX"] = torch.empty_like(p["X"])
        s["dW"] = torch.empty((h.nnzb, case["b_r"], case["b_c"]), dtype=h.dtype, device="cuda")
        s["db"] = torch.empty(case["N"], dtype=h.dtype, device="cuda")
    else:
        s.update(X=p["X"], bias=p["bias"],
                 Y=torch.empty(case["M"], case["N"], dtype=p["X"].dtype, device="cuda"))
        if kind == "linear":
            s["h"] = lpv.bsr_pack(p["W"], p["mask"], case["b_r"], case["b_c"])
        else:
            s["W"] = p["W"]
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    kind = s["kind"]
    if kind == "linear":
        return lpv.bsr_linear(s["h"], s["X"], s["bias"], s["Y"], epi=s["epi"])
    if kind == "dense":
        return lpv.dense_linear(s["W"], s["X"], s["bias"], s["Y"], epi=s["epi"])
    if kind == "backward":
        lpv.bsr_linear(s["ht"], s["G"], Y=s["dX"])
        lpv.grad_w(s["h"], s["G"], s["X"], out=s["dW"])
        lpv.bias_grad(s["G"], out=s["db"])
        return {"dX": s["dX"], "dW": s["dW"], "db": s["db"]}
    if kind == "attention":
        return lpv.attention(s["qkv"], s["n_seq"], s["T"], s["H"], out=s["out"])
    if kind == "prune":
        mask, scores = lpv.mask_topk(s["W"], s["b_r"], s["b_c"], s["sparsity"], G=s["G"])
        h = lpv.bsr_pack(s["W"], mask, s["b_r"], s["b_c"])
        ht = lpv.bsr_transpose(h)
        s["handles"] = (h, ht)
        return {"mask": mask, "scores": scores, "bsr": lpv.bsr_export(h),
                "transposed": lpv.bsr_export(ht)}
    if kind == "delta":
        return lpv.delta_curve(s["W"], s["grad"], s["samples"], s["b_r"], s["b_c"], 0.1, s["pcts"],
                               out=s["out"], workspace=s["workspace"])
    s["graph"].replay()
    return s["out"]


# ---------------------------------------------------------------- what a pass cannot do without

def _kept(case):
    """Kept elements of a layer's weight."""
    n = (case["N"] // case["b_r"]) * (case["K"] // case["b_c"])
    return ((100 - case["sparsity"]) * n + 99) // 100 * case["b_r"] * case["b_c"]


def work(case):
    kind, es = case["kind"], SIZE[case["dtype"]]
    if kind == "attention":
        rows, D = case["n_seq"] * case["T"], 64 * case["H"]
        return {"bytes": 4 * rows * D * es, "flops": 4 * rows * case["T"] * D}
    if kind == "encoder":
        D = 64 * case["H"]
        M = case["batch"] * case["T"]
        kept = case["blocks"] * 12 * D * D * 0.45  # sparsities average 55%
        return {"bytes": int(kept * es + 3 * M * D * es),
                "flops": int(2 * M * kept + case["blocks"] * 4 * M * case["T"] * D)}
    N, K = case["N"], case["K"]
    if kind == "prune":
        # W and its gradient in; scores, mask, and both packed forms out
        n = (N // case["b_r"]) * (K // case["b_c"])
        return {"bytes": 2 * N * K * es + 9 * n + 2 * _kept(case) * es, "flops": 2 * N * K}
    if kind == "delta":
        v = case["n_samples"] + 2
        return {"bytes": v * N * K * es, "flops": 2 * v * N * K}
    M = case["M"]
    kept = N * K if kind == "dense" else _kept(case)
    if kind == "backward":
        return {"bytes": (M * (N + 2 * K) + 2 * kept + N) * es, "flops": 4 * M * kept + M * N}
    return {"bytes": (M * (N + K) + kept + N) * es, "flops": 2 * M * kept}


# About four times the largest error that a pass shows against exact().
def tolerance(case):
    kind = case["kind"]
    if kind == "prune":
        return "exact"  # the mask and the raw weight bits; the scores' order of additions is fixed
    if kind == "delta":
        return {"rel": 1e-14}  # float64 sums
    if kind == "encoder":
        return {"rel": 0.03, "max": 0.3}  # roundings of one layer travel through all that follow
    if case["dtype"] == "f32":
        return {"rel": 5e-6}
    return {"rel": 8e-3 if case["dtype"] == "bf16" else 1e-3}


# ---------------------------------------------------------------- the same in 64 bits

def _expand(W, mask, b_r, b_c):
    keep = mask.bool().repeat_interleave(b_r, 0).repeat_interleave(b_c, 1)
    return torch.where(keep, W.double(), torch.zeros((), dtype=torch.float64, device=W.device))


def _affine(X, W, bias, gelu):
    z = X.double() @ W.t().contiguous() + bias.double()
    return torch.nn.functional.gelu(z) if gelu else z


def _attend(qkv, n_seq, T, H):
    q, k, v = qkv.double().reshape(n_seq, T, 3, H, 64).permute(2, 0, 3, 1, 4).contiguous()
    out = torch.empty_like(q)
    for i in range(n_seq):  # one sequence at a time: small score matrices
        w = torch.softmax(q[i] @ k[i].transpose(1, 2).contiguous() / 8.0, dim=-1)
        out[i] = w @ v[i]
    return out.permute(0, 2, 1, 3).reshape(n_seq * T, H * 64)


def _norm(x, gamma, beta, eps=1e-6):
    return torch.nn.functional.layer_norm(x, (x.shape[1],), gamma.double(), beta.double(), eps)


def _blocks(t, b_r, b_c):
    """N x K -> R x C x b_r x b_c."""
    N, K = t.shape
    return t.reshape(N // b_r, b_r, K // b_c, b_c).permute(0, 2, 1, 3)


def _bsr(W, mask, b_r, b_c):
    m = mask.bool()
    row_ptr = torch.zeros(m.shape[0] + 1, dtype=torch.int32, device=W.device)
    row_ptr[1:] = m.sum(1).cumsum(0)
    return row_ptr, m.nonzero()[:, 1].int(), _blocks(W, b_r, b_c)[m].double()


def _best(scores, sparsity):
    """The best-ranked blocks (larger score first, ties to the lower index)."""
    flat = scores.reshape(-1)
    keep = ((100 - sparsity) * flat.numel() + 99) // 100
    m = torch.zeros(flat.numel(), dtype=torch.uint8, device=flat.device)
    m[torch.sort(flat, descending=True, stable=True).indices[:keep]] = 1
    return m.reshape(scores.shape)


def exact(case, seed):
    p = _parts(case, seed)
    kind = case["kind"]
    if kind == "attention":
        return _attend(p["qkv"], case["n_seq"], case["T"], case["H"])
    if kind == "encoder":
        x = p["x0"].double()
        A = _norm(x, p["gamma"], p["beta"])
        ws = [(_expand(W, m, case["b"], case["b"]), bias, gelu) for W, m, bias, gelu in p["layers"]]
        for i in range(0, len(ws), 4):
            att = _attend(_affine(A, *ws[i]), case["batch"], case["T"], case["H"])
            x = x + _affine(att, *ws[i + 1])
            A = _norm(x, p["gamma"], p["beta"])
            x = x + _affine(_affine(A, *ws[i + 2]), *ws[i + 3])
            A = _norm(x, p["gamma"], p["beta"])
        return x, A
    W = p["W"]
    if kind == "prune":
        scores = _blocks((W.double() * p["G"].double()).abs(), case["b_r"], case["b_c"]).mean((2, 3))
        mask = _best(scores, case["sparsity"])
        return {"mask": mask, "scores": scores, "bsr": _bsr(W, mask, case["b_r"], case["b_c"]),
                "transposed": _bsr(W.t().contiguous(), mask.t().contiguous(), case["b_c"],
                                   case["b_r"])}
    if kind == "delta":
        Wd, grad = W.double(), p["grad"].double()
        scores = _blocks((Wd * grad).abs(), case["b_r"], case["b_c"]).mean((2, 3))
        out = []
        for pct in _points(case):
            dW = -Wd * (1 - _expand(torch.ones_like(Wd), _best(scores, pct), case["b_r"], case["b_c"]))
            f = torch.stack([(g.double() * dW).sum() for g in p["samples"]])
            out.append((grad * dW).sum() + 0.5 * (0.1 * (dW * dW).sum() + (f * f).mean()))
        return torch.stack(out)
    if kind == "dense":
        return _affine(p["X"], W.double(), p["bias"], case["gelu"])
    We = _expand(W, p["mask"], case["b_r"], case["b_c"])
    if kind == "linear":
        return _affine(p["X"], We, p["bias"], case["gelu"])
    G, X = p["G"].double(), p["X"].double()
    dW = _blocks(G.t().contiguous() @ X, case["b_r"], case["b_c"])[p["mask"].bool()]
    return {"dX": G @ We, "dW": dW, "db": G.sum(0)}
