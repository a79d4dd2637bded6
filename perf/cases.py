"""The work a user of the token-sparsity path has it do, as cases that can be timed and compared.

Four kinds of call sequence, each through the public binding (paper_2501_09767_amd.lemo):

  eliminate  Q, K of a layer -> token scores -> kept token list            (scoring sweeps + per-segment top-k)
  forward    the block over the kept tokens: attention, output projection added into the residual rows in place, MLP
             up-projection of the kept rows (fp32 layers: the two projections; the attention is a bf16 call)
  backward   gradients of the MLP projection (input gradient added into the kept rows, weight gradient) and the gradient
             of the selected rows scattered back
  blocks     block-wise scores -> mean threshold -> tokens of the blocks at or above it

Sizes are those of this repository's own configurations (workloads.CONFIGS), its tests' ragged lengths, and generic
layer widths; `draw` spreads over the ranges in between.
"""
import math

import torch

from paper_2501_09767_amd import lemo

CAUSAL_NO_SELF = lemo.CAUSAL | lemo.EXCLUDE_SELF


def listed():
    return [
        # one short fp32 sequence through a small model's layer: latency and launches decide
        _case("eliminate_1k_fp32", "eliminate", S=1024, H=4, H_kv=4, d=64, L=128, ratio=0.5, dtype="f32"),
        # a prompt of odd length through a grouped-query layer: segments with a ragged tail
        _case("eliminate_1000_gqa", "eliminate", S=1000, H=32, H_kv=8, d=128, L=512, ratio=0.5),
        # the usual fine-tuning length on a 32-head layer
        _case("eliminate_4k", "eliminate", S=4096, H=32, H_kv=32, d=128, L=512, ratio=0.5),
        # a bidirectional encoder with 64-wide heads, ragged length: no causal mask
        _case("eliminate_6001_d64_full", "eliminate", S=6001, H=16, H_kv=16, d=64, L=512, ratio=0.4, causal=False),
        # the long-context layer the path exists for
        _case("eliminate_32k", "eliminate", S=32768, H=32, H_kv=32, d=128, L=1024, ratio=0.3),
        # the block of a short prompt: a few hundred kept rows against full-size weights
        _case("forward_512", "forward", S=512, H=32, H_kv=32, d=128, C=4096, N=11008, L=512, ratio=0.5),
        # the block of an 8K-token training sample
        _case("forward_8k", "forward", S=8192, H=32, H_kv=32, d=128, C=4096, N=11008, L=512, ratio=0.4),
        # grouped-query block of a long sample of odd length
        _case("forward_12345_gqa", "forward", S=12345, H=32, H_kv=8, d=128, C=4096, N=14336, L=1024, ratio=0.3),
        # gradients of a small fp32 layer
        _case("backward_1k_fp32", "backward", S=1024, H=4, H_kv=4, d=64, C=256, N=256, L=128, ratio=0.5, dtype="f32"),
        # gradients of one fine-tuning sample of odd length
        _case("backward_2999", "backward", S=2999, H=32, H_kv=32, d=128, C=4096, N=11008, L=512, ratio=0.5),
        # gradients of the long-context layer
        _case("backward_32k", "backward", S=32768, H=32, H_kv=32, d=128, C=4096, N=11008, L=1024, ratio=0.3),
        # the paper's block-wise criterion at the usual fine-tuning length
        _case("blocks_4k", "blocks", S=4096, H=32, H_kv=32, d=128, b=64),
    ]


def _case(name, kind, *, S, H, H_kv, d, C=0, N=0, L=0, ratio=0.0, b=0, dtype="bf16", causal=True):
    return {"name": name, "kind": kind, "S": S, "H": H, "H_kv": H_kv, "d": d, "C": C, "N": N, "L": L, "ratio": ratio,
            "b": b, "dtype": dtype, "causal": causal}


# (query heads, key heads, head size, hidden size, MLP width) of the layers a case is drawn for
_LAYERS = [(4, 4, 64, 256, 256), (12, 12, 64, 768, 3072), (16, 16, 64, 1024, 4096), (16, 4, 128, 2048, 8192),
           (32, 32, 128, 4096, 11008), (32, 8, 128, 4096, 14336)]


def draw(rng):
    """One case of the same ranges: any of the layers above, 256 to 32768 tokens, no dearer than the dearest listed."""
    while True:
        kind = rng.choice(["eliminate", "eliminate", "forward", "forward", "backward", "backward", "blocks"])
        H, H_kv, d, C, N = rng.choice(_LAYERS)
        S = int(round(math.exp(rng.uniform(math.log(256), math.log(32768)))))
        if rng.random() < 0.3:
            S = max(256, S // 64 * 64)
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        causal = rng.random() < 0.8
        L = rng.choice([128, 256, 320, 512, 1000, 1024])
        ratio = round(rng.uniform(0.2, 0.6), 3)
        b = rng.choice([32, 64, 128])
        case = _case("", kind, S=S, H=H, H_kv=H_kv, d=d, dtype=dtype, causal=causal)
        del case["name"]
        if kind in ("forward", "backward"):
            case.update(C=C, N=N)
        if kind == "blocks":
            case.update(b=b)
        else:
            case.update(L=L, ratio=ratio)
        # binary32 products run at a sixteenth of the bf16 rate
        if work(case)["flops"] * (16 if dtype == "f32" else 1) <= work(listed()[4])["flops"]:
            return case


def _keep(case):
    """Kept tokens of every segment, and their total."""
    L, S = case["L"], case["S"]
    k = lemo.lemo_keep_k(L, case["ratio"])
    return k, lemo.lemo_kept_count(S, L, k)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    S, H, H_kv, d, C, N, L = (case[n] for n in ("S", "H", "H_kv", "d", "C", "N", "L"))

    def normal(*shape, std=1.0):
        t = torch.empty(shape, dtype=dt, device="cuda")
        # in pieces: no binary32 copy of a large tensor
        rows = max(1, (1 << 26) // max(1, t[0].numel()))
        for r in range(0, shape[0], rows):
            t[r:r + rows] = torch.randn(t[r:r + rows].shape, generator=gen, device="cuda") * std
        return t

    st = {"case": case, "flags": CAUSAL_NO_SELF if case["causal"] else lemo.EXCLUDE_SELF}
    if case["kind"] in ("eliminate", "blocks") or (case["kind"] == "forward" and dt == torch.bfloat16):
        # projections of unit-normal activations with weights of deviation 0.02 over a 4096-wide layer; a hundredth of
        # the keys is heavy (four times the norm), the columns that dominate an attention map
        st["Q"] = normal(S, H, d, std=1.28)
        st["K"] = normal(S, H_kv, d, std=1.28)
        heavy = torch.rand(S, generator=gen, device="cuda") < 0.01
        st["K"][heavy] *= 4
    if case["kind"] == "eliminate":
        st["k"], M = _keep(case)
        st["scores"] = torch.empty(S, dtype=torch.float32, device="cuda")
        st["kept"] = torch.empty(M, dtype=torch.int32, device="cuda")
        st["workspace"] = torch.empty(lemo.lemo_score_workspace_bytes(S, H, H_kv, d, lemo.F32 if dt == torch.float32 else lemo.BF16),
                                      dtype=torch.uint8, device="cuda")
        return st
    if case["kind"] == "blocks":
        st["kept"] = torch.full((S,), -1, dtype=torch.int32, device="cuda")
        st["workspace"] = torch.empty(lemo.lemo_score_blocks_workspace_bytes(S, H), dtype=torch.uint8, device="cuda")
        return st
    # a kept list as the elimination writes it: the k highest of every segment, ascending
    k, M = _keep(case)
    pick = torch.rand(S, generator=gen, device="cuda")
    parts = []
    for s in range(0, S, L):
        n = min(L, S - s)
        parts.append(pick[s:s + n].topk(lemo.lemo_kept_count(n, L, k)).indices.sort().values + s)
    st["kept"] = torch.cat(parts).to(torch.int32)
    assert st["kept"].numel() == M
    if case["kind"] == "forward":
        st["R"] = normal(S, C)                       # residual stream, updated in place
        st["W_out"] = normal(C, H * d, std=0.02)
        st["W_up"] = normal(N, C, std=0.02)
        st["Y"] = torch.empty((M, N), dtype=dt, device="cuda")
        if dt == torch.bfloat16:
            st["V"] = normal(S, H_kv, d)
            st["O"] = torch.empty((M, H, d), dtype=dt, device="cuda")
            st["workspace"] = torch.empty(lemo.lemo_kept_attention_workspace_bytes(M, H_kv, d), dtype=torch.uint8, device="cuda")
        else:
            st["O"] = normal(M, H, d)
    else:
        st["X"] = normal(S, C)
        st["W"] = normal(N, C, std=0.02)
        if dt == torch.float32:
            st["Wt"] = st["W"].t().contiguous()      # the fp32 input gradient takes the weight transposed
        st["dY"] = normal(M, N, std=0.05)
        st["G"] = normal(M, C)
        st["dX"] = torch.zeros((S, C), dtype=dt, device="cuda")
        st["dW"] = torch.empty((N, C), dtype=dt, device="cuda")
        need = lemo.lemo_gather_gemm_dw_workspace_bytes(M, C, N, lemo.F32 if dt == torch.float32 else lemo.BF16)
        st["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "eliminate":
        lemo.lemo_score_segments(st["Q"], st["K"], case["L"], st["flags"], scores=st["scores"], workspace=st["workspace"])
        lemo.lemo_select_topk(st["scores"], case["L"], st["k"], kept_idx=st["kept"])
        return st["scores"], st["kept"]
    if case["kind"] == "blocks":
        score_blocks, token_blocks = lemo.lemo_score_blocks(st["Q"], st["K"], case["b"], st["flags"], workspace=st["workspace"])
        threshold = lemo.lemo_threshold_init(token_blocks)
        kept, count = lemo.lemo_select_threshold(token_blocks, case["S"], case["b"], threshold, kept_idx=st["kept"])
        return score_blocks, token_blocks, threshold, kept, count
    if case["kind"] == "forward":
        O, M = st["O"], st["kept"].numel()
        if case["dtype"] == "bf16":
            lemo.lemo_kept_attention(st["Q"], st["K"], st["V"], st["kept"], flags=st["flags"] & lemo.CAUSAL, O=O, workspace=st["workspace"])
        lemo.lemo_gather_gemm_add(O.view(M, -1), None, st["W_out"], st["R"], st["kept"])
        lemo.lemo_gather_gemm(st["R"], st["kept"], st["W_up"], Y=st["Y"])
        return O, st["R"], st["Y"]
    if case["dtype"] == "bf16":
        lemo.lemo_gather_gemm_dx(st["dY"], st["W"], st["dX"], st["kept"])
    else:
        lemo.lemo_gather_gemm_add(st["dY"], None, st["Wt"], st["dX"], st["kept"])
    lemo.lemo_gather_gemm_dw(st["dY"], st["X"], st["kept"], dW=st["dW"], workspace=st["workspace"])
    lemo.lemo_scatter_grad(st["G"], st["kept"], st["dX"])
    return st["dX"], st["dW"]


def work(case):
    """Bytes and flops of one pass: every input read once, every output written once, the products the definition needs
    (scoring: Q K^T twice, since a column sum needs the final normaliser of every row and the matrix is not stored)."""
    e = 4 if case["dtype"] == "f32" else 2
    S, H, H_kv, d, C, N = (case[n] for n in ("S", "H", "H_kv", "d", "C", "N"))
    qk_bytes = e * S * d * (H + H_kv)

    def pairs(n):
        return H * (n * (n + 1) // 2 if case["causal"] else n * n)

    if case["kind"] == "eliminate":
        _, M = _keep(case)
        return {"bytes": qk_bytes + 4 * S + 4 * M, "flops": 4 * d * pairs(S)}
    if case["kind"] == "blocks":
        nb = -(-S // case["b"])
        return {"bytes": qk_bytes + 4 * nb * nb + 4 * nb + 4 * S, "flops": 4 * d * pairs(S)}
    _, M = _keep(case)
    if case["kind"] == "forward":
        b = e * (M * H * d + C * H * d + 2 * M * C + N * C + M * N) + 4 * M
        f = 2 * M * C * H * d + 2 * M * C * N
        if case["dtype"] == "bf16":
            b += e * M * d * (H + 2 * H_kv)
            f += 4 * d * pairs(M)
        return {"bytes": b, "flops": f}
    return {"bytes": e * (M * N + 2 * N * C + M * C + 3 * M * C) + 4 * M, "flops": 4 * M * N * C}


def tolerance(case):
    """About four times what the path shows against the same computation in 64 bits.  Scores (2-norm 9e-7, worst value
    5e-6): binary32 logits of a few tens carry 2^-24 relative error each into the exponential; kept indices: ties at the
    cut.  fp32 products 4e-7 / 3e-6.  bf16 gradients 3e-5 / 2^-7: binary32 sums in another order turn a few of the single
    roundings at the stores (two for the rows that are added to twice).  bf16 forward 3e-3 / 2e-2: the probabilities and
    the intermediates that the next product reads are rounded as well."""
    if case["kind"] in ("eliminate", "blocks"):
        return {"rel": 5e-6, "max": 5e-5, "differ": 0.01}
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    if case["kind"] == "backward":
        return {"rel": 5e-4, "max": 3.2e-2}
    return {"rel": 1e-2, "max": 8e-2}


def exact(case, seed):
    """What the first `run` on these inputs returns, in 64 bits (whole results: no value of their own, None)."""
    st = prepare(case, seed)
    S, H, H_kv, d = (case[n] for n in ("S", "H", "H_kv", "d"))
    rows = max(1, (1 << 26) // S)

    def probabilities(h, r0, r1, tokens, exclude_self):
        """Rows r0..r1 of softmax(Q K^T / sqrt(d)) of query head h over `tokens` (all if None)."""
        q, k = (st[n] if tokens is None else st[n][tokens] for n in ("Q", "K"))
        q, k = q[r0:r1, h].double(), k[:, h * H_kv // H].double()
        x = q @ k.t().contiguous() / math.sqrt(d)
        i = torch.arange(r0, r1, device="cuda").unsqueeze(1)
        j = torch.arange(k.shape[0], device="cuda").unsqueeze(0)
        if case["causal"]:
            x.masked_fill_(j > i, -math.inf)
        x = torch.softmax(x, dim=1)
        return x.masked_fill_(j == i, 0.0) if exclude_self else x

    if case["kind"] == "eliminate":
        scores = torch.zeros(S, dtype=torch.float64, device="cuda")
        for h in range(H):
            for r in range(0, S, rows):
                scores += probabilities(h, r, min(S, r + rows), None, True).sum(0)
        return scores / H, None
    if case["kind"] == "blocks":
        b = case["b"]
        nb = -(-S // b)
        score_blocks = torch.zeros((nb, nb), dtype=torch.float64, device="cuda")
        rows = max(b, rows // b * b)
        for r in range(0, S, rows):
            n = min(rows, S - r)
            mean = torch.zeros((-(-n // b) * b, nb * b), dtype=torch.float64, device="cuda")
            for h in range(H):
                mean[:n, :S] += probabilities(h, r, r + n, None, True)
            score_blocks[r // b:r // b + mean.shape[0] // b] = mean.view(-1, b, nb, b).amax(dim=(1, 3)) / H
        token_blocks = score_blocks.sum(0)
        return score_blocks, token_blocks, token_blocks.mean().reshape(1), None, None
    kept = st["kept"].long()
    M = kept.numel()
    if case["kind"] == "forward":
        O = st["O"].double()
        if case["dtype"] == "bf16":
            for h in range(H):
                v = st["V"][kept, h * H_kv // H].double()
                for r in range(0, M, rows):
                    O[r:r + rows, h] = probabilities(h, r, min(M, r + rows), kept, False) @ v
        R = st["R"].double()
        R[kept] += O.view(M, -1) @ st["W_out"].double().t().contiguous()
        return O, R, R[kept] @ st["W_up"].double().t().contiguous()
    dY = st["dY"].double()
    dX = st["dX"].double()
    dX[kept] += dY @ st["W"].double() + st["G"].double()
    return dX, dY.t().contiguous() @ st["X"][kept].double()
