"""The work this library is used for, as a list of measurable cases.

A case names one call, or one short sequence of calls, through the public binding (`paper_2509_16518_amd.fgattn`) with
its sizes and its mask recipe.  `listed()` holds the representative ones, `draw()` gives more of the same ranges,
`prepare()` builds what a program holds before the call, `run()` makes the call, `work()` and `tolerance()` say what the
call cannot do without and how far two correct implementations may be apart.

Kinds (`op`):
  forward   one sparse forward pass over a given CSR mask (ordering pre-pass included)
  dense     the same tensors at 0% sparsity
  mask      the top-p mask from block means: select, then emit into a buffer kept for the longest possible mask
  layer     mask and forward pass one after the other, as a layer that chooses its own mask runs them
  grouped   grouping of small query tiles (greedy, by distance), then the forward pass over the groups
Tokens lie on a (T, Hg, Wg) grid; masks are a window around a query block's centre token plus random fill to the stated
density (`skew`: the density varies by head, lognormally, and by block, +-50%).  Tensors are bf16, [B, H, L, d] by shape;
`layout` says how they lie in memory.
"""
import math

import torch

from paper_2509_16518_amd import fgattn as F


def _case(op, B, H, grid, d, M, N, density=0.30, window=(2, 4, 4), skew=False, layout="bhld", top_p=0.9):
    return {"op": op, "B": B, "H": H, "T": grid[0], "Hg": grid[1], "Wg": grid[2], "d": d, "M": M, "N": N, "density": density,
            "dt": window[0], "dh": window[1], "dw": window[2], "skew": skew, "layout": layout, "top_p": top_p}


def listed():
    wan, hunyuan, clip = (21, 30, 52), (33, 45, 80), (5, 17, 31)
    named = {
        # the smallest configuration: 128 work items of ten key tiles, where launches and latency count
        "tiny-16x1": _case("forward", 1, 2, (4, 16, 16), 64, 16, 1, window=(1, 3, 3)),
        # a short clip in a small model: batch of two, tokens-first storage, head dim 64, short last key group
        "clip-32x8": _case("forward", 2, 8, clip, 64, 32, 8, window=(1, 3, 3), layout="blhd"),
        # one attention layer of the Wan-2.1-1.3B shape, single keys, 70% sparsity (the benchmark's workload)
        "wan-64x1": _case("forward", 1, 12, wan, 128, 64, 1),
        # the Wan-14B shape with key groups of 8 and strongly uneven lists
        "wan-skew-64x8": _case("forward", 1, 40, wan, 128, 64, 8, skew=True),
        # square tiles smaller than the 128 rows that a group holds, run natively; the last key group is short
        "wan-32x32": _case("forward", 1, 12, wan, 128, 32, 32),
        # the HunyuanVideo shape: the longest sequence, 80% sparsity (the largest call)
        "hunyuan-128x1": _case("forward", 1, 24, hunyuan, 128, 128, 1, density=0.20, window=(2, 6, 6)),
        # layers and steps that stay dense
        "wan-dense-128": _case("dense", 1, 12, wan, 128, 128, 1, density=1.0),
        "clip-dense-64": _case("dense", 2, 8, clip, 64, 64, 1, density=1.0, layout="blhd"),
        # choosing the mask by top-p, one key at a time, at both video shapes (rows of 32 760 and 118 800 scores)
        "wan-mask-64x1": _case("mask", 1, 12, wan, 128, 64, 1),
        "hunyuan-mask-128x1": _case("mask", 1, 24, hunyuan, 128, 128, 1),
        # a whole layer at a middling length: block mask chosen from the layer's own Q and K, then the forward pass
        "layer-64x64": _case("layer", 1, 12, (6, 30, 52), 128, 64, 64, layout="blhd"),
        # small tiles merged into groups by the distance of their key sets
        "wan-grouped-16x16": _case("grouped", 1, 12, wan, 128, 16, 16),
    }
    return [dict(case, name=name) for name, case in named.items()]


def draw(rng):
    op = rng.choices(("forward", "dense", "mask", "layer", "grouped"), (10, 3, 4, 2, 2))[0]
    while True:
        grid = (rng.randint(1, 34), int(round(math.exp(rng.uniform(math.log(8), math.log(48))))),
                int(round(math.exp(rng.uniform(math.log(12), math.log(84))))))
        case = _case(op, rng.choice((1, 1, 1, 2)), int(round(math.exp(rng.uniform(0.0, math.log(40))))), grid,
                     rng.choice((64, 128, 128)), rng.choice((16, 32, 64, 64, 128)), rng.choice((1, 1, 8, 16, 32, 64, 128)),
                     density=rng.uniform(0.08, 0.55), window=(rng.randint(0, 2), rng.randint(1, 6), rng.randint(1, 6)),
                     skew=rng.random() < 0.3, layout=rng.choice(("bhld", "blhd")), top_p=rng.choice((0.8, 0.9, 0.95)))
        if op == "dense":
            case.update(M=rng.choice((64, 128)), N=1, density=1.0, skew=False)
        elif op == "grouped":
            case.update(M=rng.choice((16, 32, 64)), N=rng.choice((16, 32, 64)), skew=False)
        L, QB, G = _sizes(case)
        slices = case["B"] * case["H"]
        if not 500 <= L <= 118800:
            continue
        if op in ("mask", "layer"):
            if slices * QB * G > 1.2e9 or L < 4 * case["M"]:
                continue
        if op == "grouped" and (QB > 4096 or slices * QB > 60000):
            continue
        # (smaller tiles use less of a matrix instruction: a drawn case takes at most about a third of the largest one's time)
        if work(case)["flops"] <= {16: 1.5e12, 32: 3e12, 64: 9e12, 128: 9e12}[case["M"]]:
            return case


def _sizes(c):
    L = c["T"] * c["Hg"] * c["Wg"]
    return L, (L + c["M"] - 1) // c["M"], (L + c["N"] - 1) // c["N"]


def _tensor(c, data):
    """The values of `data` ([B, H, L, d]) in the case's storage order, seen as [B, H, L, d]."""
    if c["layout"] == "blhd":
        return data.transpose(1, 2).contiguous().transpose(1, 2)
    return data


def _normal(c, gen):
    shape = (c["B"], c["H"], _sizes(c)[0], c["d"])
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)


def _local_qk(c, gen):
    """N(0,1) draws plus random Fourier features of the grid position, one set of frequencies per head, so that scores grow
    towards tokens that are near in space and time, as those of a video model do."""
    L = _sizes(c)[0]
    idx = torch.arange(L, device="cuda")
    pos = torch.stack((idx // (c["Hg"] * c["Wg"]), (idx // c["Wg"]) % c["Hg"], idx % c["Wg"]), 1).float()
    q, k = _normal(c, gen), _normal(c, gen)
    for h in range(c["H"]):
        freq = 0.35 * torch.randn((3, c["d"] // 2), generator=gen, device="cuda")
        ang = (pos[:, :, None] * freq[None]).sum(1)
        feat = 2.5 * torch.cat((ang.cos(), ang.sin()), 1)
        q[:, h] += feat
        k[:, h] += feat
    return _tensor(c, q.bfloat16()), _tensor(c, k.bfloat16())


def _mask(c, gen):
    """CSR mask on the GPU: int64 indptr, int32 ids ascending within a work item."""
    L, QB, G = _sizes(c)
    dev = "cuda"
    block = torch.arange(QB, device=dev)
    centre = block * c["M"] + torch.clamp(L - block * c["M"], max=c["M"]) // 2
    key = torch.arange(L, device=dev)

    def coords(x):
        return x // (c["Hg"] * c["Wg"]), (x // c["Wg"]) % c["Hg"], x % c["Wg"]
    near = torch.ones((QB, L), dtype=torch.bool, device=dev)
    for a, b, reach in zip(coords(centre), coords(key), (c["dt"], c["dh"], c["dw"])):
        near &= (a[:, None] - b[None, :]).abs() <= reach
    if c["N"] > 1:
        near = torch.nn.functional.pad(near, (0, G * c["N"] - L)).view(QB, G, c["N"]).any(2)
    share = near.float().mean(1)
    counts, ids = [], []
    for _ in range(c["B"] * c["H"]):
        want = torch.full((QB,), c["density"], device=dev)
        if c["skew"]:
            sigma = 0.6
            head = math.log(c["density"]) - sigma * sigma / 2 + sigma * torch.randn((), generator=gen, device=dev)
            want = head.exp().clamp(0.05, 0.95) * (0.5 + torch.rand((QB,), generator=gen, device=dev))
            want = want.clamp(max=0.98)
        fill = ((want - share) / (1.0 - share).clamp(min=1e-6)).clamp(0.0, 1.0)
        on = near | (torch.rand((QB, G), generator=gen, device=dev) < fill[:, None])
        on[:, 0] |= ~on.any(1)
        counts.append(on.sum(1))
        ids.append(on.nonzero()[:, 1].int())
    indptr = torch.zeros(c["B"] * c["H"] * QB + 1, dtype=torch.int64, device=dev)
    indptr[1:] = torch.cat(counts).cumsum(0)
    return indptr, torch.cat(ids)


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    L, QB, G = _sizes(c)
    s = {"op": c["op"], "M": c["M"], "top_p": c["top_p"], "items": c["B"] * c["H"] * QB}
    if c["op"] in ("mask", "layer"):
        s["q"], s["k"] = _local_qk(c, gen)
    else:
        s["q"], s["k"] = _tensor(c, _normal(c, gen).bfloat16()), _tensor(c, _normal(c, gen).bfloat16())
    if c["op"] == "mask":
        s["p"] = F.make_params(s["q"], s["k"], s["k"], s["q"], c["M"], c["N"], c["d"] ** -0.5)
    else:
        s["v"] = _tensor(c, _normal(c, gen).bfloat16())
        s["out"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((c["B"], c["H"], L), dtype=torch.float32, device="cuda")
        s["p"] = F.make_params(s["q"], s["k"], s["v"], s["out"], c["M"], c["N"], c["d"] ** -0.5)
        s["ws"] = _bytes(F.fgattn_workspace_bytes(s["p"]))
    if c["op"] in ("forward", "grouped"):
        s["indptr"], s["indices"] = _mask(c, gen)
    if c["op"] in ("mask", "layer"):
        s["indptr"] = torch.empty(s["items"] + 1, dtype=torch.int64, device="cuda")
        s["mask_ws"] = _bytes(F.fgattn_mask_workspace_bytes(s["p"]))
        s["indices"] = torch.zeros(s["items"] * G, dtype=torch.int32, device="cuda")
    if c["op"] == "grouped":
        R = 128 // c["M"]
        groups = c["B"] * c["H"] * ((QB + R - 1) // R)
        s["tiles"] = torch.empty(groups * R, dtype=torch.int32, device="cuda")
        s["uptr"] = torch.empty(groups + 1, dtype=torch.int64, device="cuda")
        s["group_ws"] = _bytes(F.fgattn_group_workspace_bytes(s["p"], F.GROUP_XOR))
        s["uids"] = torch.zeros(groups * G, dtype=torch.int32, device="cuda")
        s["members"] = torch.zeros(groups * G, dtype=torch.uint8, device="cuda")
    return s


def run(state):
    s = state
    if s["op"] in ("mask", "layer"):
        F.fgattn_mask_select(s["q"], s["k"], s["p"], s["top_p"], s["indptr"], s["mask_ws"])
        F.fgattn_mask_emit(s["p"], s["indptr"], s["indices"], s["mask_ws"])
        if s["op"] == "mask":
            return s["indptr"], s["indices"]
    if s["op"] == "dense":
        F.fgattn_dense_forward(s["q"], s["k"], s["v"], s["p"], s["out"], s["lse"], s["ws"])
        return s["out"], s["lse"]
    if s["op"] in ("forward", "layer"):
        F.fgattn_forward(s["q"], s["k"], s["v"], s["indptr"], s["indices"], s["p"], s["out"], s["lse"], s["ws"])
        return (s["out"], s["lse"]) if s["op"] == "forward" else (s["out"], s["lse"], s["indptr"], s["indices"])
    F.fgattn_group_select(s["indptr"], s["indices"], s["p"], F.GROUP_XOR, s["tiles"], s["uptr"], s["group_ws"])
    F.fgattn_group_emit(s["p"], F.GROUP_XOR, s["tiles"], s["uptr"], s["uids"], s["members"], s["group_ws"])
    F.fgattn_forward_grouped(s["q"], s["k"], s["v"], s["tiles"], s["uptr"], s["uids"], s["members"], s["p"], s["out"], s["lse"],
                             s["ws"])
    return s["out"], s["lse"], s["tiles"], s["uptr"], s["uids"], s["members"]


def work(case):
    """Q, K, V (or Q, K), the mask read or written and the results, each once; 4 d operations per query row and active key,
    2 d per pair of block means.  A mask's entries are counted at the stated density."""
    c = case
    L, QB, G = _sizes(c)
    slices = c["B"] * c["H"]
    tensor = 2.0 * slices * L * c["d"]
    csr = slices * (8.0 * QB + 4.0 * QB * G * c["density"])
    means = 2.0 * c["d"] * slices * QB * G
    attention = 4.0 * c["d"] * slices * float(L) * L * c["density"]
    results = tensor + 4.0 * slices * L
    if c["op"] == "mask":
        return {"bytes": 2 * tensor + csr, "flops": means}
    if c["op"] == "dense":
        return {"bytes": 3 * tensor + results, "flops": attention}
    if c["op"] == "layer":
        return {"bytes": 3 * tensor + 2 * csr + results, "flops": means + attention}
    return {"bytes": 3 * tensor + csr + results, "flops": attention}


def tolerance(case):
    """Masks and groupings are whole numbers and exact.  Attention: P and the result are rounded to bf16 (8 bits) around
    32-bit sums; the largest deviation is that of one result's last bit plus the summed roundings of P."""
    if case["op"] == "mask":
        return "exact"
    return {"rel": 8e-3, "max": 5e-2, "differ": 0.0}
