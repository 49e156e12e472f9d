"""The calls whose time this repository is judged by, with their inputs and references.

A case is one piece of the per-frame path as a program that streams frames calls it through
`paper_2609_23286_amd.rv`: the attention of a layer, a whole layer step, a frame of the
layer stack, the admission of a frame, and the staged and fused forms of a frame.  Sizes are
those of the repository's stream configurations (synth.CONFIGS) and benchmark options, at
memory lengths from the first frame of a stream to the long-memory stress.

Keys of a case:
  mode      attend  rv.attend_frame of one layer
            step    rv.attend_frame with the saliency, then rv.admit: one layer, frame by frame
            frame   rv.attend_frame of every layer, then rv.admit_layers
            admit   rv.admit_layers (shared: one selection per layer) from a given LSE
            staged  rv.stage_frames, rv.attend_staged of every layer, rv.admit_staged_layers
            fused   rv.attend_frame_fused of every layer, then rv.admit_layers_tiled
  layers, heads, grid_h, grid_w, special, stride, budget   the frame (N = grid_h grid_w + special
            tokens, 64 per head), the query windows and the rows admitted per head
  mem       memory rows per head before the frame
  sigma     standard deviation of the Q, K, V elements (logits: 8 sigma^2)
  tail      log-normal sigma of the key norms (heavy-tailed keys), 0 for none
As in the streams, `budget` keys of every head are planted along the mean query.
"""
import math

import torch

from paper_2609_23286_amd import rv

D = 64
MODES = ("attend", "step", "frame", "admit", "staged", "fused")


def _case(name, mode, layers=1, heads=16, grid=(28, 37), special=5, stride=2, budget=10, mem=0, sigma=0.125,
          tail=0.0, shared=False):
    c = {"mode": mode, "layers": layers, "heads": heads, "grid_h": grid[0], "grid_w": grid[1], "special": special,
         "stride": stride, "budget": budget, "mem": mem, "sigma": sigma, "tail": tail, "shared": shared}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest stream (2 heads, 64 tokens, one admitted row): launches and host calls.
        _case("tiny_step", "step", heads=2, grid=(8, 8), special=0, budget=1, mem=7, sigma=0.125),
        # The first frame of a ViT-L stream: one layer, nothing remembered yet.
        _case("layer_first_frame", "step", mem=0),
        # One layer of the 1000-frame stream early on, in its middle and at its end, and with
        # logits of the size that normalised queries and keys give (sigma 1).
        _case("layer_m2000", "attend", mem=2000),
        _case("layer_m5000", "attend", mem=5000, sigma=1.0),
        _case("layer_m9990", "attend", mem=9990),
        # The long-memory stress: one layer over 52,000 remembered rows.
        _case("layer_m52000", "attend", mem=52000),
        # One layer of the square-resolution stream near its end, heavy-tailed keys, an odd length.
        _case("square_m19987", "attend", grid=(37, 37), budget=13, mem=19987, tail=0.5),
        # A whole frame of the 24-layer stack at the stream's mean context: the headline workload.
        _case("stack_frame_m5000", "frame", layers=24, mem=5000),
        # The admission alone for all 24 layers: 2x2 windows and 1 % retention (the default) ...
        _case("admit_stack", "admit", layers=24, mem=5000),
        # ... and every patch sampled with 5 % retention (the benchmark's --stride 1 --gamma 0.05).
        _case("admit_dense", "admit", layers=24, stride=1, budget=52, mem=1000),
        # The paper's policy of 7 regulated layers, frames staged in the arenas.
        _case("staged_7_layers", "staged", layers=7, mem=3210),
        # The saliency formed in the attention's epilogue, the same 7 layers.
        _case("fused_7_layers", "fused", layers=7, mem=3210),
    ]


MAX_DRAWN_FLOPS = 6.0e11  # the stack frame: 6.2e11


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    mode = rng.choice(MODES)
    heads = rng.choice((2, 4, 8, 12, 16, 16, 16))
    gh = _log_int(rng, 8, 37)
    gw = max(8, min(40, int(round(gh * rng.uniform(0.75, 1.4)))))
    special = rng.choice((0, 1, 4, 5))
    n = gh * gw + special
    layers = 1 if mode in ("attend", "step") else _log_int(rng, 1, 24)
    mem = 0 if rng.random() < 0.1 else _log_int(rng, 16, 52000)
    budget = max(1, int(n * rng.choice((0.01, 0.01, 0.02, 0.05))))
    c = _case(None, mode, layers, heads, (gh, gw), special, rng.choice((1, 2, 2, 3, 4)), budget, mem,
              rng.choice((0.125, 0.125, 0.5, 1.0)), rng.choice((0.0, 0.0, 0.5)),
              mode == "admit" and rng.random() < 0.3)
    while work(c)["flops"] > MAX_DRAWN_FLOPS or c["layers"] * c["mem"] * heads > 24 * 10000 * 16:
        if c["layers"] > 1:
            c["layers"] -= 1
        else:
            c["mem"] = c["mem"] * 3 // 4
    return c


def _n_tokens(c):
    return c["grid_h"] * c["grid_w"] + c["special"]


def _sampled(c):
    """Token indices of the sampled queries: the top-left patch of every stride x stride window."""
    r = torch.arange(0, c["grid_h"], c["stride"])
    k = torch.arange(0, c["grid_w"], c["stride"])
    return (c["special"] + r[:, None] * c["grid_w"] + k[None, :]).reshape(-1)


def work(c):
    N, H, L, M, k = _n_tokens(c), c["heads"], c["layers"], c["mem"], c["budget"]
    nq = -(-c["grid_h"] // c["stride"]) * -(-c["grid_w"] // c["stride"])
    row = H * D * 2  # bytes of one token's rows
    flops = nbytes = 0
    if c["mode"] != "admit":  # Q, K, V, out, the memory and the LSE
        flops += 4 * D * H * N * (M + N)
        nbytes += 4 * N * row + 2 * M * row + 4 * H * N
    if c["mode"] != "attend":  # the saliency, and the admitted rows written
        flops += 2 * D * H * nq * N
        nbytes += 4 * H * N + 2 * k * row + 4 * H * k + 8 * H * k
        if c["mode"] == "admit":  # sampled queries and their LSE, the frame's keys, the admitted value and key rows
            nbytes += nq * row + 4 * H * nq + N * row + k * row
    return {"bytes": float(L * nbytes), "flops": float(L * flops)}


def _inputs(c, seed):
    """Q, K, V [L, N, H, 64] and memory K, V [L, H, M, 64], bf16."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    N, H, L, M, k = _n_tokens(c), c["heads"], c["layers"], c["mem"], c["budget"]

    def normal(*shape):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(generator=g).mul_(c["sigma"])

    Q = normal(L, N, H, D).bfloat16()
    K, V = normal(L, N, H, D), normal(L, N, H, D).bfloat16()
    mK, mV = normal(L, H, M, D), normal(L, H, M, D).bfloat16()
    if c["tail"] > 0:
        for x in (K, mK):
            x *= torch.empty(x.shape[:-1] + (1,), device="cuda").normal_(generator=g).mul_(c["tail"]).exp_()
    # planted keys: three times their norm, along the head's mean query
    u = torch.nn.functional.normalize(Q.float().sum(dim=1, keepdim=True), dim=-1)
    score = torch.empty((L, N, H, 1), device="cuda").uniform_(generator=g)
    planted = score <= score.kthvalue(k, dim=1, keepdim=True).values
    K = torch.where(planted, 3.0 * K.norm(dim=-1, keepdim=True) * u, K)
    return Q, K.bfloat16(), V, mK.bfloat16(), mV


class _Arena:
    """A memory's K or V arena [H][stride][64] as an array; it keeps the memory, which owns the rows, alive."""

    def __init__(self, mem, ptr, heads, stride):
        self.mem = mem
        self.__cuda_array_interface__ = {"shape": (heads, stride, D), "typestr": "<i2", "data": (ptr, False),
                                         "version": 3}


def _arena_rows(mem, heads, first, n):
    k, v, stride = mem.view()
    return [torch.as_tensor(_Arena(mem, p, heads, stride), device="cuda")[:, first:first + n].view(torch.bfloat16)
            for p in (k, v)]


def _logits(q, k):
    return (q @ k.t()) / math.sqrt(D)


def prepare(c, seed):
    rv.init()
    Q, K, V, mK, mV = _inputs(c, seed)
    N, H, L, M, k = _n_tokens(c), c["heads"], c["layers"], c["mem"], c["budget"]
    s = {"mode": c["mode"], "budget": k, "mem_len": M, "shared": c["shared"],
         "qs": rv.qsub(c["grid_h"], c["grid_w"], c["special"], c["stride"]),
         "Q": [Q[l] for l in range(L)], "K": [K[l] for l in range(L)], "V": [V[l] for l in range(L)]}
    s["mems"] = []
    for l in range(L):
        # room for the frame's rows, as a stream that knows its length reserves it
        m = rv.Memory(H, reserve_tokens=M + N)
        if M:
            m.write(mK[l].contiguous(), mV[l].contiguous())
        s["mems"].append(m)
    f32 = {"dtype": torch.float32, "device": "cuda"}
    lse = torch.empty((L, H, N), **f32)
    s["lse"] = [lse[l] for l in range(L)]
    s["outputs"] = {}
    if c["mode"] == "admit":
        for l in range(L):  # the LSE that the attention of this frame left, as float32
            for h in range(H):
                q = Q[l, :, h].float()
                z = torch.logsumexp(_logits(q, K[l, :, h].float()), dim=1)
                if M:
                    z = torch.logaddexp(z, torch.logsumexp(_logits(q, mK[l, h].float()), dim=1))
                lse[l, h] = z
    else:
        out = torch.empty((L, N, H, D), dtype=torch.bfloat16, device="cuda")
        s["out"] = [out[l] for l in range(L)]
        s["outputs"].update(out=out, lse=lse)
    if c["mode"] != "attend":
        sal, idx = torch.empty((L, H, N), **f32), torch.empty((L, H, k), dtype=torch.int32, device="cuda")
        s["sal"], s["idx"] = [sal[l] for l in range(L)], [idx[l] for l in range(L)]
        s["outputs"].update(sal=sal, idx=idx)
        if c["mode"] == "fused":
            s["tiles"] = list(torch.empty((L, H, -(-N // rv.QUERY_BLOCK), N), **f32))
        rows = [_arena_rows(m, H, M, k) for m in s["mems"]]  # where this frame's rows are appended
        s["outputs"].update({f"mem{l}": rows[l] for l in range(min(L, 8))})
    torch.cuda.synchronize()
    return s


def run(s):
    mode, mems, qs, k = s["mode"], s["mems"], s["qs"], s["budget"]
    Q, K, V, lse = s["Q"], s["K"], s["V"], s["lse"]
    L = len(mems)
    if mode != "attend":
        for m in mems:  # a repeated pass admits the same frame again
            m.truncate(s["mem_len"])
    if mode == "attend":
        rv.attend_frame(Q[0], K[0], V[0], mems[0], s["out"][0], lse[0])
    elif mode == "step":
        rv.attend_frame(Q[0], K[0], V[0], mems[0], s["out"][0], lse[0], s["sal"][0], qs)
        rv.admit(s["sal"][0], k, K[0], V[0], mems[0], 1, s["idx"][0])
    elif mode == "frame":
        for l in range(L):
            rv.attend_frame(Q[l], K[l], V[l], mems[l], s["out"][l], lse[l])
        rv.admit_layers(Q, K, V, lse, qs, k, mems, 1, s["sal"], s["idx"])
    elif mode == "admit":
        rv.admit_layers(Q, K, V, lse, qs, k, mems, 1, s["sal"], s["idx"], shared=s["shared"])
    elif mode == "staged":
        rv.stage_frames(mems, K, V)
        for l in range(L):
            rv.attend_staged(Q[l], mems[l], s["out"][l], lse[l])
        rv.admit_staged_layers(Q, lse, qs, k, mems, 1, s["sal"], s["idx"])
    else:
        for l in range(L):
            rv.attend_frame_fused(Q[l], K[l], V[l], mems[l], s["out"][l], lse[l], s["tiles"][l], qs)
        rv.admit_layers_tiled(s["tiles"], k, K, V, mems, 1, s["sal"], s["idx"])
    return s["outputs"]


def tolerance(c):
    # bf16 outputs, probabilities and partial outputs; LSE and saliency are fp32
    return {"rel": 1e-2, "max": 0.1, "differ": 0.005}


def exact(c, seed):
    Q, K, V, mK, mV = _inputs(c, seed)
    N, H, L, M = _n_tokens(c), c["heads"], c["layers"], c["mem"]
    if L * H * N * (M + N) > 4e9:
        return None
    f64 = {"dtype": torch.float64, "device": "cuda"}
    lse, sal = torch.empty((L, H, N), **f64), torch.empty((L, H, N), **f64)
    out = torch.empty((L, N, H, D), **f64) if c["mode"] != "admit" else None
    sampled = _sampled(c).cuda()
    for l in range(L):
        for h in range(H):
            q, k = Q[l, :, h].double(), K[l, :, h].double()
            z = _logits(q, torch.cat((mK[l, h].double(), k)))
            lse[l, h] = torch.logsumexp(z, dim=1)
            if out is not None:
                out[l, :, h] = z.sub_(lse[l, h][:, None]).exp_() @ torch.cat((mV[l, h], V[l, :, h])).double()
            if c["mode"] == "admit":  # the path is given the LSE in 32 bits
                lse[l, h] = lse[l, h].float().double()
            if c["mode"] != "attend":
                sal[l, h] = (_logits(q[sampled], k) - lse[l, h][sampled][:, None]).exp_().sum(dim=0)
    got = {} if c["mode"] == "admit" else {"out": out, "lse": lse}
    if c["mode"] != "attend":
        got.update(sal=sal, idx=None, **{f"mem{l}": None for l in range(min(L, 8))})
    return got
