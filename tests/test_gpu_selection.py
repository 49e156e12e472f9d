"""The selection's two ways (ranked candidates, radix select) at the edges where they
change or could go wrong, against the oracle's stable sort."""
import numpy as np
import pytest

import oracle
from util import to_dev

pytestmark = pytest.mark.gpu

CASES = [  # (N, budget, values)
    # fewer tokens than threads, one wave's worth, exactly 256 and one to either side
    (2, 1, "spread"), (3, 2, "spread"), (63, 10, "spread"), (65, 32, "spread"), (255, 128, "spread"),
    (256, 128, "spread"), (257, 127, "spread"), (255, 50, "spread"), (256, 50, "spread"), (257, 50, "spread"),
    # budgets past the line of the largest ranked frame, one token past it, the smallest budget
    (2048, 128, "spread"), (2048, 129, "spread"), (2049, 128, "spread"), (2047, 1, "spread"),
    # all of the largest values on one thread, and on one wave
    (1041, 5, "one thread"), (1041, 40, "one wave"), (1041, 64, "descending"), (1041, 64, "ascending"),
    # ties: few levels, half the tokens equal at the bound, all equal, all zero (by radix), zeros
    # below a few values
    (1041, 10, "levels"), (1041, 52, "half equal"), (1041, 10, "equal"), (200, 128, "zero"), (1041, 52, "few"),
    # the largest budget that is ranked for a frame, and one more (40 + N / 24; half the tokens)
    (1041, 83, "spread"), (1041, 84, "spread"), (2048, 125, "spread"), (2048, 126, "spread"), (80, 40, "spread"),
    (80, 41, "spread"), (2, 1, "zero"),
    # equal values cut to those the budget needs: in every word of 64 tokens, in the last one only,
    # more values above the bound than the budget (threads hold several), and none needed
    (2048, 125, "half equal"), (2047, 1, "equal"), (2048, 70, "zero"), (2040, 20, "last equal"),
    (2048, 40, "clump equal"),
    # more candidates than fit, none of them equal
    (2048, 52, "clump"), (1041, 83, "clump"),
    # -0 is 0, ranked and by radix
    (1041, 10, "signed zeros"), (2050, 10, "signed zeros"), (2052, 10, "signed zeros"),
]


def saliency(N, values, rng):
    if values == "one thread":      # tokens t, t + 256, ... of one thread
        s = rng.random(N) + 1.0
        s[7::256] += 10.0
    elif values == "one wave":      # threads 64 .. 127
        s = rng.random(N) + 1.0 + 10.0 * ((np.arange(N) % 256) // 64 == 1)
    elif values == "descending":
        s = 2.0 - np.arange(N) / N
    elif values == "ascending":
        s = 1.0 + np.arange(N) / N
    elif values == "levels":
        s = rng.integers(1, 4, N).astype(np.float64)
    elif values == "half equal":
        s = np.where(rng.random(N) < 0.5, 1.0, rng.random(N))
        s[rng.choice(N, 20, replace=False)] = 2.0 + rng.random(20)
    elif values == "equal":
        s = np.full(N, 0.25)
    elif values == "zero":
        s = np.zeros(N)
    elif values == "last equal":    # 18 spread ones, and the last 150 tokens equal
        s = rng.random(N) * 0.5
        s[rng.choice(N - 150, 18, replace=False)] = 2.0 + rng.random(18)
        s[N - 150:] = 1.0
    elif values in ("clump", "clump equal"):    # all of the largest values on fewer threads than the budget
        s = rng.random(N) * 0.5 + (np.arange(N) % 256 < (51 if values == "clump" else 30))
        if values == "clump equal":             # ... and the bound a value that 200 others hold
            s[rng.choice(np.flatnonzero(np.arange(N) % 256 >= 40), 200, replace=False)] = 0.75
    elif values == "signed zeros":
        s = np.where(rng.random(N) < 0.5, 0.0, -0.0)
        s[rng.choice(N, 4, replace=False)] = 1.0
    elif values == "few":
        s = np.zeros(N)
        s[rng.choice(N, 40, replace=False)] = 1.0
    else:
        s = rng.random(N)
    return s.astype(np.float32)


@pytest.mark.parametrize("N,budget,values", CASES)
def test_selection_edges(N, budget, values):
    import torch

    from paper_2609_23286_amd import rv

    print(f"selection N={N} budget={budget} {values}", flush=True)
    H = 3
    rng = np.random.default_rng(N * 1000 + budget)
    sal = np.stack([saliency(N, values, rng) for _ in range(H)])
    K, V = (rng.integers(0, 1 << 15, (N, H, 64)).astype(np.uint16) for _ in range(2))
    mem = rv.Memory(H, reserve_tokens=budget)
    idx = torch.full((H, budget), -7, dtype=torch.int32, device="cuda")
    rv.admit(to_dev(sal), budget, to_dev(K), to_dev(V), mem, 42, idx)
    ref = oracle.topk(sal.astype(np.float64), budget)
    assert (idx.cpu().numpy() == ref).all()
    mk, mv, prov = mem.read()
    for h in range(H):
        assert (mk[h].numpy().view(np.uint16) == K[ref[h], h]).all()
        assert (mv[h].numpy().view(np.uint16) == V[ref[h], h]).all()
        assert (prov[h, :, 1].numpy() == ref[h]).all()
    mem.close()


@pytest.mark.parametrize("grid,special,stride,layers", [
    ((28, 37), 5, 2, 24),   # one block a wave alone, two in 24 layers
    ((28, 37), 5, 1, 8),    # several passes of staged query rows; 8 layers: past the line
    ((28, 37), 5, 2, 6),    # 6 layers: two a wave, in one round of workgroups
    ((28, 37), 5, 2, 7),    # 7 layers: one a wave, two rounds either way
    ((12, 11), 1, 3, 24),   # 5 blocks: ranges of 3 and 2
    ((8, 8), 0, 2, 24),     # 2 blocks for 4 waves
])
def test_saliency_bits_do_not_depend_on_the_launch(grid, special, stride, layers):
    """One layer alone and among others, whose launch splits the keys otherwise: the same
    saliency bits and selection, within 1e-3 of the oracle's saliency."""
    import torch

    from paper_2609_23286_amd import rv, synth

    rv.init()
    N, H, k = grid[0] * grid[1] + special, 16, 5
    qs = (*grid, special, stride)
    print(f"saliency N={N} stride={stride} layers={layers}", flush=True)
    Q, K, V = (synth.normal_bf16(77, 0, 0, tag, (N, H, 64), 0.125) for tag in range(3))
    dev = [to_dev(x) for x in (Q, K, V)]
    lse = torch.logsumexp(torch.einsum("ihd,jhd->hij", *(x.view(torch.bfloat16).float().cpu() for x in dev[:2])) / 8, 2)
    lse = lse.cuda().contiguous()
    got = []
    for L in (1, layers):
        mems = [rv.Memory(H, reserve_tokens=k) for _ in range(L)]
        sal = [torch.empty((H, N), device="cuda") for _ in range(L)]
        idx = [torch.empty((H, k), dtype=torch.int32, device="cuda") for _ in range(L)]
        rv.admit_layers(*([x] * L for x in dev), [lse] * L, qs, k, mems, 0, sal, idx)
        torch.cuda.synchronize()
        got += list(zip(sal, idx))
        for m in mems:
            m.close()
    for s, i in got[1:]:
        assert torch.equal(s, got[0][0]) and torch.equal(i, got[0][1])
    z = torch.einsum("ihd,jhd->hij", *(x.view(torch.bfloat16).double().cpu() for x in dev[:2])) / 8
    want = torch.exp(z - lse.cpu().double()[:, :, None])[:, oracle.qsub_index(*qs)].sum(1)
    assert ((got[0][0].cpu().double() - want).abs() <= 1e-3 * want).all()
