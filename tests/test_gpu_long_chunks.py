"""The forward kernel for long chunks (64 queries by 32 keys a wave, key halves merged in
LDS) against the oracle, at the edges of its tiles and segments.  RV_ATTN_* overrides make
chunks long enough with little work; each case checks that its plan is one the kernel takes."""
import numpy as np
import pytest

import oracle
from paper_2609_23286_amd import synth
from util import LSE_ATOL, OUT_ATOL, SAL_RTOL, bf16_to_f64, out_error_bound, to_dev, to_host_u16

pytestmark = pytest.mark.gpu

CASES = [  # (N, H, M, split, minimum chunk, per cent of a first chunk, keys)
    # one chunk a unit (a stream-K plan whose chunks are longer than the units); query counts around the 32- and 64-query blocks, memory tails in the
    # first key half, at its end, in the second, and none
    (1, 1, 5633, "0", "100", "100", "flat"), (31, 2, 5652, "0", "100", "100", "flat"),
    (32, 1, 5664, "0", "100", "100", "flat"), (33, 2, 5665, "0", "100", "100", "flat"),
    (64, 3, 5695, "0", "100", "100", "flat"), (65, 2, 5696, "0", "100", "100", "flat"),
    (97, 1, 5700, "0", "100", "100", "flat"), (128, 2, 5632, "0", "100", "100", "flat"),
    (300, 2, 5555, "0", "100", "100", "flat"),
    # a frame without memory (chunks that straddle its units), and two and three chunks a unit
    (5700, 1, 0, "0", "100", "100", "flat"), (180, 2, 11300, "0", "91", "100", "flat"),
    (110, 1, 17000, "0", "95", "100", "flat"),
    # stream-K chunks of 98 tiles over units of 99: segments of 1 to 8 tiles at the units' ends,
    # the shortest of them the frame's last tile alone, with one key
    (129, 32, 6100, "0", "98", "100", "flat"),
    # logits that grow along the keys (the reference is raised again and again), that fall, and
    # a few units' worth of spread
    (130, 2, 5700, "0", "100", "100", "rising"), (130, 2, 5700, "0", "100", "100", "falling"),
    (70, 2, 5700, "0", "100", "100", "spread"),
    # logits of -2^97 everywhere (exact in fp32, as is their product with log2(e): every weight is
    # the same), with a tail of one valid key, whose tile the second key half has none of
    (66, 2, 5633, "0", "100", "100", "deep"),
]


@pytest.mark.parametrize("N,H,M,split,min_chunk,first_pct,keys", CASES)
def test_long_chunks_match_oracle(N, H, M, split, min_chunk, first_pct, keys, monkeypatch):
    import torch

    from paper_2609_23286_amd import rv

    print(f"long chunks N={N} H={H} M={M} split={split} keys={keys}", flush=True)
    rv.init()
    monkeypatch.setenv("RV_ATTN_SPLIT", split)
    monkeypatch.setenv("RV_ATTN_MIN_CHUNK", min_chunk)
    monkeypatch.setenv("RV_ATTN_FIRST_PCT", first_pct)
    assert rv.attention_plan_long(rv.attention_plan(N, N, M, H, 256, 8))
    rv.reserve_workspace(N, H, M)
    sigma = 0.125 if keys == "flat" else 1.0
    Q, K, V = (synth.normal_bf16(31 + N, 0, 0, tag, (N, H, 64), sigma) for tag in range(3))
    memK, memV = (synth.normal_bf16(32 + N, 1, 0, tag, (H, M, 64), sigma) for tag in (synth.TAG_MEMK, synth.TAG_MEMV))
    if keys in ("rising", "falling"):   # logits of standard deviation 0.05 .. 12
        ramp = np.linspace(0.05, 12.0, M)[:: 1 if keys == "rising" else -1]
        memK = synth.f32_to_bf16_bits((bf16_to_f64(memK) * ramp[None, :, None]).astype(np.float32))
    if keys == "deep":
        Q, K, memK = (np.zeros_like(x) for x in (Q, K, memK))
        Q[..., 0] = 0x5880                                  # 2^50
        K[..., 0] = memK[..., 0] = 0xD880                   # -2^50
    mem = rv.Memory(H, reserve_tokens=M + 5)
    if M:
        mem.write(torch.from_numpy(memK.view(np.int16)), torch.from_numpy(memV.view(np.int16)))
    out = torch.empty((N, H, 64), dtype=torch.int16, device="cuda")
    lse = torch.empty((H, N), dtype=torch.float32, device="cuda")
    rv.attend_frame(to_dev(Q), to_dev(K), to_dev(V), mem, out, lse)
    rv.device_status()
    mem.close()
    got, got_lse = bf16_to_f64(to_host_u16(out)), lse.cpu().numpy().astype(np.float64)
    want, want_lse = oracle.attend(Q, K, V, memK, memV, M)
    vmax = max(np.abs(bf16_to_f64(V)).max(), np.abs(bf16_to_f64(memV)).max() if M else 0.0)
    # The logits are fp32 sums of 64 products: an error of up to about 64 2^-24 of the largest
    # one, relative, moves the LSE by as much and every weight by that factor.
    z_err = 64 * 2.0 ** -24 * np.abs(want_lse).max()
    assert np.isfinite(got).all() and np.isfinite(got_lse).all()
    if keys == "deep":
        # No error in the logits, and the LSE is an fp32 value of that size.  (The output is the
        # mean of the value rows: at this size exp(z - LSE) loses the log of the keys' number
        # even in fp64.)
        rows = np.concatenate((bf16_to_f64(memV), bf16_to_f64(V).transpose(1, 0, 2)), axis=1)
        want = np.broadcast_to(rows.mean(axis=1)[None], want.shape)
        assert np.abs(got - want).max() <= out_error_bound(want, vmax)
        assert np.abs(got_lse - want_lse).max() <= 2.0 ** -22 * np.abs(want_lse).max()
        return
    assert np.abs(got - want).max() <= out_error_bound(want, vmax) + 2 * z_err * vmax
    if keys == "flat":
        assert np.abs(got - want).max() <= OUT_ATOL
    assert np.abs(got_lse - want_lse).max() <= LSE_ATOL + z_err


ENTRY_CASES = [  # (N, H, M): the staged frame's last tile ends in the first key half, at a tile
                 # boundary, in the second half; M a multiple of 64 (the frame path's tiles)
    (180, 2, 11300), (176, 2, 11344), (150, 3, 11350), (200, 2, 11328),
]


@pytest.mark.parametrize("N,H,M", ENTRY_CASES)
def test_every_attention_entry_point_takes_long_chunks(N, H, M, monkeypatch):
    """Two chunks of 88 tiles or more a unit through rv_attend_frame, _noalloc, _fused and
    rv_attend_staged: the outputs within the oracle's bounds; the frame path's outputs bit for
    bit from the three calls that take the same plan, from a second call, and from the staged
    frame where it has the same tiles; the fused saliency rows against the oracle's."""
    import ctypes

    import torch

    from paper_2609_23286_amd import rv

    print(f"long chunks, entry points N={N} H={H} M={M}", flush=True)
    rv.init()
    monkeypatch.setenv("RV_ATTN_SPLIT", "0")
    monkeypatch.setenv("RV_ATTN_MIN_CHUNK", "91")
    monkeypatch.setenv("RV_ATTN_FIRST_PCT", "100")
    for n_fkeys, mem_len in ((N, M), (0, M + N)):
        p = rv.attention_plan(N, n_fkeys, mem_len, H, 256, 8)
        assert rv.attention_plan_long(p) and p.total_chunks == 2 * p.n_units
    Q, K, V = (synth.normal_bf16(41 + N, 0, 0, tag, (N, H, 64), 0.125) for tag in range(3))
    memK, memV = (synth.normal_bf16(42 + N, 1, 0, tag, (H, M, 64), 0.125) for tag in (synth.TAG_MEMK, synth.TAG_MEMV))
    mem = rv.Memory(H, reserve_tokens=M + N)
    mem.write(torch.from_numpy(memK.view(np.int16)), torch.from_numpy(memV.view(np.int16)))
    Qd, Kd, Vd = to_dev(Q), to_dev(K), to_dev(V)
    qs = (1, N, 0, 3)
    got = {}
    for name in ("frame", "again", "noalloc", "fused", "staged"):
        out = torch.full((N, H, 64), 3, dtype=torch.int16, device="cuda")
        lse = torch.full((H, N), -9.0, dtype=torch.float32, device="cuda")
        if name in ("frame", "again"):
            rv.attend_frame(Qd, Kd, Vd, mem, out, lse)
        elif name == "noalloc":
            vp = ctypes.c_void_p
            mk, mv, hs = mem.view()
            st = rv.lib().rv_attend_frame_noalloc(
                vp(Qd.data_ptr()), vp(Kd.data_ptr()), vp(Vd.data_ptr()), N, vp(mk), vp(mv), M, hs, H, 64, None,
                vp(out.data_ptr()), vp(lse.data_ptr()), None, vp(torch.cuda.current_stream().cuda_stream))
            assert st == rv.RV_OK, rv.lib().rv_last_error()
        elif name == "fused":
            tiles = torch.full((H, -(-N // 128), N), -1.0, dtype=torch.float32, device="cuda")
            rv.attend_frame_fused(Qd, Kd, Vd, mem, out, lse, tiles, qs)
        else:
            mem.stage_frame(Kd, Vd)
            rv.attend_staged(Qd, mem, out, lse)
        rv.device_status()
        got[name] = (out, lse)
    mem.close()
    want, want_lse = oracle.attend(Q, K, V, memK, memV, M)
    vmax = max(np.abs(bf16_to_f64(V)).max(), np.abs(bf16_to_f64(memV)).max())
    for name, (out, lse) in got.items():
        assert np.abs(bf16_to_f64(to_host_u16(out)) - want).max() <= min(OUT_ATOL, out_error_bound(want, vmax)), name
        assert np.abs(lse.cpu().numpy() - want_lse).max() <= LSE_ATOL, name
        if name != "staged" or M % 64 == 0:
            assert torch.equal(out, got["frame"][0]) and torch.equal(lse, got["frame"][1]), name
    rows, sampled = tiles.cpu().numpy().astype(np.float64), oracle.qsub_index(*qs)
    for b in range(rows.shape[1]):
        sel = sampled[(sampled >= 128 * b) & (sampled < 128 * (b + 1))]
        ref = oracle.column_mass(Q, sel, want_lse[:, sel], K, "frame")
        assert (np.abs(rows[:, b] - ref) <= SAL_RTOL * ref).all(), f"block {b}"
