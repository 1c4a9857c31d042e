"""The attention kernel for grids that fill the chip, at the edges of its ranges: the smallest grids it takes, lists around the
64 entries one register holds, sweeps that start inside the list (later rounds of a launch), the deeper request ring, ragged
and empty lists, lists in no order, both head dimensions.  Sampled query blocks against the oracle, at the bf16 bound; what
calls of this size promise about their bits; the second branch folded into the store; raster order."""
import numpy as np
import pytest
import torch

import gpu_util as gu
from paper_2512_05754_amd import synth

pytestmark = pytest.mark.gpu

# (batch, heads, blocks, head_dim, kmax, ragged): what the case is there for
CASES = [
    (1, 7, 110, 128, 18, False),    # 770 blocks: one round, every list starts at its first entry
    (1, 8, 128, 128, 128, False),   # exactly one round, every block listed
    (1, 22, 70, 128, 11, False),    # just above one and a half rounds; later lists start inside
    (1, 4, 390, 128, 64, False),    # 64 entries: the whole list in one register
    (1, 4, 390, 128, 65, False),    # ... and one more
    (1, 2, 900, 128, 130, False),   # more than 128 entries, one head's K and V 29 MB (stays with the kernel for small grids)
    (1, 2, 1100, 128, 130, False),  # ... 36 MB: the deeper ring (in index order)
    (1, 2, 900, 128, 380, False),   # the deeper ring, six registers of entries, with and without a work order
    (1, 3, 800, 128, 3, True),      # deeper ring, lists of 0 to 3 entries
    (2, 12, 70, 128, 9, True),      # ragged, empty lists among them
    (1, 54, 101, 64, 16, False),    # d = 64, four rounds
    (1, 14, 400, 64, 66, True),     # d = 64, ragged, up to 66 entries
    (1, 7, 670, 64, 20, False),     # d = 64, a head of more than 640 blocks
]


@pytest.mark.parametrize("B,Hh,nb,d,kmax,ragged", CASES)
@pytest.mark.parametrize("ordered", [False, True])
def test_wide_grids_against_the_oracle(usv, B, Hh, nb, d, kmax, ragged, ordered):
    w = synth.Workload("wide", B, Hh, nb * 64 - 23, d, "bf16", 2.0, kmax, seed=7000 + nb + kmax)
    Q, K, V = synth.gen_qkv(w)
    q, k, v = gu.up(Q), gu.up(K), gu.up(V)
    rng = np.random.default_rng(nb * 1000 + kmax)
    cnt = rng.integers(0, kmax + 1, size=(B, Hh, nb)).astype(np.int32) if ragged else np.full((B, Hh, nb), kmax, np.int32)
    scores = rng.random((B, Hh, nb, nb), dtype=np.float32)
    idx = np.sort(np.argsort(scores, axis=-1)[..., :kmax], axis=-1).astype(np.int32)
    idx[0, 0] = rng.permuted(idx[0, 0], axis=-1)  # one head's lists in no order
    idx[np.arange(kmax) >= cnt[..., None]] = -1
    wo = usv.attn_work_order(gu.up(cnt), kmax, idx=gu.up(idx)) if ordered else None
    out, lse = usv.block_sparse_attn(q, k, v, gu.up(idx), gu.up(cnt), seq_valid=w.seq_valid, return_lse=True,
                                     out_dtype=torch.float32, work_order=wo)
    out16 = usv.block_sparse_attn(q, k, v, gu.up(idx), gu.up(cnt), seq_valid=w.seq_valid, work_order=wo)
    gu.assert_bf16_store_is_rne(out16, out, "wide")
    o_h, l_h = gu.down(out), gu.down(lse)
    assert np.isfinite(o_h).all()
    # blocks of the first, a middle and the last round of the first, a middle and the last XCD, and the partial block
    flat = [int(x) for x in np.linspace(0, B * Hh * nb - 1, 17)] + [B * Hh * nb - 2]
    for f in flat:
        b, h, i = f // (Hh * nb), f // nb % Hh, f % nb
        ref_o, ref_l = gu.oracle_attn_blocks(Q[b, h], K[b, h], V[b, h], idx[b, h], cnt[b, h], w.seq_valid, [i])[i]
        what = f"head {b},{h} block {i} ({cnt[b, h, i]} listed)"
        gu.assert_attn_close(o_h[b, h, i * 64:(i + 1) * 64], ref_o, "bf16", what)
        live = np.isfinite(ref_l)
        got = l_h[b, h, i * 64:(i + 1) * 64]
        assert np.array_equal(np.isneginf(got), ~live), what
        assert not live.any() or np.abs(got[live] - ref_l[live]).max() <= 2e-2, what


@pytest.mark.parametrize("B,Hh,nb,d,mode", [
    (1, 13, 120, 128, "cube"),      # 1560 query blocks
    (2, 23, 120, 64, "cube"),       # 5520
    (1, 18, 120, 128, "raster"),    # 2160
    (2, 23, 120, 64, "raster"),
    (1, 18, 120, 128, "cubes"),     # one cube per block, cut cubes padded
    (1, 45, 121, 64, "cubes"),
])
@pytest.mark.parametrize("gates", ["both", "fine", "coarse", "none"])
def test_second_branch_of_a_large_launch(usv, B, Hh, nb, d, mode, gates):
    """out = gate_fine * attention + gate_coarse * coarse[cube] in the store of the kernel for large grids: both gates, one, none (an
    absent gate is 1); fp32 and bf16 output; a partial last block, cut cubes; projection layout, with a work order and without."""
    kmax, raster = 7, mode != "cube"
    rng = np.random.default_rng(nb + d + len(mode))
    valid = rng.integers(1, 65, size=nb).astype(np.int32) if mode == "cubes" else np.full(nb, 64, np.int32)
    if mode != "cubes":
        valid[-1] = 64 - 27
    Nv = int(valid.sum())
    rows = Nv if raster else nb * 64
    gen = torch.Generator(device=gu.DEV).manual_seed(nb * d)

    def tensor(scale=1.0):
        x = torch.randn((B, rows, Hh, d) if raster else (B, Hh, rows, d), device=gu.DEV, generator=gen) * scale
        x = x.to(torch.bfloat16)
        return x.transpose(1, 2) if raster else x  # raster: as a projection leaves it

    q, k, v = tensor(1.5), tensor(1.5), tensor()
    gf = tensor() if gates in ("both", "fine") else None
    gc = tensor() if gates in ("both", "coarse") else None
    coarse = torch.randn((B, Hh, nb, d), device=gu.DEV, generator=gen)
    cnt = rng.integers(0, kmax + 1, size=(B, Hh, nb)).astype(np.int32)
    idx = np.sort(np.argsort(rng.random((B, Hh, nb, nb)), axis=-1)[..., :kmax], axis=-1).astype(np.int32)
    i_g, c_g = gu.up(idx), gu.up(cnt)
    # position -> raster row (padding positions: 0, a valid token, as the order kernels write it)
    order = np.zeros((nb, 64), np.int32)
    order[np.arange(64)[None, :] < valid[:, None]] = rng.permutation(Nv) if raster else np.arange(Nv)
    kw = dict(coarse=coarse, gate_fine=gf, gate_coarse=gc, return_lse=True)
    outs = {}
    if raster:
        o_g = gu.up(order.reshape(-1))
        for wo in (None, usv.attn_work_order(c_g, kmax, idx=i_g)):
            for odt in (torch.float32, torch.bfloat16):
                outs[wo is not None, odt] = usv.block_sparse_attn_raster(
                    q, k, v, o_g, i_g, c_g, out_dtype=odt, work_order=wo, block_valid=gu.up(valid) if mode == "cubes" else None, **kw)
    else:
        for odt in (torch.float32, torch.bfloat16):
            outs[False, odt] = usv.block_sparse_attn(q, k, v, i_g, c_g, seq_valid=Nv, out_dtype=odt, **kw)
    for f in [int(x) for x in np.linspace(0, B * Hh * nb - 1, 13)]:
        b, h, i = f // (Hh * nb), f // nb % Hh, f % nb
        pick = lambda t, p: gu.down(t[b, h][torch.from_numpy(p).to(gu.DEV).long()]).astype(np.float64)
        mine = order[i, :valid[i]]
        keys = np.concatenate([order[j, :valid[j]] for j in idx[b, h, i, :cnt[b, h, i]]]) if cnt[b, h, i] else np.zeros(0, int)
        attn, lse = np.zeros((valid[i], d)), np.full(valid[i], -np.inf)
        if len(keys):
            S = pick(q, mine) @ pick(k, keys).T / np.sqrt(d)
            m = S.max(axis=1, keepdims=True)
            P = np.exp(S - m)
            attn, lse = P @ pick(v, keys) / P.sum(axis=1, keepdims=True), m[:, 0] + np.log(P.sum(axis=1))
        g1 = pick(gf, mine) if gf is not None else np.ones((valid[i], d))
        g2 = pick(gc, mine) if gc is not None else np.ones((valid[i], d))
        want = g1 * attn + g2 * gu.down(coarse[b, h, i]).astype(np.float64)
        for (ordered, odt), (out, out_lse) in outs.items():
            if odt != torch.float32:
                continue
            what = f"{gates} head {b},{h} block {i} ({cnt[b, h, i]} listed) ordered {ordered}"
            err = np.abs(pick(out, mine) - want)  # (the gate scales the attention's error)
            assert (err <= gu.BF16_MAX_ABS * np.maximum(1.0, np.abs(g1))).all(), (what, err.max())
            got = pick(out_lse[..., None], mine)[:, 0]
            assert np.array_equal(np.isneginf(got), np.isneginf(lse)), what
            assert not len(keys) or np.abs(got - lse).max() <= 2e-2, what
    for ordered in {o for o, _ in outs}:
        gu.assert_bf16_store_is_rne(outs[ordered, torch.bfloat16][0], outs[ordered, torch.float32][0], f"{mode} {gates}")
    if not raster:  # padded rows are written as 0
        assert not gu.down(outs[False, torch.float32][0])[:, :, Nv:].any()


@pytest.mark.parametrize("B,Hh,nb,d,kmax,raster", [
    (1, 4, 390, 128, 60, False),   # later lists start inside
    (1, 8, 700, 128, 50, False),   # the deeper ring, several rounds (a head beyond the L2)
    (2, 14, 200, 64, 30, False),   # d = 64
    (1, 4, 600, 128, 60, True),    # raster order
    (1, 7, 800, 64, 40, True),     # ... d = 64
])
def test_what_a_large_launch_promises(usv, B, Hh, nb, d, kmax, raster):
    """The same call gives the same bits (nothing in the hand-counted waits of the request ring depends on timing), and calls
    whose lists start elsewhere (other work orders, another slot of the launch, another kmax) differ by the rounding of the
    weights to bf16: 2^-8 of a weight in either, so 2^-7 of the row sum between the two and 2^-7 of a mean of |v - out|, which is at
    most twice the largest |v|; and 2e-3 of the 2-norm, twice what such inputs show."""
    Nv = nb * 64 - (0 if raster else 37)
    gen = torch.Generator(device=gu.DEV).manual_seed(nb + kmax)
    def tensor():
        x = torch.randn((B, Hh, nb, 64, d), device=gu.DEV, generator=gen) + 2 * torch.randn((B, Hh, nb, 1, d), device=gu.DEV, generator=gen)
        return x.view(B, Hh, nb * 64, d).to(torch.bfloat16)
    q, k, v = tensor(), tensor(), tensor()
    idx = torch.rand((B, Hh, nb, nb), device=gu.DEV, generator=gen).topk(kmax, dim=-1).indices.sort(-1).values.int()
    cnt = torch.full((B, Hh, nb), kmax, dtype=torch.int32, device=gu.DEV)
    order = torch.randperm(nb * 64, device=gu.DEV, generator=gen).int()

    def run(wo=None, i=idx, c=cnt, qkv=(q, k, v)):
        if raster:
            return usv.block_sparse_attn_raster(*qkv, order, i, c, out_dtype=torch.float32, return_lse=True, work_order=wo)
        return usv.block_sparse_attn(*qkv, i, c, seq_valid=Nv, out_dtype=torch.float32, return_lse=True, work_order=wo)

    sorted_order = usv.attn_work_order(cnt, kmax, idx=idx)
    shuffled = torch.rand((B, Hh, nb), device=gu.DEV, generator=gen).argsort(-1).int()
    plain, plain_lse = run()
    for wo in (None, sorted_order, shuffled):
        first, first_lse = run(wo)
        for _ in range(4):
            again, again_lse = run(wo)
            assert torch.equal(again.view(torch.int32), first.view(torch.int32))
            assert torch.equal(again_lse.view(torch.int32), first_lse.view(torch.int32))

    def close(out, lse, what):
        diff = (out - plain).double()
        assert diff.abs().max() <= 2.0 ** -6 * v.abs().max(), what
        assert diff.norm() <= 2e-3 * plain.double().norm(), (what, float(diff.norm() / plain.double().norm()))
        live = torch.isfinite(plain_lse)
        assert torch.equal(live, torch.isfinite(lse)), what
        assert (lse - plain_lse)[live].abs().max() <= 2.0 ** -7 * 1.01, what

    close(*run(sorted_order), "sorted work order")
    close(*run(shuffled), "random work order")
    # the same heads in another slot of the launch
    rolled = [t.roll(1, dims=1) for t in (q, k, v)]
    out, lse = run(None, idx.roll(1, dims=1), cnt, rolled)
    close(out.roll(-1, dims=1), lse.roll(-1, dims=1), "another head slot")
    # the same lists in rows of another length (past the sixth of the blocks up to which lists start inside)
    long = torch.full((B, Hh, nb, nb // 5), -1, dtype=torch.int32, device=gu.DEV)
    long[..., :kmax] = idx
    close(*run(None, long, cnt), "another kmax")


@pytest.mark.parametrize("Hh,nb,d,kmax", [(13, 125, 128, 9), (4, 650, 128, 100), (10, 700, 128, 40), (45, 125, 64, 9)])
def test_raster_order_gives_the_bits_of_gathered_tensors(usv, Hh, nb, d, kmax):
    """On both sides of the rule between the kernels and with the deeper ring (which raster order has not got)."""
    gen = torch.Generator(device=gu.DEV).manual_seed(nb)
    q, k, v = (torch.randn((1, Hh, nb * 64, d), device=gu.DEV, generator=gen).to(torch.bfloat16) for _ in range(3))
    idx = torch.rand((1, Hh, nb, nb), device=gu.DEV, generator=gen).topk(kmax, dim=-1).indices.sort(-1).values.int()
    cnt = torch.full((1, Hh, nb), kmax, dtype=torch.int32, device=gu.DEV)
    order = torch.randperm(nb * 64, device=gu.DEV, generator=gen)
    out, lse = usv.block_sparse_attn_raster(q, k, v, order.int(), idx, cnt, out_dtype=torch.float32, return_lse=True)
    want, want_lse = usv.block_sparse_attn(*(t[:, :, order].contiguous() for t in (q, k, v)), idx, cnt, out_dtype=torch.float32,
                                           return_lse=True)
    assert torch.equal(out[:, :, order].view(torch.int32), want.view(torch.int32))
    assert torch.equal(lse[:, :, order].view(torch.int32), want_lse.view(torch.int32))


# Grids that fill the chip and stay with the kernel for small ones all the same: its sweeps start at the first entry, so the
# result does not depend on the order the query blocks are walked in, bit for bit.
@pytest.mark.parametrize("B,Hh,nb,d,kmax", [
    (1, 4, 650, 128, 100),    # a head beyond the L2, lists that drift apart
    (1, 3, 660, 128, 66),     # ... with a work order, lists past 64 entries
    (2, 12, 41, 128, 20),     # one full round, ragged, a short head with a work order
    (1, 2, 1200, 128, 300),   # 1/6 to 1/3 of the blocks of a larger head, with and without
    (1, 4, 1300, 64, 180),    # d = 64, with a work order
])
def test_calls_that_stay_with_the_small_grids_kernel(usv, B, Hh, nb, d, kmax):
    w = synth.Workload("stay", B, Hh, nb * 64 - 31, d, "bf16", 2.0, kmax, seed=nb + kmax)
    Q, K, V = synth.gen_qkv(w)
    q, k, v = gu.up(Q), gu.up(K), gu.up(V)
    rng = np.random.default_rng(nb)
    cnt = rng.integers(kmax // 4, kmax + 1, size=(B, Hh, nb)).astype(np.int32)
    idx = np.sort(np.argsort(rng.random((B, Hh, nb, nb), dtype=np.float32), axis=-1)[..., :kmax], axis=-1).astype(np.int32)
    i_g, c_g = gu.up(idx), gu.up(cnt)
    run = lambda wo: gu.down(usv.block_sparse_attn(q, k, v, i_g, c_g, seq_valid=w.seq_valid, out_dtype=torch.float32, work_order=wo))
    wo = usv.attn_work_order(c_g, kmax, idx=i_g)
    ordered, mixed = run(wo), run(gu.up(np.stack([[rng.permutation(nb) for _ in range(Hh)] for _ in range(B)]).astype(np.int32)))
    assert np.array_equal(ordered, mixed)
    plain = run(None)
    for f in np.linspace(0, B * Hh * nb - 1, 9).astype(int):
        b, h, i = f // (Hh * nb), f // nb % Hh, f % nb
        ref, _ = gu.oracle_attn_blocks(Q[b, h], K[b, h], V[b, h], idx[b, h], cnt[b, h], w.seq_valid, [i])[i]
        for o in (ordered, plain):
            gu.assert_attn_close(o[b, h, i * 64:(i + 1) * 64], ref, "bf16", f"head {b},{h} block {i} ({cnt[b, h, i]} listed)")


@pytest.mark.parametrize("d,Hh", [(128, 8), (128, 98), (64, 8), (64, 340)])  # 128 and 1568, 128 and 5440 query blocks
def test_hugely_negative_logits_are_still_a_softmax(usv, d, Hh):
    """Logits of -2^113 sqrt(d) (bf16 inputs reach them), all alike in a row: every listed key has the same weight, so a row is
    the mean of its keys' V, whatever the size of the logits; both kernels, the reference raised from nothing on the first tile.
    (Powers of two, so that the scaled logits are exact and their differences are 0 in any arithmetic.)"""
    nb, kmax, Nv = 16, 3, 16 * 64 - 5
    rng = np.random.default_rng(d + Hh)
    v = rng.standard_normal((1, Hh, nb * 64, d), dtype=np.float32)
    V = synth.f32_to_bf16_bits(v)
    v = synth.as_f32(V).astype(np.float64)
    q = torch.full((1, Hh, nb * 64, d), 2.0 ** 57, dtype=torch.bfloat16, device=gu.DEV)
    k = torch.full((1, Hh, nb * 64, d), -2.0 ** 56, dtype=torch.bfloat16, device=gu.DEV)
    idx = np.sort(np.argsort(rng.random((1, Hh, nb, nb)), axis=-1)[..., :kmax], axis=-1).astype(np.int32)
    cnt = np.full((1, Hh, nb), kmax, np.int32)
    out, lse = usv.block_sparse_attn(q, k, gu.up(V), gu.up(idx), gu.up(cnt), seq_valid=Nv, return_lse=True, out_dtype=torch.float32)
    o, l = gu.down(out), gu.down(lse)
    logit = float(q[0, 0, 0, 0]) * float(k[0, 0, 0, 0]) * np.sqrt(d)  # d terms / sqrt(d)
    for h in (0, Hh // 2, Hh - 1):
        for i in (0, 7, nb - 1):
            keys = np.concatenate([np.arange(j * 64, min(j * 64 + 64, Nv)) for j in idx[0, h, i]])
            rows = slice(i * 64, min(i * 64 + 64, Nv))
            want = np.broadcast_to(v[0, h, keys].mean(axis=0), o[0, h, rows].shape)
            # equal weights are exact in bf16: what is left is the fp32 sum of 192 values
            np.testing.assert_allclose(o[0, h, rows], want, rtol=0, atol=192 * 2.0 ** -24 * 4)
            np.testing.assert_allclose(l[0, h, rows], logit, rtol=1e-6)


# Both sides of the lines at which lists start inside, waves take turns and long heads change kernels.
@pytest.mark.parametrize("Hh,nb,d,kmax", [
    (16, 257, 128, 51),    # just past four rounds and 256 blocks: turns; a fifth of the blocks
    (16, 256, 128, 51),    # no turns
    (3, 561, 128, 30),     # turns on a long head, under two rounds
    (3, 561, 128, 130),    # past a fifth: starts inside in index order only
    (3, 561, 128, 225),    # past two fifths: at the first entry
    (2, 1281, 128, 256),   # beyond 1280 blocks a fifth is the line for the kernel, too
    (2, 1281, 128, 257),
    (7, 801, 64, 80),      # d = 64: three waves of a SIMD take turns
    (7, 800, 64, 80),      # ... none do
    (3, 1000, 64, 100),    # two rounds of a long head with short lists
    (3, 1000, 64, 101),
])
def test_lines_of_the_rules_for_large_launches(usv, Hh, nb, d, kmax):
    """Against a 64-bit evaluation of sampled blocks, within the bf16 bound, and three times the same bits."""
    Nv = nb * 64 - 17
    gen = torch.Generator(device=gu.DEV).manual_seed(nb + kmax)
    q, k, v = ((torch.randn((1, Hh, nb, 64, d), device=gu.DEV, generator=gen) + 2 * torch.randn((1, Hh, nb, 1, d), device=gu.DEV, generator=gen))
               .view(1, Hh, nb * 64, d).to(torch.bfloat16) for _ in range(3))
    idx = torch.rand((1, Hh, nb, nb), device=gu.DEV, generator=gen).topk(kmax, dim=-1).indices.sort(-1).values.int()
    cnt = torch.full((1, Hh, nb), kmax, dtype=torch.int32, device=gu.DEV)
    for wo in (None, usv.attn_work_order(cnt, kmax, idx=idx)):
        runs = [usv.block_sparse_attn(q, k, v, idx, cnt, seq_valid=Nv, out_dtype=torch.float32, return_lse=True, work_order=wo) for _ in range(3)]
        assert all(torch.equal(a.view(torch.int32), b.view(torch.int32)) for r in runs[1:] for a, b in zip(r, runs[0]))
        for f in np.linspace(0, Hh * nb - 1, 11).astype(int):
            h, i = f // nb, f % nb
            keys = (idx[0, h, i].long()[:, None] * 64 + torch.arange(64, device=gu.DEV)).view(-1)
            keys = keys[keys < Nv]
            rows = slice(i * 64, min(i * 64 + 64, Nv))
            S = q[0, h, rows].double() @ k[0, h][keys].double().T / d ** 0.5
            what = f"head {h} block {i} ordered {wo is not None}"
            gu.assert_attn_close(gu.down(runs[0][0][0, h, rows]), (S.softmax(-1) @ v[0, h][keys].double()).cpu().numpy(), "bf16", what)
            assert (runs[0][1][0, h, rows] - S.logsumexp(-1)).abs().max() <= 2e-2, what


@pytest.mark.parametrize("Hh,nb,d,packed", [(13, 130, 128, True), (13, 130, 128, False), (43, 130, 64, True)])
def test_raster_rows_far_apart(usv, Hh, nb, d, packed):
    """Row offsets of a raster launch: tokens far apart (other columns of a wider projection lie between them), in random order, against the
    same tensors gathered; lists of 0, 1, 2 and more entries (the steps whose order entries are requested before the loop)."""
    gen = torch.Generator(device=gu.DEV).manual_seed(nb + d)
    N = nb * 64
    def tensor():
        x = torch.randn((1, N, Hh, d) if packed else (1, Hh, N, 3 * d), device=gu.DEV, generator=gen).to(torch.bfloat16)
        return x.transpose(1, 2) if packed else x[..., d:2 * d]
    q, k, v = tensor(), tensor(), tensor()
    idx = torch.rand((1, Hh, nb, nb), device=gu.DEV, generator=gen).topk(5, dim=-1).indices.sort(-1).values.int()
    cnt = torch.randint(0, 6, (1, Hh, nb), device=gu.DEV, generator=gen, dtype=torch.int32)
    order = torch.randperm(N, device=gu.DEV, generator=gen)
    out, lse = usv.block_sparse_attn_raster(q, k, v, order.int(), idx, cnt, out_dtype=torch.float32, return_lse=True)
    want, want_lse = usv.block_sparse_attn(*(t[:, :, order].contiguous() for t in (q, k, v)), idx, cnt, out_dtype=torch.float32, return_lse=True)
    assert torch.equal(out[:, :, order].view(torch.int32), want.view(torch.int32))
    assert torch.equal(lse[:, :, order].view(torch.int32), want_lse.view(torch.int32))
