"""The fp32 attention kernel where splitting its operands into bf16 parts could go wrong: infinities, NaN, values beyond the largest
bf16, values whose lower parts run out of exponent (in V, and in one of Q and K with the other as large; weights that do so
beside values as large), padding of any finite value, halves of a block without a valid key."""
import numpy as np
import pytest
import torch

import gpu_util as gu

pytestmark = pytest.mark.gpu

FLT_MAX = np.float32(3.4028234e38)


def edit(what, Q, K, V, Nv):
    if what == "inf in v": V[0, 0, 70, 5] = np.inf
    if what == "nan in v": V[0, 0, 70, 5] = np.nan
    if what == "nan in q": Q[0, 1, 3, 5] = np.nan
    if what == "-inf logit":  # weight 0, not NaN
        Q[0, 0, :, 3] = np.abs(Q[0, 0, :, 3]) + 0.1
        K[0, 0, 70, 3] = -np.inf
    # Rounds to infinity as bf16 (above 3.396e38).  Not FLT_MAX itself: the largest weight is 2^(x - round(x)), |x| < 64 here, so it
    # may be 1 + 2^-19, and the sum before the division overflowed on fp32 operands too; 3.4e38 leaves 8e-4.
    if what == "beyond bf16": V[0, 0, 70, 5] = 3.4e38
    if what == "tiny v": V[..., 7] *= 1e-33
    if what == "tiny v, lower parts subnormal": V[..., 7] *= 1e-36
    if what == "subnormal v": V[..., 7] *= 1e-41
    if what == "zero v": V[..., 7] = 0
    if what == "huge q, tiny k":  # logits as of "plain"; the lower parts of k have no place in bf16
        Q *= np.float32(2.0 ** 118)
        K *= np.float32(2.0 ** -118)
    if what == "tiny q, huge k":
        Q *= np.float32(2.0 ** -120)
        K *= np.float32(2.0 ** 120)
    if what == "tiny weight, huge v":  # weights of about 2^-123 against values of 2^127
        Q *= np.float32(0.1)
        Q[..., 3] = 8
        K[..., 3] = 0
        K[:, :, 70, 3] = -85.5 * np.sqrt(Q.shape[-1]) / 8
        V[:, :, 70, 5] = 2.0 ** 127
    if what == "huge padding": Q[:, :, Nv:], K[:, :, Nv:], V[:, :, Nv:] = FLT_MAX, FLT_MAX, -FLT_MAX


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tail", [0, 44, 62, 32])  # padded rows of the last block: none, its second half empty, two keys, half
@pytest.mark.parametrize("what", ["plain", "inf in v", "nan in v", "nan in q", "-inf logit", "beyond bf16", "tiny v",
                                  "tiny v, lower parts subnormal", "subnormal v", "zero v", "huge q, tiny k", "tiny q, huge k",
                                  "tiny weight, huge v", "huge padding"])
@pytest.mark.parametrize("Hh", [2, 14, 52])  # 10 query blocks: sixteen rows to a workgroup; 70: eight waves a block; 260, just past one per CU: four
def test_f32_attention_special_values(usv, d, tail, what, Hh):
    nb, Nv = 5, 5 * 64 - tail
    rng = np.random.default_rng(d + tail)
    Q, K, V = (rng.standard_normal((1, Hh, nb * 64, d), dtype=np.float32) for _ in range(3))
    edit(what, Q, K, V, Nv)
    lists = [[0, 1, 2, 3, 4], [4], [1, 4], [], [3, 2, 1]]
    idx = np.full((1, Hh, nb, nb), -1, np.int32)
    cnt = np.zeros((1, Hh, nb), np.int32)
    for i, js in enumerate(lists):
        idx[:, :, i, :len(js)], cnt[:, :, i] = js, len(js)
    out, lse = usv.block_sparse_attn(gu.up(Q), gu.up(K), gu.up(V), gu.up(idx), gu.up(cnt), seq_valid=Nv, return_lse=True)
    o, l = gu.down(out), gu.down(lse)
    with np.errstate(all="ignore"):
        for h in (0, 1, Hh - 1):
            for i, js in enumerate(lists):
                got, rows = o[0, h, i * 64:(i + 1) * 64], max(0, min(64, Nv - i * 64))
                assert (got[rows:] == 0).all()
                keys = np.concatenate([np.arange(j * 64, min(j * 64 + 64, Nv)) for j in js]) if js else np.zeros(0, int)
                if not len(keys):
                    assert (got == 0).all() and np.isneginf(l[0, h, i * 64:(i + 1) * 64]).all()
                    continue
                S = Q[0, h, i * 64:i * 64 + rows].astype(np.float64) @ K[0, h, keys].astype(np.float64).T / np.sqrt(d)
                P = np.exp(S - S.max(axis=1, keepdims=True))
                ref = (P / P.sum(axis=1, keepdims=True)) @ V[0, h, keys].astype(np.float64)
                if what == "nan in q":  # a row without a row sum is written as zeros
                    bad = np.isnan(S).any(axis=1)
                    assert (got[:rows][bad] == 0).all()
                    got, ref, rows = got[:rows][~bad], ref[~bad], int((~bad).sum())
                got = got[:rows].astype(np.float64)
                assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref)), (what, h, i)
                # fp32 rounding of the inputs' products over at most 320 keys: 1e-5 of what the channel's values average
                fin = np.isfinite(ref)
                scale = np.abs(np.where(np.isfinite(V[0, h, keys]), V[0, h, keys], 0)).astype(np.float64).mean(axis=0)
                err = np.abs(np.where(fin, got - ref, 0))
                if what == "tiny weight, huge v":
                    # in channel 5 stands this one key's weight times 2^127.  Its product q k of about 970 rounds by 2^-15 in each of at
                    # most 32 sums of a partial sum, times log2(e) / sqrt(d) < 2^-2.4; the exponent of 123 by 2^-18 twice
                    rel = (32 * 2.0 ** -17.4 + 2 * 2.0 ** -18) * np.log(2)
                    own = (P / P.sum(axis=1, keepdims=True))[:, keys == 70].sum(axis=1) * 2.0 ** 127
                    assert (err[:, 5] <= rel * own + 1e-6).all(), (h, i, (err[:, 5] / own).max())
                    err[:, 5] = 0
                # (values of 1e-36 leave results a few of whose last bits lie under the fp32 normal range)
                assert (err <= 1e-5 * scale + 2.0 ** -126 * 1e-5 + 2.0 ** -149).all(), (what, h, i, (err / np.maximum(scale, 1e-45)).max())


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hh,nb", [(1, 1), (3, 21), (2, 32), (5, 13)])  # 1, 63, 64 query blocks: sixteen rows to a workgroup; 65: a block
@pytest.mark.parametrize("kmax", [1, 2, 4, 5, 13])  # halves of blocks for eight waves: fewer, just as many, one more round, several
def test_f32_attention_few_blocks(usv, d, Hh, nb, kmax):
    """Both sides of the rule for few query blocks against a 64-bit evaluation: ragged lists, empty ones, a partial last block."""
    kmax, Nv = min(kmax, nb), nb * 64 - 37
    rng = np.random.default_rng(nb * 100 + kmax)
    Q, K, V = (rng.standard_normal((1, Hh, nb * 64, d), dtype=np.float32) for _ in range(3))
    cnt = rng.integers(0, kmax + 1, size=(1, Hh, nb)).astype(np.int32)
    idx = np.sort(np.argsort(rng.random((1, Hh, nb, nb)), axis=-1)[..., :kmax], axis=-1).astype(np.int32)
    out, lse = usv.block_sparse_attn(gu.up(Q), gu.up(K), gu.up(V), gu.up(idx), gu.up(cnt), seq_valid=Nv, return_lse=True)
    o, l = gu.down(out), gu.down(lse)
    for h in range(Hh):
        for i in range(nb):
            rows = min(64, Nv - i * 64)
            keys = [np.arange(j * 64, min(j * 64 + 64, Nv)) for j in idx[0, h, i, :cnt[0, h, i]]]
            keys = np.concatenate(keys) if keys else np.zeros(0, int)
            assert (o[0, h, i * 64 + rows:(i + 1) * 64] == 0).all() and np.isneginf(l[0, h, i * 64 + rows:(i + 1) * 64]).all()
            got, got_l = o[0, h, i * 64:i * 64 + rows], l[0, h, i * 64:i * 64 + rows]
            if not len(keys):
                assert (got == 0).all() and np.isneginf(got_l).all()
                continue
            S = Q[0, h, i * 64:i * 64 + rows].astype(np.float64) @ K[0, h, keys].astype(np.float64).T / np.sqrt(d)
            m = S.max(axis=1, keepdims=True)
            P = np.exp(S - m)
            gu.assert_f32_close(got, P @ V[0, h, keys].astype(np.float64) / P.sum(axis=1, keepdims=True), f"head {h} block {i}")
            assert np.abs(got_l - (m[:, 0] + np.log(P.sum(axis=1)))).max() <= 1e-4
