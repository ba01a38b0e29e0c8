"""The residual selection where its route changes: one slice, two stages, the bucket filter
with a final selection in registers and a streamed one; scores that crowd into one bucket
(ties, zeros), that leave the buckets' range, and infinite or NaN ones.  The selected rows
follow the keys' order exactly, so each is compared with a stable sort of the keys that
the scoring left in the workspace (which other tests hold against the oracle's scores)."""
import numpy as np
import pytest

from tests._util import kv_all

pytestmark = pytest.mark.gpu


def _mass(kind, shape, seed):
    g = np.random.default_rng(seed)
    m = np.exp(3.0 * g.standard_normal(shape)).astype(np.float32)
    if kind == "zeros":  # most scores are 0 and tie
        m[g.random(shape) < 0.99] = 0.0
    elif kind == "signed":  # above, at and below the zeros that tie at the last place
        r = g.random(shape)
        m[r < 0.7] = 0.0
        m[r < 0.2] = -1.0
        m[r > 0.71] = 0.0
    elif kind == "same":  # every score is 0: one bucket holds all
        m[:] = 0.0
    elif kind == "wide":  # scores from below the lowest bucket's to the largest masses
        m = (np.exp2(g.uniform(-149, 127, shape))).astype(np.float32)
    elif kind == "odd":
        m[g.random(shape) < 0.01] = np.inf
        m[g.random(shape) < 0.01] = np.nan
        m[g.random(shape) < 0.3] *= -1
    return m


# slices * kept > 8192 takes the filter (with more than one slice): 8192 keys are one slice,
# (8193, 4096) is the last two-stage pair and (8193, 4097) the first filtered one;
# (16448, 8192) ends in registers or streamed by its list's length, 12000 always streamed
@pytest.mark.parametrize("T,n", [(8192, 5000), (8193, 4096), (8193, 4097), (16448, 8192), (20011, 12000),
                                 (20011, 20011), (40000, 1700), (131071, 2621)])
@pytest.mark.parametrize("kind", ["spread", "zeros", "signed", "same", "wide", "odd"])
def test_selection_follows_the_keys(gpu, T, n, kind):
    import torch
    B, H = (2, 2) if T < 131071 else (1, 1)
    ks, vs = kv_all(81, 1, 1, 4096)
    at = np.arange(T) * 7 % 4096  # every row is one of 4096: equal masses tie
    k = torch.from_numpy(np.broadcast_to(ks[:, :, at], (B, H, T, 128)).copy().view(np.int16)).cuda()
    v = torch.from_numpy(np.broadcast_to(vs[:, :, at], (B, H, T, 128)).copy().view(np.int16)).cuda()
    lv = np.full(-(-T // 64), 2, np.int8)
    if T % 64:
        lv[-1] = 16  # a partial block is exact
    cache = gpu.GradedCache.build(k, v, Hq=2 * H, levels=lv, nres_cap=n)
    for seed in (1, 2):  # the second call finds the first one's lists
        cache.rd_residual_select(k, v, torch.from_numpy(_mass(kind, (B, H, T), seed)).cuda(), n)
        stride = cache.nblk_cap * 64
        keys = cache.workspace(2)[: B * H * stride * 8].view(torch.int64).view(B, H, stride)[:, :, :T]
        keys = keys.cpu().numpy().view(np.uint64)
        rows = cache.res_idx.cpu().numpy()
        mask = cache.res_mask.cpu().numpy().view(np.uint64)
        off = cache.res_off.cpu().numpy()
        for b in range(B):
            for h in range(H):
                want = np.sort(np.argsort(~keys[b, h], kind="stable")[:n])
                np.testing.assert_array_equal(rows[b, h, :n], want)
                bits = np.zeros(stride, np.uint8)
                bits[want] = 1
                np.testing.assert_array_equal(mask[b, h], np.packbits(bits, bitorder="little").view(np.uint64))
                np.testing.assert_array_equal(off[b, h], np.concatenate([[0], np.cumsum(bits.reshape(-1, 64).sum(1))]))
