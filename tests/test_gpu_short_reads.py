"""Dense reads at the sizes where the read changes kernels: one workgroup per (sequence,
KV head) up to 32 two-tile pieces (16 blocks), several workgroups up to 4096 pieces over all
of them, the planned kernel beyond; ragged lengths, residual rows, values per token and
groups of more than 8 heads in each.  Against the oracle within the attention tolerance, and
the staged calls and the certificate read against the plain call bit for bit."""
import numpy as np
import pytest

from oracle import cache as ocache, ladder as olad
from paper_2608_23599_amd import synth
from tests._util import TOL, kv_all, max_err, q_group

pytestmark = pytest.mark.gpu


def _staged(gpu, cache, q):
    import torch
    out = torch.empty_like(cache.decode(q))
    cache.attn_plan()
    cache.attn_partials(q)
    cache.attn_merge(out)
    return out


# blocks: 16 is the last one-workgroup read, 17 the first split one; with 8 KV heads 256
# blocks make 4096 pieces and 257 go to the planned kernel
@pytest.mark.parametrize("prof", ["tiny", "graded"])
@pytest.mark.parametrize("T,Hq,Hkv", [(1, 4, 2), (17, 4, 2), (64, 32, 2), (64 * 15 + 33, 12, 2), (64 * 16, 12, 2),
                                      (64 * 16 + 1, 12, 2), (64 * 40 - 7, 20, 2), (64 * 256, 8, 8),
                                      (64 * 256 + 1, 8, 8)])
def test_dense_reads_across_the_kernels(gpu, T, Hq, Hkv, prof):
    import torch
    vtok = T % 2 == 1
    G = Hq // Hkv
    ks, vs = kv_all(71, 1, Hkv, T)
    lv = olad.ladder(prof, T)
    cache = gpu.GradedCache.build(ks, vs, Hq=Hq, levels=lv, v_per_token=vtok)
    q = synth.queries(71, 1, Hq)
    out = cache.decode(q)
    assert torch.equal(out, cache.decode(q)) and torch.equal(out, _staged(gpu, cache, q))
    assert torch.equal(out, cache.decode_bound(q)[0])
    for h in (0, Hkv - 1):
        uc = ocache.UnitCache(ks[0, h], vs[0, h], lv, v_per_token=vtok)
        assert max_err(out[0, h * G:(h + 1) * G].cpu().numpy(), uc.decode_dense(q_group(q, 0, h, G))) <= TOL


@pytest.mark.parametrize("T,pct", [(64 * 6 + 11, 10), (64 * 15, 10), (64 * 20, 25), (64 * 12, 0)])
def test_short_reads_with_residual_rows(gpu, T, pct):
    """Residual pseudo-blocks count as pieces; a block all of whose tokens in one piece are
    residual rows reads nothing there."""
    Hq, Hkv = 8, 2
    ks, vs = kv_all(72, 1, Hkv, T)
    lv = olad.ladder("tiny", T)
    n = T * pct // 100
    mass = np.stack([synth.mass_unit(72, 0, h, T) for h in range(Hkv)])[None].astype(np.float32)
    mass[:, :, 64:96] += 1.0  # one whole piece of block 1
    cache = gpu.GradedCache.build(ks, vs, Hq=Hq, levels=lv, nres_cap=max(n, 1))
    cache.rd_residual_select(ks, vs, mass, n)
    q = synth.queries(72, 1, Hq)
    out = cache.decode(q).cpu().numpy()
    for h in range(Hkv):
        uc = ocache.UnitCache(ks[0, h], vs[0, h], lv)
        uc.select_residual(ks[0, h], vs[0, h], mass[0, h], n)
        assert max_err(out[0, h * 4:(h + 1) * 4], uc.decode_dense(q_group(q, 0, h, 4))) <= TOL


@pytest.mark.parametrize("lens", [(1, 64 * 3, -1, 64 * 9 + 5), (64 * 30, 7, 64 * 16, 64)])
def test_short_reads_of_ragged_batches(gpu, lens):
    """Each sequence reads its own pieces; a retired one's output is zero."""
    T, Hq, Hkv = max(lens), 8, 2
    ks, vs = kv_all(73, len(lens), Hkv, T)
    nblk = -(-T // 64)
    lv = np.full((len(lens), Hkv, nblk), 16, np.int8)
    for b, t in enumerate(lens):
        if t > 0:
            lv[b, :, :-(-t // 64)] = olad.ladder("tiny", t)
    cache = gpu.GradedCache.build(ks, vs, Hq=Hq, levels=lv, seq_lens=list(lens))
    q = synth.queries(73, len(lens), Hq)
    out = cache.decode(q).cpu().numpy()
    for b, t in enumerate(lens):
        for h in range(Hkv):
            got = out[b, h * 4:(h + 1) * 4]
            if t < 0:
                assert not got.any()
                continue
            uc = ocache.UnitCache(ks[b, h, :t], vs[b, h, :t], olad.ladder("tiny", t))
            assert max_err(got, uc.decode_dense(q_group(q, b, h, 4))) <= TOL
