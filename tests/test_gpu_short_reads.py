"""Dense reads at the sizes where the read changes kernels: one workgroup per (sequence,
KV head) up to 16 two-tile pieces (8 blocks), several workgroups up to 4096 pieces over all
of them, with more than one piece a wavefront where more workgroups than are resident would
be needed, the planned kernel beyond; ragged lengths, residual rows, values per token and
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


# blocks: 8 is the last one-workgroup read, 9 the first split one; with 8 KV heads 128 blocks
# are one piece a wavefront of 32 workgroups each, 129 some second ones, 256 make 4096 pieces
# and 257 go to the planned kernel
@pytest.mark.parametrize("prof", ["tiny", "graded"])
@pytest.mark.parametrize("T,Hq,Hkv", [(1, 4, 2), (17, 4, 2), (64, 32, 2), (64 * 15 + 33, 12, 2), (64 * 16, 12, 2),
                                      (64 * 16 + 1, 12, 2), (64 * 40 - 7, 20, 2), (64 * 8, 20, 2),
                                      (64 * 8 + 1, 20, 2), (64 * 128 + 1, 8, 8), (64 * 256, 8, 8),
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


@pytest.mark.parametrize("lens", [(1, 64 * 3, -1, 64 * 9 + 5), (64 * 30, 7, 64 * 16, 64),
                                  (64 * 300 + 5, 7, -1, 64 * 130 + 1)])  # the last one: the planned kernel
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


# 65536 tokens of one unit are 256 workgroups' pieces, the most the merge holds; one token
# more, or residual pseudo-blocks past 1024 blocks in all, go to the planned kernel
@pytest.mark.parametrize("T,Hq,nres,vtok", [(65536, 4, 0, False), (65537, 16, 0, False), (131072, 4, 0, False),
                                            (900 * 64, 4, 124 * 64, False), (900 * 64, 4, 124 * 64 + 1, False),
                                            (65537, 4, 0, True), (65600, 12, 0, True)])
def test_one_long_unit_at_the_merge_limit(gpu, T, Hq, nres, vtok):
    """The long ones are the planned kernel's: its certificate for packed and unpacked groups,
    residual rows and values per token."""
    import torch
    ks, vs = kv_all(74, 1, 1, T)
    lv = olad.ladder("tiny", T)
    cache = gpu.GradedCache.build(ks, vs, Hq=Hq, levels=lv, nres_cap=nres, v_per_token=vtok)
    uc = ocache.UnitCache(ks[0, 0], vs[0, 0], lv, v_per_token=vtok)
    if nres:
        mass = synth.mass_unit(74, 0, 0, T)[None, None].astype(np.float32)
        cache.rd_residual_select(ks, vs, mass, nres)
        uc.select_residual(ks[0, 0], vs[0, 0], mass[0, 0], nres)
    q = synth.queries(74, 1, Hq)
    out = cache.decode(q)
    assert torch.equal(out, cache.decode(q)) and torch.equal(out, _staged(gpu, cache, q))
    with_bound, bound = cache.decode_bound(q)
    assert max_err(out[0].cpu().numpy(), uc.decode_dense(q[0])) <= TOL
    assert max_err(with_bound[0].cpu().numpy(), uc.decode_dense(q[0])) <= TOL
    want = uc.certificate(q[0])
    assert np.all(np.abs(bound[0].cpu().numpy() - want) <= 2e-3 * want + 1e-6)


# 1024 pieces of a unit's pages are 256 workgroups
@pytest.mark.parametrize("page,topk", [(16, 1023), (16, 1024), (32, 1024), (64, 511), (64, 512)])
@pytest.mark.parametrize("Hq,Hkv", [(4, 1), (32, 8)])
def test_many_pages_at_the_merge_limit(gpu, page, topk, Hq, Hkv):
    T = page * (topk + 40) + 5
    G = Hq // Hkv
    ks, vs = kv_all(75, 1, Hkv, T)
    lv = olad.ladder("tiny", T)
    cache = gpu.GradedCache.build(ks, vs, Hq=Hq, levels=lv, page=page)
    q = synth.queries(75, 1, Hq)
    pages = cache.quest_select(q, topk)
    out = cache.decode(q, pages=pages).cpu().numpy()
    for h in {0, Hkv - 1}:
        uc = ocache.UnitCache(ks[0, h], vs[0, h], lv)
        ref = uc.decode_quest(q_group(q, 0, h, G), pages[0, h].cpu().numpy(), page)
        assert max_err(out[0, h * G:(h + 1) * G], ref) <= TOL


# 64 (sequence, KV head) share 768 workgroups: 12 each, whose 48 wavefronts take a piece each
# up to 48 pieces and more beyond; 800 leave one workgroup each
@pytest.mark.parametrize("B,Hkv,page,topk", [(16, 4, 16, 47), (16, 4, 16, 48), (16, 4, 32, 100), (16, 4, 64, 60),
                                             (100, 8, 16, 21)])
def test_pages_beyond_one_piece_a_wavefront(gpu, B, Hkv, page, topk):
    T = page * (topk + 9) + 3
    G = 4
    ks, vs = kv_all(76, 1, Hkv, T)
    ks, vs = np.repeat(ks, B, 0), np.repeat(vs, B, 0)
    lv = olad.ladder("tiny", T)
    cache = gpu.GradedCache.build(ks, vs, Hq=Hkv * G, levels=lv, page=page)
    q = synth.queries(76, B, Hkv * G)
    pages = cache.quest_select(q, topk)
    out = cache.decode(q, pages=pages)
    assert np.array_equal(out.cpu().numpy(), cache.decode(q, pages=pages).cpu().numpy())
    for b, h in ((0, 0), (B - 1, Hkv - 1)):
        uc = ocache.UnitCache(ks[b, h], vs[b, h], lv)
        ref = uc.decode_quest(q_group(q, b, h, G), pages[b, h].cpu().numpy(), page)
        assert max_err(out[b, h * G:(h + 1) * G].cpu().numpy(), ref) <= TOL
