"""Reads of different kinds and caches on one workspace, in stream order: a read whose
partials lie where an earlier call's layout keeps its dense plan must not leave that plan
valid.  Every output against the same call on a workspace of its own, bit for bit."""
import ctypes

import numpy as np
import pytest

from oracle import ladder as olad
from paper_2608_23599_amd import synth
from tests._util import kv_all
from tests.test_attn_split import PLANNED, extents

pytestmark = pytest.mark.gpu

BATCH, HKV, GROUP, T, PAGE, TOPK = 4, 4, 4, 10000, 16, 200


def _extents(gpu, c, topk=0):
    return extents(gpu, c.B, c.Hkv, c.Hq // c.Hkv, c.T, c.nblk_cap, c.c.nres, c.c.nres_cap, c.page, topk)


class Shared:
    """Calls on one caller workspace, or on the library's own array."""

    def __init__(self, gpu, noalloc, nbytes):
        import torch
        self.gpu, self.noalloc = gpu, noalloc
        self.ws = None if noalloc else torch.zeros(nbytes, dtype=torch.uint8, device="cuda")

    def read(self, c, q, pages=None):
        import torch
        gpu, out = self.gpu, torch.full((c.B, c.Hq, 128), float("nan"), device="cuda")
        head = (gpu._dptr(q), ctypes.byref(c.c), gpu._dptr(pages), 0 if pages is None else pages.shape[-1],
                gpu._dptr(out))
        if self.noalloc:
            assert gpu._attn_noalloc(*head, gpu._stream()) == 0
        else:
            assert gpu._attn(*head, gpu._dptr(self.ws), self.ws.numel(), gpu._stream()) == 0
        return out

    def tag(self):
        import torch
        torch.cuda.synchronize()
        return [int(x) for x in self.ws[:96].cpu().numpy().view(np.uint64)]


def _cache(gpu, wl, batch, hkv, hq, tokens, **kw):
    ks, vs = kv_all(wl, batch, hkv, tokens)
    c = gpu.GradedCache.build(ks, vs, Hq=hq, levels=olad.ladder("tiny", tokens), **kw)
    return c, gpu._as_bits(synth.queries(wl, batch, hq), c._dev)


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("residual", [False, True])
def test_dense_quest_dense(gpu, noalloc, residual):
    """With residual rows the sparse read runs the planned kernel, without them the short one."""
    import torch
    nres = 200 if residual else 0
    c, q = _cache(gpu, 91, BATCH, HKV, HKV * GROUP, T, page=PAGE, nres_cap=nres)
    if residual:
        ks, vs = kv_all(91, BATCH, HKV, T)
        mass = np.stack([np.stack([synth.mass_unit(91, b, h, T) for h in range(HKV)]) for b in range(BATCH)])
        c.rd_residual_select(ks, vs, mass, nres)
    d, s = _extents(gpu, c), _extents(gpu, c, TOPK)
    assert d["waves"] == PLANNED and (s["waves"] == PLANNED) == residual
    assert residual or s["part_end"] > d["lists"]  # the sparse partials reach the dense plan
    pages = c.quest_select(q, TOPK)
    want, want_sparse = c.decode(q), c.decode(q, pages=pages)
    sh = Shared(gpu, noalloc, max(d["total"], s["total"]))
    for _ in range(2):
        assert torch.equal(sh.read(c, q), want)
        assert noalloc or sh.tag()[0] == c.c.version
        assert torch.equal(sh.read(c, q), want)  # on the kept plan
        assert torch.equal(sh.read(c, q, pages), want_sparse)
        assert noalloc or sh.tag()[0] == 0
    assert torch.equal(sh.read(c, q), want)


@pytest.mark.parametrize("noalloc", [False, True])
def test_unstamped_short_read_between_planned_reads(gpu, noalloc):
    """A cache whose version is 0 (unknown state) is read on the short path between two
    planned reads of another cache."""
    import torch
    a, qa = _cache(gpu, 92, BATCH, HKV, HKV * GROUP, T)
    b, qb = _cache(gpu, 93, 2, 8, 128, 64 * 128)
    b.c.version = 0
    da, db = _extents(gpu, a), _extents(gpu, b)
    assert da["waves"] == PLANNED and db["waves"] != PLANNED and db["part_end"] > da["lists"]
    want_a, want_b = a.decode(qa), b.decode(qb)
    sh = Shared(gpu, noalloc, max(da["total"], db["total"]))
    for _ in range(2):
        assert torch.equal(sh.read(a, qa), want_a)
        assert torch.equal(sh.read(b, qb), want_b)
        assert noalloc or sh.tag()[0] == 0
    assert torch.equal(sh.read(a, qa), want_a)
