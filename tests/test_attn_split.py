"""The attention read's split over workgroups and its workspace ranges, on the host: over
the accepted shapes neither kernel makes more workgroups per (sequence, KV head) than the
merge kernel's LDS holds, and the partials stay inside the workspace."""
import ctypes
import itertools

import numpy as np
import pytest

PLANNED = 0


@pytest.fixture(scope="module")
def B():
    from paper_2608_23599_amd import binding
    return binding


def extents(B, batch, kv, group, T, cap=None, nres=0, nres_cap=0, page=0, topk=0):
    """gkv_attn_extents of a cache of these sizes (the call reads no table), or its error."""
    c = B.CacheStruct()
    c.B, c.Hkv, c.Hq, c.D, c.T = batch, kv, kv * group, 128, T
    c.nblk_cap = cap or -(-T // 64)
    c.nres, c.nres_cap, c.page = nres, max(nres, nres_cap), page
    out = (ctypes.c_int64 * 8)()
    st = B.lib.gkv_attn_extents(ctypes.byref(c), ctypes.c_int32(topk), out)
    if st != 0:
        return st
    return dict(zip(("waves", "nsplit", "limit", "part", "part_end", "lists", "lists_end", "total"), out))


def _dense_shapes():
    tokens = [1, 64, 65, 1024, 1025, 2048, 16384, 16385, 32768, 60000, 65535, 65536, 65537, 70001, 98304, 131072,
              131073, 1 << 20, 2097024]
    for batch, kv, group, T in itertools.product((1, 2, 3, 4, 8, 64), (1, 2, 4, 8), (1, 4, 16), tokens):
        nb = -(-T // 64)
        for nres in {0, 1, T // 50, T // 10}:
            for cap in (nb, nb + 2048):
                if cap + -(-nres // 64) <= 32767:
                    yield dict(batch=batch, kv=kv, group=group, T=T, cap=cap, nres=nres)


def _quest_shapes():
    topks = [1, 2, 3, 30, 31, 128, 256, 510, 511, 512, 600, 1022, 1023, 1024, 1025, 2000, 2047, 2048, 4095, 8000, 8191]
    for batch, kv, group, page, topk, nres_cap in itertools.product((1, 2, 8, 33), (1, 4, 8), (1, 4, 16),
                                                                    (16, 32, 64), topks, (0, 100)):
        for nres in {0, nres_cap}:
            yield dict(batch=batch, kv=kv, group=group, T=1 << 20, nres=nres, nres_cap=nres_cap, page=page, topk=topk)


@pytest.mark.parametrize("shapes", [_dense_shapes, _quest_shapes])
def test_splits_fit_the_merge_and_the_workspace(B, shapes):
    seen = set()
    for s in shapes():
        e = extents(B, **s)
        if not isinstance(e, dict):
            assert e == -6 and s.get("topk"), (s, e)  # more read tiles than the call accepts
            continue
        seen.add(e["waves"] == PLANNED)
        if e["waves"] != PLANNED and e["nsplit"] > 1:  # resident at once: one dense workgroup on each
            # of 256 compute units, three of a page read
            assert s["batch"] * s["kv"] * e["nsplit"] <= (768 if s.get("topk") else 256), (s, e)
        assert 1 <= e["nsplit"] <= e["limit"] == 256, (s, e)
        assert e["part"] >= 256 and e["part_end"] <= e["total"], (s, e)
        assert e["lists_end"] <= e["total"] and (e["waves"] != PLANNED or e["part_end"] <= e["lists"]), (s, e)
        # the planned kernel's layout that fits the library's array (32 MiB) is not refused
        # for the short read's partials
        assert e["total"] <= max(e["lists_end"] + 512, 32 << 20), (s, e)
    assert seen == {True, False}  # both kernels are among them


def test_splits_at_the_merge_limit(B):
    """256 workgroups are the most a read is split into; one more goes to the planned kernel."""
    for e in (extents(B, 1, 1, 16, 65536), extents(B, 1, 1, 4, 900 * 64, nres=124 * 64),
              extents(B, 1, 1, 4, 1 << 20, page=16, topk=1023), extents(B, 1, 1, 4, 1 << 20, page=64, topk=511)):
        assert e["waves"] != PLANNED and e["nsplit"] == 256, e
    for e in (extents(B, 1, 1, 16, 65537), extents(B, 1, 1, 16, 131072), extents(B, 1, 1, 4, 900 * 64, nres=124 * 64 + 1),
              extents(B, 1, 1, 4, 1 << 20, page=16, topk=1024), extents(B, 1, 8, 4, 1 << 20, page=32, topk=1024),
              extents(B, 1, 1, 4, 1 << 20, page=64, topk=512)):
        assert e["waves"] == PLANNED and e["nsplit"] <= 256, e


def test_short_partials_may_reach_another_layouts_plan(B):
    """Calls that share a workspace have layouts of their own: a sparse read's partials can
    lie where a dense read keeps its plan (the reason why no read without a plan of its own
    leaves a plan's tag valid)."""
    for batch, kv, T, topk in ((8, 8, 131072, 128), (8, 8, 16384, 128), (4, 4, 10000, 200)):
        d = extents(B, batch, kv, 4, T, page=16)
        s = extents(B, batch, kv, 4, T, page=16, topk=topk)
        assert d["waves"] == PLANNED and d["part_end"] <= d["lists"] <= d["lists_end"] <= d["total"]
        assert s["waves"] != PLANNED and d["lists"] < s["part_end"] <= s["total"]


def test_dense_workspace_is_the_planned_kernels(B):
    """The dense workspace of a cache whose lists outweigh the short read's partials: the
    tag, the planned kernel's partials and splits, and 32 + 4 * 16 + 8 * 16 bytes per visit."""
    for batch, kv, group, T, nres in ((8, 4, 7, 131072, 2621), (8, 8, 4, 131072, 0), (4, 4, 4, 140000, 0),
                                      (2, 2, 16, 65536, 1000)):
        units, visits = batch * kv, -(-T // 64) + -(-nres // 64)
        e = extents(B, batch, kv, group, T, nres=nres)
        ncap = -(-min(2048 // units, visits) // 4)
        lists = 256 + -(-units * ncap * group * 133 * 4 // 256) * 256
        assert e["lists"] == lists, e
        up = lambda x: -(-x // 256) * 256
        want = (lists + up(units * 2 * (4 * ncap + 1) * 4) + up(units * visits * 32) + up(units * visits * 64) +
                units * visits * 128 + 512)
        assert e["total"] == want, (e, want)


def test_noalloc_array_takes_the_largest_planned_layout(B):
    """The longest dense read whose planned layout fits the array's 32 MiB is not refused."""
    units, group = 64, 16
    T = max(t for t in range(64 * 1900, 64 * 2100, 64)
            if extents(B, 8, 8, group, t)["lists_end"] + 512 <= 32 << 20)
    assert extents(B, 8, 8, group, T)["total"] <= 32 << 20
