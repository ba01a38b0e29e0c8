"""The block encoder at the inputs where its fast paths hand over to the fp64 ones: exact
ties of the quotient, margins, subnormal scales, near and equal centroid distances, large
and tiny magnitudes; every stored code, scale, zero, centroid and id against the oracle."""
import numpy as np
import pytest

from oracle import cache as ocache
from oracle.quant import P, D, encode_fp16, demote as odemote, decode as odecode
from tests._util import compare_record

pytestmark = pytest.mark.gpu


def _block(kind, g):
    x = g.standard_normal((P, D)).astype(np.float64)
    if kind == "grid":  # few distinct values: exact half-integer quotients everywhere
        x = np.rint(4 * x) / 8
    elif kind == "grid_outliers":
        x = np.rint(4 * x) / 8
        x[:, ::17] *= 64
    elif kind == "subnormal":  # scales below the fp16 normal range, or zero
        x *= 2.0 ** g.integers(-24, -14, D)[None, :]
    elif kind == "wide":  # magnitudes from the smallest subnormal to the largest value
        x *= 2.0 ** g.integers(-22, 13, D)[None, :]
        x = np.clip(x, -65504, 65504)
    elif kind == "constant":
        x[:] = x[0]
        x[:, 5] = 0.0
    elif kind == "equal_rows":  # rows in a few groups: equal centroid distances, empty clusters
        x = x[g.integers(0, 3, P)]
    elif kind == "mirrored":  # tokens equally far from two initial centroids
        x[16] = -x[0]
        x[48] = -x[32]
        x[1::2] = 0.0
        x[48] = -x[32]
    elif kind == "near_rows":  # distances that differ in the last places
        x = x[:1] + np.rint(g.standard_normal((P, D))) * 2.0 ** -9
    elif kind in ("near_zero", "near_zero_ulp"):  # tokens near zero, centroids of (nearly) equal norm
        far = x[0] * 4
        x *= 2.0 ** -14
        for i in (0, 16, 32, 48):
            x[i] = g.permutation(far) * g.choice((-1.0, 1.0), D)
        if kind == "near_zero_ulp":
            x[32, 7] *= 1 + 2.0 ** -10
            x[1::3] = 0.0
    elif kind == "random":
        x[:, ::31] *= 10
    else:
        raise ValueError(kind)
    return x.astype(np.float16).view(np.uint16)


KINDS = ("random", "grid", "grid_outliers", "subnormal", "wide", "constant", "equal_rows", "mirrored", "near_rows",
         "near_zero", "near_zero_ulp")


def _tensors(seed):
    g = np.random.default_rng(seed)
    k = np.concatenate([_block(kind, g) for kind in KINDS])[None, None]
    v = np.concatenate([_block(kind, g) for kind in KINDS])[None, None]
    return k, v


@pytest.mark.parametrize("per_token", (False, True))
@pytest.mark.parametrize("level", (8, 4, 2, 1, 0))
def test_encode_edges_match_oracle(gpu, level, per_token):
    k, v = _tensors(10 * level + per_token)
    n = len(KINDS)
    levels = np.full(n, level, np.int8)
    cache = gpu.GradedCache.build(k, v, Hq=1, levels=levels, v_per_token=per_token)
    uc = ocache.UnitCache(k[0, 0], v[0, 0], levels, v_per_token=per_token)
    cert = cache.cert[0, 0].cpu().numpy().astype(np.float64)
    for i in range(n):
        for t, recs in ((0, uc.k_recs), (1, uc.v_recs)):
            compare_record(cache, uc, 0, 0, i, t)
            x = (k, v)[t][0, 0, i * P:(i + 1) * P].view(np.float16).astype(np.float64)
            err = np.sqrt(((x - odecode(recs[i])) ** 2).sum(-1).max())
            # fp64 sums rounded up to fp32: at least the error, at most one fp32 step above
            assert err * (1 - 1e-12) <= cert[i, t] <= err * (1 + 2.4e-7) + 1e-44, (KINDS[i], t)
        nrm = np.sqrt((v[0, 0, i * P:(i + 1) * P].view(np.float16).astype(np.float64) ** 2).sum(-1).max())
        assert nrm * (1 - 1e-12) <= cert[i, 2] <= nrm * (1 + 2.4e-7) + 1e-44, KINDS[i]


@pytest.mark.parametrize("per_token", (False, True))
@pytest.mark.parametrize("chain", ((8, 4, 2, 1, 0), (4, 1), (2, 0), (8, 2)))
def test_demotion_edges_match_oracle(gpu, chain, per_token):
    k, v = _tensors(100 + sum(chain) + per_token)
    n = len(KINDS)
    cache = gpu.GradedCache.build(k, v, Hq=1, levels=np.full(n, 16, np.int8), v_per_token=per_token,
                                  slack={lv: n for lv in chain}, extra_blocks=0)
    recs = {(t, i): encode_fp16(16, (k, v)[t][0, 0, i * P:(i + 1) * P], per_token and t == 1)
            for t in (0, 1) for i in range(n)}
    uc = ocache.UnitCache(k[0, 0], v[0, 0], np.full(n, 16, np.int8), v_per_token=per_token)
    for lv in chain:
        cache.demote([(0, 0, i) for i in range(n)], [lv] * n)
        recs = {key: odemote(r, lv) for key, r in recs.items()}
        uc.k_recs = [recs[0, i] for i in range(n)]
        uc.v_recs = [recs[1, i] for i in range(n)]
        for i in range(n):
            for t in (0, 1):
                compare_record(cache, uc, 0, 0, i, t)


@pytest.mark.parametrize("per_token", (False, True))
@pytest.mark.parametrize("chain", ((8, 4, 2, 1, 0), (2, 1), (4, 0)))
def test_demotion_in_place(gpu, chain, per_token):
    """The new record at its old record's offset: the same bytes as in a slot of its own."""
    import ctypes
    k, v = _tensors(200 + sum(chain) + per_token)
    k, v = np.tile(k, (1, 1, 7, 1)), np.tile(v, (1, 1, 7, 1))  # several workgroups on a compute unit
    n = k.shape[2] // P
    apart = gpu.GradedCache.build(k, v, Hq=1, levels=np.full(n, 16, np.int8), v_per_token=per_token,
                                  slack={lv: n for lv in chain})
    inplace = gpu.GradedCache.build(k, v, Hq=1, levels=np.full(n, 16, np.int8), v_per_token=per_token)
    jobs = np.array([(0, 0, i) for i in range(n)], np.int32)
    ko, vo = inplace.koff_host[0, 0].copy(), inplace.voff_host[0, 0].copy()
    for lv in chain:
        to = np.full(n, lv, np.int8)
        apart.demote([tuple(j) for j in jobs], to)
        st = gpu._demote(ctypes.byref(inplace.c), n, gpu._np_ptr(jobs), gpu._np_ptr(to), gpu._np_ptr(ko),
                         gpu._np_ptr(vo), gpu._stream())
        assert st == 0
        for i in range(n):
            for t in (0, 1):
                assert inplace.record_bytes(0, 0, i, t) == apart.record_bytes(0, 0, i, t), (lv, KINDS[i % len(KINDS)], t)
    assert np.array_equal(inplace.cert.cpu().numpy(), apart.cert.cpu().numpy())
