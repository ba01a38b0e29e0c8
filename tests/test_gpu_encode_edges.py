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


# ---------------------------------------------------------------- infinities and NaN
# The encoder's rules where the oracle's numpy ones differ: a NaN is ignored by a group's
# minimum and maximum unless it is the group's first element, then both are NaN; a quotient
# that is NaN gives code 0; a centroid is nearer only where its distance compares below.


def _odd_block(kind, g):
    b = g.standard_normal((P, D)).astype(np.float16).view(np.uint16)
    def put(n, bits, rows):
        b[g.choice(rows, n), g.integers(0, D, n)] = g.choice(np.array(bits, np.uint16), n)
    inf, nan = (0x7C00, 0xFC00), (0x7E00, 0xFE00, 0x7E55)
    every = np.arange(P)
    if kind == "inf":
        put(1, inf, every)
    elif kind == "infs":
        put(40, inf, every)
    elif kind == "nan":
        put(1, nan, every[1:])
    elif kind == "nans":
        put(40, nan, every)
    elif kind == "first":  # a channel's first row, a token's first channel
        put(5, nan + inf, every[:1])
        b[20:24, 0] = (0x7E00, 0x7C00, 0xFC00, 0xFE00)
    elif kind == "seeds":  # the rows that the centroids start from
        put(9, nan + inf, every[::16])
    elif kind == "lines":
        b[:, 5], b[:, 9], b[:, 11], b[3], b[17] = 0x7E00, 0x7C00, 0xFC00, 0xFE00, 0x7C00
    elif kind == "largest":
        b[:] = g.choice(np.array((0x7BFF, 0xFBFF), np.uint16), (P, D))
    else:
        b[:] = {"all_nan": 0x7E00, "all_inf": 0x7C00}[kind]
    return b


ODD = ("inf", "infs", "nan", "nans", "first", "seeds", "lines", "largest", "all_nan", "all_inf")


def _f16(x):
    return (x + 0.0).astype(np.float16)  # -0 gives +0


def _ref_scalar(x, bits, axis):
    x = x if axis == 0 else x.T
    first = np.isnan(x[0])
    with np.errstate(all="ignore"):
        mn, mx = np.fmin.reduce(x, 0), np.fmax.reduce(x, 0)
        mn[first] = mx[first] = np.nan
        q = (1 << bits) - 1
        z, s = _f16(mn), _f16((mx - mn) / q)
        t = np.rint((x - z.astype(np.float64)) / s.astype(np.float64))
        t = np.where(np.isnan(t) | (s == 0), 0, np.clip(t, 0, q)).astype(np.int32)
    return (t if axis == 0 else t.T), s, z


def _ref_lloyd(x, k):
    def nearest(c):
        d = np.zeros((P, k))
        for ch in range(D):
            d = d + (x[:, ch, None] - c[None, :, ch]) ** 2
        best = np.zeros(P, np.int32)
        for j in range(1, k):
            best = np.where(d[:, j] < d[np.arange(P), best], j, best)
        return best

    with np.errstate(all="ignore"):
        if k == 1:
            return _f16(np.add.accumulate(x, 0)[-1:] / P), np.zeros(P, np.int32)
        c, prev = x[::P // k].copy(), None
        for _ in range(10):
            a = nearest(c)
            if prev is not None and np.array_equal(a, prev):
                break
            prev = a
            for j in range(k):
                if (a == j).any():
                    c[j] = np.add.accumulate(x[a == j], 0)[-1] / (a == j).sum()
        c = _f16(c)
        return c, nearest(c.astype(np.float64))


@pytest.mark.parametrize("per_token", (False, True))
@pytest.mark.parametrize("level,demoted", [(lv, d) for lv in (16, 8, 4, 2, 1, 0) for d in (False, True) if lv < 16 or not d])
def test_infinities_and_nan(gpu, level, demoted, per_token):
    """Encoded from rows, and demoted from an exact record."""
    g = np.random.default_rng(300 + level)
    k, v = (np.concatenate([_odd_block(kind, g) for kind in ODD])[None, None] for _ in range(2))
    n = len(ODD)
    cache = gpu.GradedCache.build(k, v, Hq=1, levels=np.full(n, 16 if demoted else level, np.int8),
                                  v_per_token=per_token, slack={level: n})
    if demoted:
        cache.demote([(0, 0, i) for i in range(n)], [level] * n)
    for i in range(n):
        for t in (0, 1):
            x = (k, v)[t][0, 0, i * P:(i + 1) * P].view(np.float16).astype(np.float64)
            got = cache.record(0, 0, i, t)
            what = f"{ODD[i]} {t}"
            if level == 16:
                np.testing.assert_array_equal(got["values"], x, err_msg=what)
            elif level in (1, 0):
                cent, ids = _ref_lloyd(x, 4 if level else 1)
                np.testing.assert_array_equal(got["cent16"].view(np.float16), cent, err_msg=what)
                np.testing.assert_array_equal(got["ids"], ids, err_msg=what)
            else:
                codes, s, z = _ref_scalar(x, level, 1 if per_token and t else 0)
                np.testing.assert_array_equal(got["s16"].view(np.float16), s, err_msg=what)
                np.testing.assert_array_equal(got["z16"].view(np.float16), z, err_msg=what)
                np.testing.assert_array_equal(got["codes"], codes, err_msg=what)
