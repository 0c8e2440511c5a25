"""The split pass's launch geometry where its rule changes: one generation of eight-wave workgroups, four-wave
workgroups that divide better, and several splits with more sequences than compute units."""
import numpy as np
import pytest

import oracle
from helpers import GpuLayerCache, assert_head_matches

pytestmark = pytest.mark.gpu


# (batch, kv heads, group, tokens, splits the rule gives on 256 compute units)
@pytest.mark.parametrize("bt,hkv,g,n,splits", [
    (3, 16, 2, 16 * 160 + 3, 5),      # 48 sequences: floor(256 / 48), not 6
    (1, 2, 4, 16 * 60 + 4, 4),        # 2: a quad per four-wave workgroup's wave, each wave with a SIMD to itself
    (13, 10, 1, 16 * 40 + 1, 3),      # 130: three four-wave workgroups each instead of one of eight waves
    (25, 8, 1, 16 * 30, 1),           # 200: both forms take as many rounds
    (36, 8, 1, 16 * 96 + 5, 3),       # 288: one split would leave the second half of the chip idle
    (32, 16, 1, 16 * 9, 1),           # 512: exactly one generation
    (70, 8, 2, 16 * 64 + 2, 2),       # 560: two generations, the second of 48 workgroups, cost more than three of half the rounds
])
def test_results_do_not_depend_on_the_launch_geometry(bt, hkv, g, n, splits):
    import torch
    print("geometry", bt, hkv, g, n, flush=True)
    rng = np.random.default_rng(n + bt)
    k = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    v = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    q = rng.standard_normal((bt, hkv * g, 128)).astype(np.float16)
    rows = [0, bt // 2, bt - 1]
    oc = oracle.OracleLayerCache(len(rows), hkv)
    oc.append(k[rows], v[rows])
    ref = oc.certified_decode(q[rows], oracle.Tolerances())
    with GpuLayerCache(bt, hkv * g, hkv, n + 16, tier2=False) as gc:
        gc.append(k, v)
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert gc.cqa.cqa_decode_splits(gc.h, 0) == splits
        O, cert, flags, lm = gc.certified_decode(q, want_logmass=True)
        for (i, h), r in zip([(i, h) for i in range(len(rows)) for h in range(hkv * g)], ref):
            assert_head_matches(r, O[rows[i], h], cert[rows[i], h], flags[rows[i], h], (bt, hkv, g, rows[i], h))
            assert np.abs(lm[rows[i], h] - r["blk_logmass"]).max() <= 1e-4
        # the other sequences against one more geometry: a different split moves O only by the rounding of its
        # weights against another running maximum (2^-17 per weight, the bound of the split-invariance test)
        gc.cqa.cqa_set_splits(gc.h, splits + 1)
        O2, cert2, _ = gc.certified_decode(q)
        assert np.abs(O2 - O).max() <= 1e-4 * np.abs(O).max()
        assert np.allclose(cert2["lse"], cert["lse"], rtol=5e-6, atol=0)


@pytest.mark.parametrize("bt,hkv,g,n", [(2, 8, 4, 125), (17, 1, 4, 125), (9, 2, 4, 70), (40, 8, 4, 333), (40, 8, 2, 125), (33, 8, 1, 200)])
def test_steps_of_one_split_give_the_same_rows_on_both_routes(bt, hkv, g, n):
    """A sequence of one workgroup is finished by the split pass, with or without a mirror of its flags: the host-resolved step
    and the plain call bit for bit, few rows and many."""
    print("one split", bt, hkv, g, n, flush=True)
    rng = np.random.default_rng(n + bt)
    k = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    v = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    q = rng.standard_normal((bt, hkv * g, 128)).astype(np.float16)
    oc = oracle.OracleLayerCache(1, hkv)
    oc.append(k[-1:], v[-1:])
    ref = oc.certified_decode(q[-1:], oracle.Tolerances())
    with GpuLayerCache(bt, hkv * g, hkv, n + 16) as gc:
        gc.append(k, v)
        assert gc.cqa.cqa_decode_splits(gc.h, 0) == 1
        O, cert, flags = [x.copy() for x in gc.certified_decode(q)]
        for h, r in enumerate(ref):
            assert_head_matches(r, O[-1, h], cert[-1, h], flags[-1, h], (bt, hkv, g, h))
        for _ in range(2):
            gc.O.fill_(float("nan"))
            rung, O2, cert2, flags2 = gc.decode_step(q)
            assert rung == 0
            assert np.array_equal(O, O2) and cert.tobytes() == cert2.tobytes() and (flags == flags2).all()


@pytest.mark.parametrize("bt,hkv,g,n", [(1, 1, 4, 125), (9, 2, 1, 125), (9, 2, 2, 125), (9, 2, 4, 125), (17, 1, 4, 70), (70, 8, 2, 64 * 16 + 2)])
def test_a_host_resolved_step_serves_the_heads_that_ask(bt, hkv, g, n):
    """The host reads every head's own flag word: a threshold between the heads' bounds, the rows over it are served and no other."""
    print("mirror", bt, hkv, g, n, flush=True)
    rng = np.random.default_rng(n + bt + g)
    k = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    v = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    q = rng.standard_normal((bt, hkv * g, 128)).astype(np.float16)
    with GpuLayerCache(bt, hkv * g, hkv, n + 16) as gc:
        gc.append(k, v)
        O, cert, _ = [x.copy() for x in gc.certified_decode(q)]
        total = cert["E_key"] + cert["E_val"]
        order = np.sort(total.ravel())
        for i in (len(order) // 3, len(order) - 2):
            eps = float(np.float32(0.5 * (order[i] + order[i + 1])))
            over = total > np.float32(eps)
            rung, O2, cert2, flags2 = gc.decode_step(q, gc.cqa.Tolerances(eps_total=eps))
            assert rung == 3 and 0 < over.sum() < over.size
            assert ((flags2 & gc.cqa.FLAG_TOTAL) != 0).tolist() == over.tolist()
            assert (cert2["served_rung"] == np.where(over, 3, 0)).all()
            assert np.array_equal(O2[~over], O[~over]) and np.isfinite(O2).all()


@pytest.mark.parametrize("bt,hkv,g,n", [(70, 8, 2, 64 * 16 + 2), (70, 8, 4, 64 * 16), (72, 8, 2, 64 * 24 + 5)])
def test_many_rows_of_several_splits_give_the_same_rows_on_both_routes(bt, hkv, g, n):
    """More than 1024 rows are reduced by one wave each where their flags are mirrored to the host and by several waves
    otherwise: bit for bit the same, with and without trailing tokens."""
    print("several splits", bt, hkv, g, n, flush=True)
    rng = np.random.default_rng(n + bt)
    k = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    v = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    q = rng.standard_normal((bt, hkv * g, 128)).astype(np.float16)
    oc = oracle.OracleLayerCache(1, hkv)
    oc.append(k[-1:], v[-1:])
    ref = oc.certified_decode(q[-1:], oracle.Tolerances())
    with GpuLayerCache(bt, hkv * g, hkv, n + 16, tier2=False) as gc:
        gc.append(k, v)
        assert 2 <= gc.cqa.cqa_decode_splits(gc.h, 0) <= 8
        O, cert, flags = [x.copy() for x in gc.certified_decode(q)]
        for h, r in enumerate(ref):
            assert_head_matches(r, O[-1, h], cert[-1, h], flags[-1, h], (bt, hkv, g, h))
        for _ in range(2):
            gc.O.fill_(float("nan"))
            rung, O2, cert2, flags2 = gc.decode_step(q)
            assert rung == 0
            assert np.array_equal(O, O2) and cert.tobytes() == cert2.tobytes() and (flags == flags2).all()


@pytest.mark.parametrize("int8", [False, True])
@pytest.mark.parametrize("bt,hkv,g,n,splits", [
    (1, 8, 4, 64 * 32 - 5, 8),        # every wave exactly one quad, the last one short of a block
    (1, 8, 2, 64 * 32 + 16, 9),       # ... and a ninth workgroup with a single quad of one block
    (2, 4, 1, 64 * 9 + 40, 3),        # two waves of the last workgroup without one
    (1, 1, 4, 64 * 130, 33),          # more sets than one trip of four merging waves holds
    (1, 1, 2, 64 * 512, 128),         # the most sets of four-wave workgroups ...
    (1, 1, 2, 64 * 512 + 3 * 16, 65), # ... one quad more: eight waves
    (8, 8, 4, 64 * 5 + 20, 1),        # eight waves, finished by the pass itself
])
def test_contexts_of_one_quad_per_wave(bt, hkv, g, n, splits, int8):
    """Short contexts, where no wave of the split pass takes a second quad, in both scoring modes."""
    import torch
    print("one quad", bt, hkv, g, n, int8, flush=True)
    rng = np.random.default_rng(n + bt)
    k = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    v = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    q = rng.standard_normal((bt, hkv * g, 128)).astype(np.float16)
    oc = oracle.OracleLayerCache(bt, hkv)
    oc.append(k, v)
    ref = oc.certified_decode(q, oracle.Tolerances(int8_query=int8))
    with GpuLayerCache(bt, hkv * g, hkv, n + 16, tier2=False) as gc:
        gc.append(k, v)
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert gc.cqa.cqa_decode_splits(gc.h, 0) == splits
        O, cert, flags, lm = gc.certified_decode(q, gc.cqa.Tolerances(int8_query=int8), want_logmass=True)
        for i, r in enumerate(ref):
            at = divmod(i, hkv * g)
            assert_head_matches(r, O[at], cert[at], flags[at], (bt, hkv, g, at, int8))
            assert np.abs(lm[at] - r["blk_logmass"]).max() <= 1e-4
