"""The list of promoted blocks as the promoted-block pass makes it from the selection masks, against the list of a cache
whose FP16 scratch is in use (a launch of its own) and against the oracle's exploration draw, where the pieces of
a mask word change size, in the last, partial word, and where the list is full; and merges of many partial sets."""
import functools

import numpy as np
import pytest

import oracle
import workloads
from oracle import adaptive as ad
from helpers import GpuLayerCache, assert_head_matches
from test_gpu_adaptive import check_against_oracle, gpu_adaptive

pytestmark = pytest.mark.gpu


def run(gc, q, tol, sel):
    gc.cqa.cqa_adaptive_decode(gc.h, 0, gc.to_dev(q), tol, sel, gc.O, gc.cert, gc.flags)
    O, cert, flags = [x.copy() for x in gc.results()]
    st = gc.cqa.cqa_adaptive_state(gc.h, 0, gc.bt, gc.hq, gc.hkv)
    return O, cert, flags, st


# blocks: 8, 4, 2 or 1 pieces a word (up to 32, 64, 128 words), one and several sweeps of 256 words
@pytest.mark.parametrize("blocks", [1, 31, 33, 32 * 32, 32 * 33 + 1, 32 * 64 + 7, 32 * 129 + 3, 8192 + 40])
@pytest.mark.parametrize("hkv,g,per_head,values", [(2, 4, True, 24), (2, 2, False, 24), (1, 1, False, 0)])
def test_the_list_from_the_masks_is_the_list_of_the_scratch_path(blocks, hkv, g, per_head, values):
    n = blocks * 16 + 5
    rng = np.random.Generator(np.random.Philox(blocks))
    k, v = workloads.student_t3_f16(rng, (1, hkv, n, 128)), workloads.normal_f16(rng, (1, hkv, n, 128))
    qs = [workloads.normal_f16(rng, (1, hkv * g, 128)) for _ in range(2)]
    print("list", blocks, hkv, g, flush=True)
    got = []
    for slots in (0, 16):
        with GpuLayerCache(1, hkv * g, hkv, n + 16) as gc:
            gc.append(k, v)
            gc.cqa.cqa_set_scratch_slots(gc.h, min(slots, 1 << max(0, (blocks - 1).bit_length())))
            tol = gc.cqa.Tolerances(rank_depth=3, v_tol=0.02 if values else float("inf"))
            sel = gc.cqa.Selector(0.995, 2, 40, 48, v_limit=values, canary=True, explore_frac=0.03, explore_seed=5, per_head=per_head)
            got.append([run(gc, q, tol, sel) for q in qs])     # the second call takes the first one's list back
            if slots == 0 and blocks <= 32 * 33 + 1:
                oc = oracle.OracleLayerCache(1, hkv)
                oc.append(k, v)
                otol = oracle.Tolerances(rank_depth=3, v_tol=0.02 if values else float("inf"))
                osel = ad.SelectorParams(0.995, 2, 40, 48, values, False, True, 0.03, 5, per_head)
                check_against_oracle(oc, qs[0], otol, osel, gpu_adaptive(gc, qs[0], otol, osel))
    for a, b, q in zip(got[0], got[1], qs):
        assert np.array_equal(a[0], b[0]) and a[1].tobytes() == b[1].tobytes() and (a[2] == b[2]).all()
        for i in (0, 2, 3, 4, 8):                              # K*, flags, both log-masses, deviations
            assert np.array_equal(a[3][i], b[3][i]), i
        prom = a[3][2]
        par = ad.SelectorParams(explore_frac=0.03, explore_seed=5)
        for grp in range(hkv):
            drawn = np.asarray(ad.explored_blocks(blocks, grp, par), dtype=bool)
            assert (prom[0, grp, :blocks][drawn] & 1).all()


# the list full within the first part of 8192 blocks, within the second, and nowhere
@pytest.mark.parametrize("blocks,frac", [(4096, 1.0), (4200, 1.0), (9000, 1.0), (2 * 8192 + 33, 0.3), (2 * 8192 + 33, 0.01), (8192, 0.0), (8193, 0.0)])
@pytest.mark.parametrize("slots", [0, 16])
def test_a_full_list_leaves_the_last_blocks_in_int8(blocks, frac, slots):
    """Explored blocks beyond the 4096 that fit the list stay unpromoted and keep their INT8 mass, which is summed in parts
    of 8192 blocks."""
    n = blocks * 16
    rng = np.random.Generator(np.random.Philox(blocks))
    k, v = workloads.normal_f16(rng, (1, 1, n, 128)), workloads.normal_f16(rng, (1, 1, n, 128))
    q = workloads.normal_f16(rng, (1, 2, 128))
    print("full list", blocks, frac, slots, flush=True)
    with GpuLayerCache(1, 2, 1, n + 16) as gc:
        gc.append(k, v)
        gc.cqa.cqa_set_scratch_slots(gc.h, slots)
        sel = gc.cqa.Selector(0.995, 2, 16, 16, explore_frac=frac, explore_seed=1)
        O, cert, flags, st = run(gc, q, gc.cqa.Tolerances(), sel)
        keys = (st[2][0, 0, :blocks] & 1).astype(bool)
        wanted = np.asarray(ad.explored_blocks(blocks, 0, ad.SelectorParams(explore_frac=frac, explore_seed=1)), dtype=bool)
        last = np.flatnonzero(keys)[-1]
        assert keys.sum() <= 4096 and keys[:last + 1][wanted[:last + 1]].all()
        if wanted.sum() >= 4096:
            assert keys.sum() == 4096
        else:
            assert keys[wanted].all()
        s8, _, _, lm = gc.certified_decode(q, want_logmass=True)
        kd, vd, qd = k[0, 0].astype(np.float64), v[0, 0].astype(np.float64), q[0].astype(np.float64)
        for h in range(2):
            # the mass left in INT8, from the first pass's log-masses (binary32 exponentials: 1e-5)
            l8 = lm[0, h, :blocks].astype(np.float64)
            tail = np.exp(l8[~keys] - np.logaddexp.reduce(l8)).sum()
            assert abs(cert[0, h]["alpha_tail_hat"] - tail) <= 1e-5 * tail + 1e-12
            # the best block left, against the best promoted one
            if not keys.all():
                lx = st[4][0, h, :blocks][keys].max()
                assert abs(cert[0, h]["rank_margin"] - (lx - (l8[~keys].max() + cert[0, h]["delta_h"]))) <= 1e-4
            # listed blocks with FP16 scores, all others with the first pass's log-masses
            s = kd @ qd[h] / np.sqrt(128.0)
            m = s.max()
            l16 = np.log(np.exp(s - m).reshape(blocks, 16).sum(1)) + m
            assert abs(cert[0, h]["lse"] - np.logaddexp.reduce(np.where(keys, l16, l8))) <= 1e-4


# (batch, kv heads, group, blocks): up to one workgroup per compute unit, somewhat more, two and more (sums by a wave each and
# by a workgroup each), sums in one part and in two, short lists, which reach few of a group's workgroups
# (sums last there, too, with the FP16 scratch in use)
@pytest.mark.parametrize("bt,hkv,g,blocks,slots", [
    (1, 7, 2, 300, 0), (1, 8, 4, 300, 0), (1, 8, 4, 300, 16), (2, 5, 4, 130, 0), (1, 8, 2, 8200, 0), (1, 12, 4, 90, 0), (2, 10, 4, 65, 0),
    (4, 8, 4, 3, 0), (4, 8, 4, 13, 0), (5, 7, 2, 28, 0), (4, 9, 1, 29, 0), (1, 9, 1, 25, 0), (4, 9, 2, 513, 0), (4, 9, 2, 40, 16),
    (2, 8, 4, 2048, 0), (2, 8, 4, 2049, 0)])
def test_rows_do_not_depend_on_the_order_of_the_workgroups(bt, hkv, g, blocks, slots):
    """Every KV group's rows are bit for bit those of a cache of its own, whose workgroups all lie one after another."""
    n = blocks * 16 + 3
    rng = np.random.Generator(np.random.Philox(blocks * 100 + hkv))
    k, v = workloads.student_t3_f16(rng, (bt, hkv, n, 128)), workloads.normal_f16(rng, (bt, hkv, n, 128))
    q = workloads.normal_f16(rng, (bt, hkv * g, 128))
    print("order", bt, hkv, g, blocks, slots, flush=True)
    for b, h in [(slice(None), slice(None))] + [(i, j) for i in range(bt) for j in range(hkv)][::3]:
        whole = isinstance(b, slice)
        kk, vv, qq = (k, v, q) if whole else (k[b:b + 1, h:h + 1], v[b:b + 1, h:h + 1], q[b:b + 1, h * g:(h + 1) * g])
        with GpuLayerCache(kk.shape[0], kk.shape[1] * g, kk.shape[1], n + 16) as gc:
            gc.append(kk, vv)
            gc.cqa.cqa_set_splits(gc.h, 2)
            gc.cqa.cqa_set_scratch_slots(gc.h, slots)
            tol = gc.cqa.Tolerances(rank_depth=2, v_tol=0.02)
            O, cert, flags, st = run(gc, qq, tol, gc.cqa.Selector(0.995, 2, 40, 40, v_limit=16, canary=True))
        if whole:
            all_O, all_cert, all_flags, all_st = O, cert, flags, st
            continue
        rows = slice(h * g, (h + 1) * g)
        assert np.array_equal(all_O[b, rows], O[0]) and all_cert[b, rows].tobytes() == cert[0].tobytes()
        assert (all_flags[b, rows] == flags[0]).all() and np.array_equal(all_st[2][b, h], st[2][0, 0])


@pytest.mark.parametrize("blocks,where", [(40, 39), (300, 17), (1500, 1400), (11000, 10)])
@pytest.mark.parametrize("value", [np.inf, -np.inf])
def test_a_block_without_a_log_mass_takes_no_place_from_one_that_has(blocks, where, value):
    """One infinite key: its block has no log-mass, is last in the ranking, and with it no prefix of the ranking covers
    anything, so every head selects its K_max best other blocks."""
    n = blocks * 16 + 5
    rng = np.random.default_rng(blocks)
    k, v = (rng.standard_normal((1, 2, n, 128), dtype=np.float32).astype(np.float16) for _ in range(2))
    q = rng.standard_normal((1, 8, 128)).astype(np.float16)
    k[0, 0, where * 16 + 3, 7] = value
    print("no log-mass", blocks, where, value, flush=True)
    with GpuLayerCache(1, 8, 2, n + 16) as gc:
        gc.append(k, v)
        _, _, _, st = run(gc, q, gc.cqa.Tolerances(), gc.cqa.Selector(0.995, 2, 16, 16))
        for h in range(4):
            l8 = st[3][0, h]
            assert np.flatnonzero(~np.isfinite(l8)).tolist() == [where] and st[0][0, h] == 16
            best = np.argsort(-np.where(np.isfinite(l8), l8, -np.inf), kind="stable")[:16]
            assert st[1][0, h, :16].tolist() == best.tolist(), h


@functools.lru_cache(maxsize=1)
def long_head():
    """One KV head of 128K tokens with 4 query heads: 2048 quads, 256 sets of eight waves."""
    rng = np.random.default_rng(256)
    k, v = (rng.standard_normal((1, 1, 131072 + 7, 128), dtype=np.float32).astype(np.float16) for _ in range(2))
    q = rng.standard_normal((1, 4, 128)).astype(np.float16)
    oc = oracle.OracleLayerCache(1, 1)
    oc.append(k, v)
    return k, v, q, oc, oc.certified_decode(q, oracle.Tolerances())


@pytest.mark.parametrize("splits", [1, 8, 9, 17, 64, 65, 130, 200, None])
def test_merging_any_number_of_partial_sets(splits):
    """A wave merges eight sets a trip, eight waves share a head's sets: up to 64 in one trip, more in several.  None: as
    many as the launch rule gives, 256 on 256 compute units."""
    k, v, q, oc, ref = long_head()
    print("sets", splits, flush=True)
    with GpuLayerCache(1, 4, 1, k.shape[2] + 16) as gc:
        gc.append(k, v)
        if splits is not None:
            gc.cqa.cqa_set_splits(gc.h, splits)
            assert gc.cqa.cqa_decode_splits(gc.h, 0) == splits
        elif gc.torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert gc.cqa.cqa_decode_splits(gc.h, 0) == 256
        O, cert, flags = gc.certified_decode(q)
        for h, r in enumerate(ref):
            assert_head_matches(r, O[0, h], cert[0, h], flags[0, h], (splits, h))
        # the selector reduces the same sets, and the adaptive reduction merges 32 more
        tol, sel = oracle.Tolerances(), ad.SelectorParams(0.995, 2, 16, 16)
        check_against_oracle(oc, q, tol, sel, gpu_adaptive(gc, q, tol, sel))
