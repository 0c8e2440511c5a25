"""The seal launch at its edges: codes at ties and extremes bit-exact, appends that start, end and lie inside a
block, and a cache that is reused after a reset (records hold the previous sequence beyond the last block)."""
import numpy as np
import pytest

import oracle
from helpers import GpuLayerCache

pytestmark = pytest.mark.gpu


def _special(rng, shape):
    """Values whose quotients sit on or next to half-integers, constant and tiny ranges, the largest FP16 numbers."""
    x = rng.standard_normal(shape).astype(np.float16)
    n = shape[2]
    x[:, :, :, 0] = np.float16(0.75)                                        # constant channel
    x[:, :, :, 1] = (rng.integers(0, 511, shape[:3]) / np.float16(2)).astype(np.float16)       # ties when the range is 255
    x[:, :, :, 2] = rng.choice([0.0, 255.0, 0.5, 1.5, 2.5, 127.5, 128.5], shape[:3]).astype(np.float16)
    x[:, :, :, 3] = rng.choice([-65504.0, 65504.0, 0.0, 1.0], shape[:3]).astype(np.float16)
    x[:, :, :, 4] = (rng.integers(0, 8, shape[:3]) * 2.0 ** -24).astype(np.float16)            # subnormal range
    x[:, :, :, 5] = (1000.0 + rng.integers(0, 2, shape[:3]) * 0.5).astype(np.float16)
    # values: a group of 16 channels with range exactly 15 and halves (ties), one constant, one subnormal
    x[:, :, :, 16:32] = (rng.integers(0, 31, shape[:3] + (16,)) / 2).astype(np.float16)
    x[:, :, :, 16], x[:, :, :, 17] = np.float16(0), np.float16(15)
    x[:, :, :, 32:48] = np.float16(-3.25)
    x[:, :, :, 48:64] = (rng.integers(0, 30, shape[:3] + (16,)) * 2.0 ** -24).astype(np.float16)
    x[:, :, n // 2:, 64:80] *= np.float16(100)
    return x


def _check(gc, oc, where, some=None):
    for b in range(gc.bt):
        for h in range(gc.hkv):
            nb = gc.length() // 16
            for blk in (range(nb) if some is None else sorted({0, 1, nb - 2, nb - 1, *some.integers(0, nb, 12).tolist()})):
                kc, sg, z, vc, vs, vo, eta, nu = gc.export(b, h, blk)
                assert np.array_equal(kc, oc.k_codes[b, h][blk]), (where, b, h, blk)
                assert np.array_equal(sg, oc.sigma[b, h][blk]) and np.array_equal(z, oc.z[b, h][blk]), (where, blk)
                assert np.array_equal(vc, oc.v_codes[b, h][blk]), (where, b, h, blk)
                assert np.array_equal(vs, oc.v_scale[b, h][blk]) and np.array_equal(vo, oc.v_offset[b, h][blk]), (where, blk)
                assert abs(eta - oc.eta[b, h][blk]) <= 1e-6 * abs(oc.eta[b, h][blk])
                assert abs(nu - oc.nu[b, h][blk]) <= 1e-6 * abs(oc.nu[b, h][blk])


@pytest.mark.parametrize("pieces", [[16 * 9], [5, 11 + 16 * 3, 7], [15, 2, 14 + 16, 1, 16, 17, 16], [3, 4, 5, 4, 32, 9]])
def test_codes_bit_exact_at_ties_extremes_and_block_edges(pieces):
    print("seal", pieces, flush=True)
    rng = np.random.default_rng(sum(pieces))
    n = sum(pieces)
    k, v = _special(rng, (2, 3, n, 128)), _special(rng, (2, 3, n, 128))
    oc = oracle.OracleLayerCache(2, 3)
    with GpuLayerCache(2, 6, 3, n + 16) as gc:
        at = 0
        for p in pieces:
            gc.append(k[:, :, at:at + p], v[:, :, at:at + p])
            oc.append(k[:, :, at:at + p], v[:, :, at:at + p])
            at += p
            _check(gc, oc, (pieces, at))


def test_runs_of_blocks_after_waiting_tokens():
    """4 x 8 sequences of 151 blocks: every workgroup seals a run of two, the first one starting in the trailing block."""
    print("seal runs", flush=True)
    rng = np.random.default_rng(3)
    n = 9 + 16 * 150 + 12
    k, v = _special(rng, (4, 8, n, 128)), _special(rng, (4, 8, n, 128))
    oc = oracle.OracleLayerCache(4, 8)
    with GpuLayerCache(4, 8, 8, n + 16) as gc:
        for a, b in ((0, 9), (9, n)):
            gc.append(k[:, :, a:b], v[:, :, a:b])
            oc.append(k[:, :, a:b], v[:, :, a:b])
        _check(gc, oc, "runs", rng)


@pytest.mark.parametrize("first,second", [(16 * 11 + 3, 16 * 5 + 9), (16 * 4, 16 * 1 + 2), (16 * 9, 5), (40, 16 * 6 + 1)])
@pytest.mark.parametrize("int8_query", [0, 1])
def test_a_reset_cache_equals_a_fresh_one(first, second, int8_query):
    print("reset", first, second, int8_query, flush=True)
    rng = np.random.default_rng(first * 7 + second)
    kv = [(rng.standard_normal((2, 2, n, 128)) * s).astype(np.float16) for n, s in ((first, 30.0), (first, 30.0), (second, 1.0), (second, 1.0))]
    step = [(rng.standard_normal((6, 2, 2, 1, 128))).astype(np.float16) for _ in range(2)]
    q = rng.standard_normal((2, 8, 128)).astype(np.float16)

    def fill(gc):
        out = []
        gc.append(kv[2], kv[3])
        tol = gc.cqa.Tolerances(int8_query=int8_query)
        for i in range(6):
            out.append([x.copy() for x in gc.certified_decode(q, tol)])
            gc.append(step[0][i], step[1][i])
        rung, O, cert, flags = gc.decode_step(q, gc.cqa.Tolerances(force_flags=gc.cqa.FLAG_TOTAL))
        assert rung == 3
        out.append([O.copy(), cert.copy(), flags.copy()])
        # every head served from the stored originals: the dense result over the tokens themselves
        kk = np.concatenate([kv[2], *step[0]], axis=2)
        vv = np.concatenate([kv[3], *step[1]], axis=2)
        for b in range(2):
            for h in range(8):
                dense = oracle.softmax_attention(q[b, h], kk[b, h // 4], vv[b, h // 4])
                assert np.linalg.norm(O[b, h] - dense) <= 1e-3 * np.linalg.norm(dense) + 1e-6, (b, h)
        return out

    with GpuLayerCache(2, 8, 2, 512) as fresh:
        want = fill(fresh)
    with GpuLayerCache(2, 8, 2, 512) as gc:
        for rounds in range(3):
            kx, vx = kv[0].copy(), kv[1].copy()
            if rounds == 1:
                kx[..., 7], vx[..., 40] = np.inf, np.nan        # what is left behind is not even finite
            gc.append(kx, vx)
            gc.certified_decode(q)
            gc.cqa.cqa_cache_reset(gc.h, 0)
            if rounds == 2:                         # an empty epoch, and one without a sealed block
                gc.cqa.cqa_cache_reset(gc.h, 0)
                gc.append(kv[0][:, :, :7], kv[1][:, :, :7])
                gc.cqa.cqa_cache_reset(gc.h, 0)
            got = fill(gc)
            for a, b in zip(got, want):
                for x, y in zip(a, b):
                    assert np.array_equal(x, y), (rounds, x.dtype)
            gc.cqa.cqa_cache_reset(gc.h, 0)


@pytest.mark.parametrize("bt,hkv,pieces", [
    (40, 32, [5, 16 * 3 + 4, 16]),      # more heads than workgroups: one each takes all blocks, the waiting tokens' among them
    (16, 16, [16 * 9 + 3, 16 * 7]),     # four workgroups of a head: two or three blocks each, the last block with the first one
    (8, 16, [7, 16 * 8 + 10]),          # eight: one block each, a record left half empty
    (65, 8, [16 * 11 + 5, 16 * 41]),    # two workgroups a head would fill five of a compute unit's six places: runs of two, then of eight blocks
    (35, 32, [3, 16 * 19 + 6]),         # one a head, unevenly: runs of eight, a record left half empty
])
def test_blocks_dealt_round_the_workgroups(bt, hkv, pieces):
    print("seal dealt", bt, hkv, pieces, flush=True)
    rng = np.random.default_rng(bt)
    n = sum(pieces)
    k, v = _special(rng, (bt, hkv, n, 128)), _special(rng, (bt, hkv, n, 128))
    oc = oracle.OracleLayerCache(bt, hkv)
    with GpuLayerCache(bt, hkv, hkv, n + 16) as gc:
        at = 0
        for p in pieces:
            gc.append(k[:, :, at:at + p], v[:, :, at:at + p])
            oc.append(k[:, :, at:at + p], v[:, :, at:at + p])
            at += p
        _check(gc, oc, pieces)
