"""The no-allocation decode under HIP graph capture: the call is recorded into a graph (it launches
kernels and does nothing else: no allocation, no memory-set node, no host wait) and replayed several
times with eager work and synchronisations between the replays; every replay must reproduce the
eager result bit for bit, also after the query buffer has been refilled in place.
"""
import numpy as np
import pytest

import workloads
from helpers import GpuLayerCache

pytestmark = pytest.mark.gpu


def test_noalloc_decode_replays_from_a_graph():
    print("graph capture of cqa_certified_decode_noalloc: l8k shape, 4 replays, 3 queries", flush=True)
    sh = workloads.SHAPES["l8k"]
    n = 8192 - 11
    k, v = workloads.make_kv("l8k", seed=0, context=n)
    qs = [workloads.make_q("l8k", i, seed=0) for i in range(3)]
    with GpuLayerCache(sh.batch, sh.n_q_heads, sh.n_kv_heads, 8192 + 64) as gc:
        t, cqa = gc.torch, gc.cqa
        gc.append(k, v)
        tol = cqa.Tolerances()
        qd = gc.to_dev(qs[0]).clone()                 # the buffer the graph reads
        eager = []
        for q in qs:
            qd.copy_(gc.to_dev(q))
            cqa.cqa_certified_decode_noalloc(gc.h, 0, qd, tol, gc.O, gc.cert, gc.flags)
            eager.append(gc.results())
        s = t.cuda.Stream()
        g = t.cuda.CUDAGraph()
        qd.copy_(gc.to_dev(qs[0]))
        t.cuda.synchronize()
        with t.cuda.graph(g, stream=s):
            cqa.cqa_certified_decode_noalloc(gc.h, 0, qd, tol, gc.O, gc.cert, gc.flags, s.cuda_stream)
        for rep, qi in enumerate((0, 1, 2, 1)):
            qd.copy_(gc.to_dev(qs[qi]))
            gc.O.fill_(float("nan"))                  # eager work between the replays
            gc.cert.zero_()
            gc.flags.fill_(-1)
            t.cuda.synchronize()
            g.replay()
            t.cuda.synchronize()
            O, cert, flags = gc.results()
            O0, c0, f0 = eager[qi]
            assert np.array_equal(O, O0), ("replay", rep, "O")
            assert cert.tobytes() == c0.tobytes(), ("replay", rep, "cert")
            assert (flags == f0).all(), ("replay", rep, "flags")
            # an eager call of the ordinary entry point in between (it shares nothing with the graph's scratch)
            cqa.cqa_certified_decode(gc.h, 0, qd, tol, gc.O, gc.cert, gc.flags, None)
            assert np.array_equal(gc.results()[0], O0)


# Scales of keys and queries of successive prompts.  The decode pass brings q * sigma into FP16 range with a power
# of two taken from the running maximum of sigma: at the first scale q * sigma is far beyond 65504, at the second
# it lies among the FP16 subnormals, so a maximum of another prompt (or none) shows in the results.
SCALES = ((4000.0, 500.0), (0.01, 0.005), (6000.0, 900.0), (1.0, 1.0), (0.02, 0.01))


def _prompt(rng, bt, hkv, hq, n, scales):
    k = (rng.standard_normal((bt, hkv, n, 128)) * scales[0]).astype(np.float16)
    v = rng.standard_normal((bt, hkv, n, 128)).astype(np.float16)
    # queries nearly orthogonal to most keys: one channel each, so that logits stay moderate at every scale
    q = np.zeros((bt, hq, 128), dtype=np.float16)
    for h in range(hq):
        q[:, h, (7 * h) % 128] = scales[1] * (1.0 + h / 8.0)
    return k, v, q


@pytest.mark.parametrize("bt,hkv,g,n", [(1, 2, 4, 16 * 70 + 5), (2, 3, 2, 16 * 5 + 1), (1, 8, 4, 16 * 129)])
def test_a_recorded_decode_follows_resets_and_refills(bt, hkv, g, n):
    """Recorded once at one length, replayed on every later prompt of that length: the recorded launches hold
    addresses, so nothing they read may move when the cache is reset."""
    print("recorded decode over resets", bt, hkv, g, n, flush=True)
    rng = np.random.default_rng(n)
    hq = hkv * g
    with GpuLayerCache(bt, hq, hkv, n + 32) as gc:
        t, cqa = gc.torch, gc.cqa
        tol = cqa.Tolerances()
        prompts = [_prompt(rng, bt, hkv, hq, n, s) for s in SCALES]
        qd = gc.to_dev(prompts[0][2]).clone()
        calls = {"noalloc": lambda st: cqa.cqa_certified_decode_noalloc(gc.h, 0, qd, tol, gc.O, gc.cert, gc.flags, st),
                 "step": lambda st: cqa.cqa_decode_step_enqueue(gc.h, 0, None, None, qd, tol, gc.O, gc.cert, gc.flags, st)}
        gc.append(prompts[0][0], prompts[0][1])
        graphs = {}
        for name, call in calls.items():
            s, graphs[name] = t.cuda.Stream(), t.cuda.CUDAGraph()
            t.cuda.synchronize()
            with t.cuda.graph(graphs[name], stream=s):
                call(s.cuda_stream)
        for epoch, (k, v, q) in enumerate(prompts):
            if epoch > 0:
                cqa.cqa_cache_reset(gc.h, 0)
                gc.append(k, v)
            qd.copy_(gc.to_dev(q))
            for name, call in calls.items():
                call(None)
                O0, c0, f0 = [x.copy() for x in gc.results()]
                for rep in range(2):
                    gc.O.fill_(float("nan"))
                    gc.cert.zero_()
                    gc.flags.fill_(-1)
                    t.cuda.synchronize()
                    graphs[name].replay()
                    O, cert, flags = gc.results()
                    assert np.array_equal(O, O0), (name, epoch, rep)
                    assert cert.tobytes() == c0.tobytes() and (flags == f0).all(), (name, epoch, rep)


def test_a_recorded_prefill_and_decode_starts_afresh_after_a_reset():
    """Prompt and first decode recorded together on an empty cache; after a reset the replay sees another prompt in
    the same buffers and gives what a fresh cache gives."""
    print("recorded append and decode over resets", flush=True)
    bt, hkv, g, n = 1, 4, 2, 16 * 90 + 3
    hq = hkv * g
    rng = np.random.default_rng(5)
    prompts = [_prompt(rng, bt, hkv, hq, n, s) for s in SCALES]
    want = []
    for k, v, q in prompts:
        with GpuLayerCache(bt, hq, hkv, n + 32) as gc:
            gc.append(k, v)
            want.append([x.copy() for x in gc.certified_decode(q)])
    with GpuLayerCache(bt, hq, hkv, n + 32) as gc:
        t, cqa = gc.torch, gc.cqa
        kd, vd, qd = (gc.to_dev(x).clone() for x in prompts[0])
        s, graph = t.cuda.Stream(), t.cuda.CUDAGraph()
        t.cuda.synchronize()
        with t.cuda.graph(graph, stream=s):
            cqa.cqa_cache_append(gc.h, 0, kd, vd, n, s.cuda_stream)
            cqa.cqa_certified_decode_noalloc(gc.h, 0, qd, cqa.Tolerances(), gc.O, gc.cert, gc.flags, s.cuda_stream)
        for epoch, (prompt, ref) in enumerate(zip(prompts, want)):
            for dst, src in zip((kd, vd, qd), prompt):
                dst.copy_(gc.to_dev(src))
            gc.O.fill_(float("nan"))
            t.cuda.synchronize()
            if epoch > 0:
                cqa.cqa_cache_reset(gc.h, 0)
            graph.replay()
            for x, y in zip(gc.results(), ref):
                assert x.tobytes() == y.tobytes(), epoch
