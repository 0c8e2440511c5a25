"""Enqueue-only steps whose split pass reduces its partial sets itself: the last workgroup of a KV group to arrive finishes the
rows, or, where the group's workgroups are not on one die, the ladder's launch does.  Rows are those of the certified call, which
reduces in a launch of its own, bit for bit up to 64 sets."""
import numpy as np
import pytest

from helpers import GpuLayerCache

pytestmark = pytest.mark.gpu


def make(bt, hkv, g, n):
    rng = np.random.default_rng(n + 31 * bt + hkv)
    k = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    v = rng.standard_normal((bt, hkv, n, 128), dtype=np.float32).astype(np.float16)
    return k, v, rng.standard_normal((bt, hkv * g, 128)).astype(np.float16)


def step(gc, q, tol, kv=(None, None)):
    gc.O.fill_(float("nan"))
    gc.cqa.cqa_decode_step_enqueue(gc.h, 0, kv[0], kv[1], gc.to_dev(q), tol, gc.O, gc.cert, gc.flags)
    return [x.copy() for x in gc.results()]


# (batch, kv heads, group, tokens, sets): every form of the kernel that reduces (heads per group, waves, quads per wave) at every
# number of trips that it takes, first and last of what some take, groups that do not divide among the dies
SHAPES = [
    (1, 8, 4, 64 * 8 + 16, 3),        # four quad waves and four without, one quad in the last workgroup
    (1, 8, 4, 64 * 32 + 5, 8),        # ... the most sets of one trip
    (1, 8, 4, 64 * 32 + 17, 9),       # twelve waves, two trips
    (1, 4, 4, 64 * 64, 16),           # ... the most; nothing behind the sealed blocks
    (1, 1, 4, 64 * 64 + 16, 17),      # one set more: the reduction's launch
    (2, 4, 2, 64 * 96, 24),           # three trips of three rows of waves
    (1, 8, 1, 64 * 128 + 3, 32),      # four trips, the most that four quad waves keep
    (3, 1, 2, 64 * 20 + 9, 5),        # three KV groups, one to a die
    (11, 1, 4, 64 * 40 + 1, 10),      # eleven, two on some dies
    (11, 1, 1, 64 * 80 + 1, 20),      # ... with more workgroups there than compute units: the reduction's launch
    (4, 8, 4, 64 * 63 + 40, 8),       # eight quad waves, one quad each
    (16, 8, 4, 64 * 16 + 1, 2),       # ... two sets, a workgroup on every compute unit
    (1, 16, 1, 64 * 400 + 30, 16),    # ... several quads each, two trips
    (36, 8, 1, 16 * 96 + 5, 3),       # more KV groups than compute units
    (21, 8, 1, 16 * 129 + 5, 3), (21, 8, 2, 16 * 129, 3),   # fewer, two workgroups on most
    (9, 8, 4, 16 * 98 + 5, 7), (9, 8, 4, 16 * 98, 7), (19, 8, 4, 7000, 3),   # four quad waves with a wave per head and no more
    # what the rows of waves deal among themselves, form by form: four quad waves and no more, two heads and one
    (18, 8, 2, 16 * 33, 3), (17, 8, 2, 16 * 65 + 5, 3), (9, 8, 2, 3145, 7),
    (17, 8, 1, 16 * 33 + 3, 3), (7, 8, 1, 16 * 129, 9), (7, 8, 1, 16 * 257 + 7, 9), (3, 8, 1, 16 * 321 + 15, 21), (3, 8, 1, 16 * 642, 21),
    # ... four quad waves and four without
    (1, 1, 2, 16 * 129 + 2, 9), (1, 2, 1, 16 * 33 + 1, 3), (1, 3, 1, 16 * 129 + 5, 9), (5, 1, 1, 16 * 257 + 2, 17),
    # ... eight quad waves with a quad each
    (11, 8, 2, 16 * 33 + 8, 2), (13, 1, 2, 16 * 305 + 1, 10), (7, 1, 2, 16 * 577, 19),
    (11, 8, 1, 16 * 33 + 9, 2), (13, 1, 1, 16 * 305, 10), (7, 1, 1, 16 * 577 + 3, 19), (5, 1, 1, 16 * 817 + 11, 26),
    # ... with several
    (13, 8, 4, 16 * 130 + 10, 2), (13, 8, 4, 16 * 128 + 10, 2), (13, 8, 2, 16 * 65 + 1, 2), (3, 8, 2, 16 * 337 + 13, 10), (13, 8, 1, 16 * 65 + 4, 2), (1, 8, 1, 16 * 1027 + 6, 32),
]

# ... of these the reduction is a launch of its own
OWN_LAUNCH = [(1, 1, 4, 64 * 64 + 16, 17), (11, 1, 1, 64 * 80 + 1, 20), (36, 8, 1, 16 * 96 + 5, 3), (9, 8, 4, 16 * 98 + 5, 7), (9, 8, 4, 16 * 98, 7),
              (19, 8, 4, 7000, 3), (13, 8, 4, 16 * 128 + 10, 2)]


@pytest.mark.parametrize("int8", [False, True])
@pytest.mark.parametrize("bt,hkv,g,n,sets", SHAPES)
def test_rows_are_those_of_the_certified_call(bt, hkv, g, n, sets, int8):
    import torch
    print("split reduces", bt, hkv, g, n, int8, flush=True)
    k, v, q = make(bt, hkv, g, n)
    with GpuLayerCache(bt, hkv * g, hkv, n + 32) as gc:
        gc.append(k, v)
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert gc.cqa.cqa_decode_splits(gc.h, 0) == sets
        tol = gc.cqa.Tolerances(int8_query=int8)
        O, cert, flags = [x.copy() for x in gc.certified_decode(q, tol)]
        assert np.isfinite(O).all()
        for on in (0, 0, 1, 0):
            gc.cqa.cqa_set_scatter(gc.h, on)
            O2, cert2, flags2 = step(gc, q, tol)
            if torch.cuda.get_device_properties(0).multi_processor_count == 256:
                reduces = (bt, hkv, g, n, sets) not in OWN_LAUNCH
                assert gc.cqa.cqa_step_route(gc.h) == (0 if not reduces else 1 + on)
            assert (flags2 == flags).all()
            if on == 0 or sets <= 8:
                assert np.array_equal(O, O2) and cert.tobytes() == cert2.tobytes(), on
            else:
                # one wave merges eight sets after the other: another order of the same binary32 sums (8 trips of 2^-23)
                assert np.abs(O2 - O).max() <= 1e-5 * np.abs(O).max()
                for f in ("E_key", "E_val", "lse", "alpha_tail_hat"):
                    assert np.allclose(cert2[f], cert[f], rtol=1e-5, atol=1e-9), f
                assert (cert2["top_block"] == cert["top_block"]).all()


@pytest.mark.parametrize("scatter", [0, 1])
@pytest.mark.parametrize("bt,hkv,g,n", [(1, 8, 4, 64 * 20 + 7), (2, 4, 2, 64 * 30 + 11), (1, 8, 1, 64 * 30), (16, 8, 4, 64 * 12 + 3),
                                        (9, 8, 4, 16 * 98 + 5)])
def test_heads_over_a_threshold_are_served(bt, hkv, g, n, scatter):
    """Rung 3 for the heads that ask and no other, Rung 4 with a limit on the groups, the token of the step among the
    attended ones; on both routes, and a plain step behind each."""
    print("split reduces, served", bt, hkv, g, n, scatter, flush=True)
    k, v, q = make(bt, hkv, g, n + 1)
    with GpuLayerCache(bt, hkv * g, hkv, n + 32) as gc, GpuLayerCache(bt, hkv * g, hkv, n + 32) as other:
        gc.append(k[:, :, :n], v[:, :, :n])
        other.append(k, v)
        O, cert, _ = [x.copy() for x in other.certified_decode(q)]
        total = cert["E_key"] + cert["E_val"]
        order = np.sort(total.ravel())
        eps = float(np.float32(0.5 * (order[-3] + order[-2])))
        over = total > np.float32(eps)
        assert 0 < over.sum() < over.size
        cqa = gc.cqa
        cqa.cqa_set_scatter(gc.h, scatter)
        new = [gc.to_dev(np.ascontiguousarray(x[:, :, n:])) for x in (k, v)]
        O2, cert2, flags2 = step(gc, q, cqa.Tolerances(eps_total=eps), new)
        assert (cert2["served_rung"] == np.where(over, 3, 0)).all()
        assert (((flags2 & cqa.FLAG_TOTAL) != 0) == over).all()
        assert np.array_equal(O2[~over], O[~over])
        dense = step(other, q, cqa.Tolerances(force_flags=cqa.FLAG_TOTAL))[0]
        assert np.abs(O2 - dense)[over].max() <= 1e-5 * np.abs(dense).max()   # binary32 sums in another order
        O4, cert4, _ = step(gc, q, cqa.Tolerances(eps_total=eps, rung4_min_groups=1))
        assert (cert4["served_rung"] == 4).all() and np.abs(O4 - dense).max() <= 1e-5 * np.abs(dense).max()
        for on in (scatter, 0):
            cqa.cqa_set_scatter(gc.h, on)
            O5, cert5, flags5 = step(gc, q, cqa.Tolerances())
            assert np.array_equal(O5, O) and (cert5["served_rung"] == 0).all() and (flags5 == 0).all()


@pytest.mark.parametrize("bt,hkv,g,n", [(1, 8, 4, 64 * 20 + 7), (1, 8, 4, 64 * 40 + 7)])
def test_recorded_steps_find_their_counters_cleared(bt, hkv, g, n):
    """A recorded pair of steps, the first left to the ladder's launch, replayed with eager steps in between."""
    print("split reduces, recorded", bt, hkv, g, n, flush=True)
    k, v, q = make(bt, hkv, g, n)
    with GpuLayerCache(bt, hkv * g, hkv, n + 32) as gc:
        t, cqa = gc.torch, gc.cqa
        gc.append(k, v)
        tol = cqa.Tolerances()
        O, cert, _ = [x.copy() for x in gc.certified_decode(q)]
        qd, O1 = gc.to_dev(q).clone(), t.zeros_like(gc.O)
        s, graph = t.cuda.Stream(), t.cuda.CUDAGraph()
        t.cuda.synchronize()
        with t.cuda.graph(graph, stream=s):
            cqa.cqa_set_scatter(gc.h, 1)
            cqa.cqa_decode_step_enqueue(gc.h, 0, None, None, qd, tol, O1, gc.cert, gc.flags, s.cuda_stream)
            cqa.cqa_set_scatter(gc.h, 0)
            cqa.cqa_decode_step_enqueue(gc.h, 0, None, None, qd, tol, gc.O, gc.cert, gc.flags, s.cuda_stream)
        for _ in range(3):
            gc.O.fill_(float("nan"))
            O1.fill_(float("nan"))
            t.cuda.synchronize()
            graph.replay()
            t.cuda.synchronize()
            assert np.array_equal(gc.results()[0], O) and gc.results()[1].tobytes() == cert.tobytes()
            assert np.abs(O1.cpu().numpy() - O).max() <= 1e-5 * np.abs(O).max()
            cqa.cqa_set_scatter(gc.h, 0)     # (the first of the pair has told the host that steps stray)
            assert np.array_equal(step(gc, q, tol)[0], O) and cqa.cqa_step_route(gc.h) == 1


@pytest.mark.parametrize("bt,hkv,g,n", [(1, 8, 4, 64 * 20 + 7), (16, 8, 4, 64 * 12 + 3)])
def test_a_device_that_deals_otherwise_is_left_alone_after_its_first_step(bt, hkv, g, n):
    """The step whose KV groups were not together is reduced behind it, the host learns of it, and the steps that follow reduce in a
    launch of their own, served heads among them; a token rides on each."""
    print("split reduces, strays once", bt, hkv, g, n, flush=True)
    k, v, q = make(bt, hkv, g, n + 3)
    with GpuLayerCache(bt, hkv * g, hkv, n + 32) as gc, GpuLayerCache(bt, hkv * g, hkv, n + 32) as other:
        cqa = gc.cqa
        gc.append(k[:, :, :n], v[:, :, :n])
        other.append(k[:, :, :n], v[:, :, :n])
        cqa.cqa_set_scatter(gc.h, 2)
        for i, (route, force) in enumerate(((2, 0), (0, 0), (0, cqa.FLAG_TOTAL))):
            new = [np.ascontiguousarray(x[:, :, n + i:n + i + 1]) for x in (k, v)]
            other.append(*new)
            tol = cqa.Tolerances(force_flags=force)
            O, cert, flags = step(gc, q, tol, [gc.to_dev(x) for x in new])
            if gc.torch.cuda.get_device_properties(0).multi_processor_count == 256:
                assert cqa.cqa_step_route(gc.h) == route, i
            O2, cert2, flags2 = step(other, q, tol)
            assert np.array_equal(O, O2) and cert.tobytes() == cert2.tobytes() and (flags == flags2).all(), i
        cqa.cqa_set_scatter(gc.h, 0)
        step(gc, q, cqa.Tolerances())
        if gc.torch.cuda.get_device_properties(0).multi_processor_count == 256:
            assert cqa.cqa_step_route(gc.h) == 1


# (batch, kv heads, group, tokens, route of the first step): either side of each limit of the ladder's launch
FEW = [(1, 1, 4, 2048, 3), (1, 1, 4, 2049, 3), (1, 1, 4, 16 * 129, 1), (1, 2, 4, 1024, 3), (1, 2, 4, 1025, 1), (2, 1, 1, 16 * 36, 3), (1, 4, 1, 1009, 1),
       (1, 3, 2, 1008, 3), (5, 1, 1, 1504, 3), (1, 8, 1, 605, 1), (1, 9, 1, 1008, 1), (1, 1, 1, 16 * 33 + 1, 3)]


@pytest.mark.parametrize("bt,hkv,g,n,first", FEW)
def test_few_rows_are_reduced_by_the_ladders_launch(bt, hkv, g, n, first):
    """Up to eight rows and sets without trailing tokens or with one KV group, and with any after a step that has strayed: plain steps, steps with
    heads served by either rung, and a token that rides, against the calls that reduce in a launch of their own."""
    import torch
    print("few rows", bt, hkv, g, n, first, flush=True)
    k, v, q = make(bt, hkv, g, n + 1)
    with GpuLayerCache(bt, hkv * g, hkv, n + 32) as gc:
        cqa = gc.cqa
        gc.append(k[:, :, :n], v[:, :, :n])
        whole = torch.cuda.get_device_properties(0).multi_processor_count == 256
        few = gc.cqa.cqa_decode_splits(gc.h, 0) <= 8 and bt * hkv * g <= 8
        O, cert, flags = [x.copy() for x in gc.certified_decode(q)]
        total = np.sort((cert["E_key"] + cert["E_val"]).ravel())
        eps = float(np.float32(0.5 * (total[-1] + total[-2]))) if total.size > 1 else -1.0
        assert np.isfinite(O).all()
        for strays in (0, 2):
            cqa.cqa_set_scatter(gc.h, strays)
            for i in range(2):
                O2, cert2, flags2 = step(gc, q, cqa.Tolerances())
                if whole:
                    want = first if strays == 0 else (3 if few and (first == 3 or i == 1) else (0 if i == 1 else 2))
                    assert cqa.cqa_step_route(gc.h) == want, (strays, i)
                if few or cqa.cqa_step_route(gc.h) != 2:
                    assert np.array_equal(O, O2) and cert.tobytes() == cert2.tobytes() and (flags == flags2).all(), (strays, i)
            for tol, rung in ((cqa.Tolerances(eps_total=eps), 3), (cqa.Tolerances(eps_total=eps, rung4_min_groups=1), 4),
                              (cqa.Tolerances(force_flags=cqa.FLAG_TOTAL), 3)):
                O2, cert2, flags2 = step(gc, q, tol)
                _, O3, cert3, flags3 = gc.decode_step(q, tol)
                served = cert2["served_rung"] == rung
                assert served.any() and (flags2 == flags3).all() and cert2.tobytes() == cert3.tobytes()
                assert np.array_equal(O2[~served], O3[~served])
                assert np.abs(O2 - O3)[served].max() <= 1e-5 * np.abs(O3).max()     # binary32 sums in another order
        new = [gc.to_dev(np.ascontiguousarray(x[:, :, n:])) for x in (k, v)]
        O2, cert2, flags2 = step(gc, q, cqa.Tolerances(), new)
        if whole:
            assert cqa.cqa_step_route(gc.h) == (2 if first == 3 and bt * hkv > 1 else (3 if few else 0))    # the first one to stray, or not
        O, cert, flags = gc.certified_decode(q)
        assert np.array_equal(O, O2) and cert.tobytes() == cert2.tobytes()


@pytest.mark.parametrize("bt,hkv,n,recorded,eager", [(1, 8, 64 * 40, 0, 1), (1, 1, 4000, 0, 1), (1, 8, 64 * 40 + 1, 1, 1), (2, 8, 64 * 40, 0, 1), (1, 8, 64 * 32, 1, 1)])
def test_steps_of_many_sets_recorded_and_not(bt, hkv, n, recorded, eager):
    """Nine to sixteen sets, four heads, no trailing tokens: recorded with a launch for the reduction, without when called."""
    print("split reduces, recorded or not", bt, hkv, n, flush=True)
    k, v, q = make(bt, hkv, 4, n)
    with GpuLayerCache(bt, hkv * 4, hkv, n + 32) as gc:
        t, cqa = gc.torch, gc.cqa
        whole = t.cuda.get_device_properties(0).multi_processor_count == 256
        gc.append(k, v)
        tol = cqa.Tolerances()
        O, cert, _ = [x.copy() for x in gc.certified_decode(q)]
        qd = gc.to_dev(q).clone()
        s, graph = t.cuda.Stream(), t.cuda.CUDAGraph()
        t.cuda.synchronize()
        with t.cuda.graph(graph, stream=s):
            cqa.cqa_decode_step_enqueue(gc.h, 0, None, None, qd, tol, gc.O, gc.cert, gc.flags, s.cuda_stream)
        graph.replay()
        if whole:
            assert cqa.cqa_step_route(gc.h) == recorded
        for _ in range(3):
            gc.O.fill_(float("nan"))
            t.cuda.synchronize()
            graph.replay()
            assert np.array_equal(gc.results()[0], O) and gc.results()[1].tobytes() == cert.tobytes()
            assert np.array_equal(step(gc, q, tol)[0], O)
            if whole:
                assert cqa.cqa_step_route(gc.h) == eager
