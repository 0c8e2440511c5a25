"""Dense FP16 attention on the GPU at the edges of its launch geometry: a single token, tiles that are not
full, one split per group (no reduction), more groups than compute units, and the workspace's exact size."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,hq,hkv,n", [
    (1, 1, 1, 1), (1, 4, 1, 31), (2, 4, 2, 33), (1, 8, 8, 129), (1, 4, 1, 257), (3, 8, 2, 511),
    (1, 32, 8, 4097), (1, 2, 1, 20011), (40, 16, 8, 300), (1, 4, 1, 131072 + 200),
])
def test_dense_attention_at_the_edges_of_its_geometry(batch, hq, hkv, n):
    import torch

    from paper_2605_20868_amd import binding as cqa
    print("dense", batch, hq, hkv, n, flush=True)
    rng = np.random.default_rng(n)
    q = rng.standard_normal((batch, hq, 128)).astype(np.float16)
    k = rng.standard_normal((batch, hkv, n, 128)).astype(np.float16)
    v = rng.standard_normal((batch, hkv, n, 128)).astype(np.float16)
    need = cqa.cqa_dense_workspace_bytes(batch, hq, n)
    ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    O = torch.full((batch, hq, 128), float("nan"), dtype=torch.float32, device="cuda")
    dev = [torch.from_numpy(x).to("cuda") for x in (q, k, v)]
    cqa.cqa_dense_attention(*dev, batch, hq, hkv, n, O, ws)
    torch.cuda.synchronize()
    assert (ws[need:] == 0x5A).all()                     # nothing past the size the library asked for
    got = O.cpu().numpy().astype(np.float64)
    g = hq // hkv
    some = [(0, 0), (batch - 1, hq - 1), (batch // 2, hq // 2)]
    for b, h in some:
        ref = oracle.softmax_attention(q[b, h], k[b, h // g], v[b, h // g])
        # FP32 products and sums: a score is off by at most 128 * 2^-24 * sum|q k| / sqrt(d) ~ 1e-4 in the worst case and
        # ~1e-6 in practice, and a weight by the same factor; 1e-5 of the largest value that is averaged
        assert np.abs(got[b, h] - ref).max() <= 1e-5 * np.abs(v[b, h // g].astype(np.float64)).max()
    assert np.isfinite(got).all()


# (batch, kv heads, group, tokens): layers of so many KV groups that the dense call has one or a few workgroups per group,
# with a last split or last rounds of a wave that are short, and sizes on both sides of the single-wave rule
@pytest.mark.parametrize("bt,hkv,g,n", [(17, 8, 4, 1350), (9, 8, 4, 7003), (33, 8, 1, 2100), (3, 7, 2, 5000), (5, 8, 1, 20000), (6, 8, 2, 9000),
                                        (1, 8, 4, 3000), (9, 1, 4, 3090), (20, 8, 2, 880), (1, 16, 4, 33000)])
def test_fallback_rows_equal_the_dense_call_in_large_layers(bt, hkv, g, n):
    """The fallback attends one KV group at a time, by single waves where the dense call gives a group few workgroups, and
    merges them in the same order."""
    import torch

    from helpers import GpuLayerCache
    print("fallback", bt, hkv, g, n, flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    k, v = (torch.randn((bt, hkv, n, 128), generator=gen, device="cuda", dtype=torch.float32).half() for _ in range(2))
    q = torch.randn((bt, hkv * g, 128), generator=gen, device="cuda", dtype=torch.float32).half()
    with GpuLayerCache(bt, hkv * g, hkv, n + 16) as gc:
        cqa = gc.cqa
        gc.append(k, v)
        need = cqa.cqa_dense_workspace_bytes(bt, hkv * g, n)
        ws = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        dense = torch.empty((bt, hkv * g, 128), dtype=torch.float32, device="cuda")
        cqa.cqa_dense_attention(q, k, v, bt, hkv * g, hkv, n, dense, ws)
        gc.O.fill_(float("nan"))
        cqa.cqa_dense_fallback(gc.h, 0, q, None, 1, 4, gc.O)
        torch.cuda.synchronize()
        assert (ws[need:] == 0x5A).all()
        assert torch.equal(gc.O, dense)
        sel = np.zeros((bt, hkv * g), dtype=np.uint32)
        sel[bt - 1, 1] = sel[bt // 2, hkv * g - 1] = 1
        gc.O.fill_(7.0)
        cqa.cqa_dense_fallback(gc.h, 0, q, sel, 0, 3, gc.O)
        torch.cuda.synchronize()
        on = torch.from_numpy(sel != 0)
        assert torch.equal(gc.O.cpu()[on], dense.cpu()[on]) and (gc.O.cpu()[~on] == 7.0).all()
        for b, h in ((0, 0), (bt - 1, hkv * g - 1)):
            kk, vv = k[b, h // g].cpu().numpy(), v[b, h // g].cpu().numpy()
            ref = oracle.softmax_attention(q[b, h].cpu().numpy(), kk, vv)
            # as above: 1e-5 of the largest value that is averaged
            assert np.abs(dense[b, h].cpu().numpy().astype(np.float64) - ref).max() <= 1e-5 * np.abs(vv.astype(np.float64)).max()


def test_a_paged_group_of_a_large_layer_takes_no_longer_than_one_of_a_small_layer():
    """One head of one KV group falls back, in a layer of 8 groups and in one of 136: the same bytes of the same pinned
    arrays over the host link, and the same attention.  372 and 470 us; 814 us for the large layer with the dense
    call's one workgroup per group."""
    import time

    import torch

    from helpers import load_binding
    print("fallback time", flush=True)
    cqa = load_binding()
    n, most, took = 32768, 17, []
    t2 = [torch.empty(most * 8 * n * 128, dtype=torch.float16, pin_memory=True) for _ in range(2)]
    for bt in (1, most):
        h = cqa.cqa_cache_create_caller_tier2(1, bt, 32, 8, n, t2[0], t2[1], t2[0].numel() * 2)
        try:
            k = torch.randn((bt, 8, n, 128), device="cuda", dtype=torch.float16)
            q = torch.randn((bt, 32, 128), device="cuda", dtype=torch.float16)
            O = torch.empty((bt, 32, 128), device="cuda", dtype=torch.float32)
            cqa.cqa_cache_append(h, 0, k, k, n)
            sel = np.zeros((bt, 32), dtype=np.uint32)
            sel[0, 5] = 1
            times = []
            for _ in range(12):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                cqa.cqa_dense_fallback(h, 0, q, sel, 0, 3, O)
                torch.cuda.synchronize()
                times.append(time.perf_counter() - t0)
            took.append(min(times))
        finally:
            cqa.cqa_cache_destroy(h)
    assert took[1] <= 1.6 * took[0], took


def test_more_kv_groups_than_one_launch_holds():
    """A grid dimension holds fewer than 2^32 threads, 8388607 workgroups of 512; one more group of one token each.  The
    softmax of a single score is 1 and the sum of one value that value: exact."""
    import torch

    from helpers import load_binding
    print("dense launches", flush=True)
    cqa = load_binding()
    groups = 8388608 + 5
    v = torch.randn((groups, 128), device="cuda", dtype=torch.float16)
    O = torch.full((groups, 128), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(cqa.cqa_dense_workspace_bytes(1, groups, 1), dtype=torch.uint8, device="cuda")
    cqa.cqa_dense_attention(v, v, v, 1, groups, groups, 1, O, ws)
    torch.cuda.synchronize()
    assert torch.equal(O, v.float())


@pytest.mark.parametrize("bt,hkv,g,n", [(1, 1, 2, 4800), (1, 1, 2, 16 * 41), (1, 2, 4, 48), (2, 1, 4, 16 * 300), (40, 8, 1, 16 * 21), (17, 8, 1, 16 * 143),
                                        (1, 1, 4, 16)])
def test_an_infinite_value_stays_infinite(bt, hkv, g, n):
    """The last token's value has an infinite element: infinite in the result, through the dense call, the fallback and the
    ladder, at whole blocks that leave tiles, splits and trips of the reduction ragged; every other channel untouched."""
    import torch

    from helpers import GpuLayerCache
    print("infinite value", bt, hkv, g, n, flush=True)
    rng = np.random.default_rng(n)
    q = rng.standard_normal((bt, hkv * g, 128)).astype(np.float16)
    k, v = (rng.standard_normal((bt, hkv, n, 128)).astype(np.float16) for _ in range(2))
    v[:, :, n - 1, 7], v[:, :, n - 1, 70] = np.inf, -np.inf
    with GpuLayerCache(bt, hkv * g, hkv, n + 16) as gc:
        cqa = gc.cqa
        gc.append(k, v)
        qd, kd, vd = (gc.to_dev(x) for x in (q, k, v))
        ws = torch.empty(cqa.cqa_dense_workspace_bytes(bt, hkv * g, n), dtype=torch.uint8, device="cuda")
        outs = []
        cqa.cqa_dense_attention(qd, kd, vd, bt, hkv * g, hkv, n, gc.O, ws)
        outs.append(gc.results()[0])
        cqa.cqa_dense_fallback(gc.h, 0, qd, None, 1, 4, gc.O)
        outs.append(gc.results()[0])
        cqa.cqa_decode_step_enqueue(gc.h, 0, None, None, qd, cqa.Tolerances(force_flags=cqa.FLAG_PRECOND), gc.O, gc.cert, gc.flags)
        outs.append(gc.results()[0])
        finite = [c for c in range(128) if c not in (7, 70)]
        for o in outs:
            assert (o[..., 7] == np.inf).all() and (o[..., 70] == -np.inf).all()
            for b, h in ((0, 0), (bt - 1, hkv * g - 1)):
                ref = oracle.softmax_attention(q[b, h], k[b, h // g], v[b, h // g][:, finite])
                assert np.linalg.norm(o[b, h][finite] - ref) <= 1e-3 * np.linalg.norm(ref) + 1e-6


@pytest.mark.parametrize("bt,hkv,g,n", [
    (1, 1, 4, 1),          # one item in a row of eight workgroups
    (3, 3, 4, 33),         # nine items, the last row of eight nearly empty; one split
    (1, 5, 2, 700),        # heads one by one, several splits
    (8, 8, 4, 130),        # 64 workgroups: all four heads apart
    (13, 5, 4, 130),       # 65: in halves
    (16, 8, 4, 40),        # 128: the last size in halves
    (43, 3, 4, 40),        # 129: together
    (2, 8, 4, 4000),       # the workspace allows two splits
])
def test_heads_of_a_group_in_parts(bt, hkv, g, n):
    """Few workgroups: the heads of a KV group are served by workgroups of their own."""
    import torch

    from helpers import load_binding
    cqa = load_binding()
    print("parts", bt, hkv, g, n, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + bt)
    k, v = (torch.randn((bt, hkv, n, 128), generator=gen, device="cuda").half() for _ in range(2))
    q = torch.randn((bt, hkv * g, 128), generator=gen, device="cuda").half()
    guard = 64
    O = torch.full((bt * hkv * g * 128 + guard,), float("nan"), device="cuda")
    nb = cqa.cqa_dense_workspace_bytes(bt, hkv * g, n)
    ws = torch.full((nb + guard,), 0x5A, dtype=torch.uint8, device="cuda")
    cqa.cqa_dense_attention(q, k, v, bt, hkv * g, hkv, n, O, ws)
    torch.cuda.synchronize()
    assert torch.isnan(O[-guard:]).all() and (ws[nb:] == 0x5A).all()
    s = torch.einsum("bhgd,bhnd->bhgn", q.view(bt, hkv, g, 128).cpu().double(), k.cpu().double()) / 128 ** 0.5
    ref = torch.einsum("bhgn,bhnd->bhgd", torch.softmax(s, -1), v.cpu().double()).reshape(bt, hkv * g, 128)
    got = O[:-guard].view(bt, hkv * g, 128).cpu().double()
    # binary32 throughout: 128 products per score, n weights, each rounded once (1e-7 relative)
    assert (got - ref).norm() <= 3e-6 * ref.norm() and (got - ref).abs().max() <= 1e-5 * ref.abs().max()
