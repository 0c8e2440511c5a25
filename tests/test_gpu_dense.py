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
