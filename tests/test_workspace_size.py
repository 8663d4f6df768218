"""A workspace sized for an upper bound of the sequence lengths serves every shorter call: its size
never falls as max_seqlen or the total grows (host only)."""
import pytest

import paper_2509_05165_amd as kv


@pytest.mark.parametrize("dtype,d,hq,hkv,window,more", [
    (kv.KVC_BF16, 64, 32, 8, 200, {}), (kv.KVC_F32, 256, 16, 2, 4096, {}), (kv.KVC_BF16, 80, 48, 12, 300, {}),
    (kv.KVC_BF16, 64, 32, 4, 100, dict(value_norm=1)), (kv.KVC_BF16, 128, 32, 8, 64, {}),
    (kv.KVC_BF16, 128, 40, 8, 64, dict(order=kv.KVC_ORDER_POSITION, unstructured=1)),
])
def test_workspace_never_shrinks(dtype, d, hq, hkv, window, more):
    p = kv.KvcParams(4, 80, hq, hkv, d, window, dtype, **more)
    for total in (5000, 80000, 600000):
        sizes = [kv.kvc_workspace_size(p, total, n) for n in range(1, total + 1, max(1, total // 997))]
        assert sizes == sorted(sizes)
    sizes = [kv.kvc_workspace_size(p, t, 3000) for t in range(3000, 400000, 997)]
    assert sizes == sorted(sizes)
