"""More lookups in one call than a launch has threads for."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def test_more_than_a_launch():
    """2^30 + 70 001 lookups (four lanes each: beyond the 2^32 threads of a grid) of
    4096 values over and over, against the oracle's for them.  Tolerance 0."""
    import torch

    import paper_1807_03249_amd as sb

    rng = np.random.default_rng(30)
    g = rng.integers(0, 256, (6, 7, 4)).astype(np.uint8)
    q = rng.integers(0, 256, (4096, 4)).astype(np.uint8)
    want = torch.from_numpy(oracle.nn_query_n(g, 2, q).view(np.int32)).cuda()
    n = (1 << 30) + 70001
    print(f"[gpu-case] {n} lookups", flush=True)
    st = sb.Style(np.zeros((6, 7, 3), np.uint8), g, channels=2)
    texels = torch.from_numpy(q).cuda().repeat(n // 4096 + 1, 1)[:n]
    got = st.query(texels)
    whole = n // 4096
    for part in got[:whole * 4096].view(whole, 4096).split(1 << 15):
        assert bool((part == want).all())
    assert torch.equal(got[whole * 4096:].flatten(), want[:n - whole * 4096])
