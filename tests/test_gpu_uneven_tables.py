"""16-bit lookup tables whose source pixels crowd in few buckets, or fill them just
within and just beyond what the table's kernel takes for evenly filled, against the
oracle (tolerance 0: every entry is a source coordinate); and that such a table costs
no more for having fewer bins."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sb():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1807_03249_amd as m

    m.lib()
    return m


def _buckets(rng, side, counts):
    """A guide of 2^14 pixels, counts[i] of them in cell i of a grid of side x side."""
    cell = np.repeat(np.arange(side * side), counts)
    w = 65536 // side
    g = np.stack([cell % side * w, cell // side * w], -1) + rng.integers(0, w, (len(cell), 2))
    return g[rng.permutation(len(g))].reshape(128, 128, 2).astype(np.uint16)


# 128 x 128 pixels fall in 64 x 64 buckets (from 7 bits on): four each, one of 32 and
# one of 33, half of them empty and one more than half; and all bins' smallest number
@pytest.mark.parametrize("spread,bits", [("four", 9), ("full", 8), ("fuller", 8), ("half", 8),
                                         ("emptier", 8), ("one", 7), ("few", 7), ("one", 1),
                                         ("emptier", 2)])
def test_uneven_buckets(sb, spread, bits):
    rng = np.random.default_rng(len(spread) * 100 + bits)
    counts = np.full(4096, 4)
    if spread in ("full", "fuller"):
        counts[1000] = 32 if spread == "full" else 33
        counts[2000:2000 + counts[1000] - 4] -= 1
    elif spread in ("half", "emptier"):
        counts[rng.permutation(4096)[:2048 + (spread == "emptier")]] = 0
        held = np.flatnonzero(counts)
        counts[held] = 8
        counts[held[:16384 - counts.sum()]] += 1
    elif spread in ("one", "few"):
        counts[:] = 0
        counts[rng.permutation(4096)[:1 if spread == "one" else 5]] = 1
        counts[np.flatnonzero(counts)] = 16384 // counts.sum()
        counts[np.flatnonzero(counts)[0]] += 16384 - counts.sum()
    g = _buckets(rng, 64, counts)
    print(f"[gpu-case] uneven buckets {spread} bits={bits}", flush=True)
    st = sb.Style(np.zeros((128, 128, 3), np.uint8), g, bits)
    np.testing.assert_array_equal(st.lut.cpu().numpy().view(np.uint32), oracle.lut_build(g, bits))


def test_crowded_table_cost(sb):
    """All pixels at one value: every bin of the table walks to their bucket, so a
    sixteenth of the bins takes less time (a third of it; with too few threads for
    their long walks it took as long)."""
    import torch

    g = torch.full((128, 128, 2), 21845, dtype=torch.int16, device="cuda")
    rgb = torch.zeros(128, 128, 3, dtype=torch.uint8, device="cuda")

    def ms(bits):
        best = float("inf")
        for _ in range(3):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            torch.cuda.synchronize()
            t[0].record()
            sb.Style(rgb, g, bits)
            t[1].record()
            t[1].synchronize()
            best = min(best, t[0].elapsed_time(t[1]))
        return best

    print("[gpu-case] cost of a crowded table", flush=True)
    assert ms(9) < 0.6 * ms(11)
