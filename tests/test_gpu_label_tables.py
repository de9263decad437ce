"""8-bit lookup tables at the edges of the separable passes' short lines, and tables
per label for few and many labels, against the oracle (tolerance 0); and what many
labels cost."""
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


# values along each channel: two channels search a line of up to 128 whole at 8 bits
# (one column a workgroup) and of any length at 7, three channels (16 columns) of up
# to 8 at 8 bits and 32 at 6
@pytest.mark.parametrize("channels,bits,values", [
    (2, 8, (127, 3)), (2, 8, (128, 128)), (2, 8, (129, 129)), (2, 8, (1, 200)), (2, 7, (256, 256)),
    (3, 8, (7, 8, 9)), (3, 6, (31, 32, 33)), (3, 6, (33, 5, 32)),
    (3, 1, (3, 256, 2))])
def test_short_lines(sb, channels, bits, values):
    rng = np.random.default_rng(channels * 100 + bits + sum(values))
    sh, sw = 53, 59
    g = rng.integers(0, 256, (sh, sw, 4 if channels == 3 else 2)).astype(np.uint8)
    for c, n in enumerate(values):
        held = np.sort(rng.permutation(256)[:n]).astype(np.uint8)
        g[..., c] = held[rng.integers(0, n, (sh, sw))]
    weights = [5, 1, 127] if channels == 3 and bits == 6 else None
    print(f"[gpu-case] short lines channels={channels} bits={bits} {values}", flush=True)
    st = sb.Style(np.zeros((sh, sw, 3), np.uint8), g, bits, weights=weights)
    want = oracle.lut_build(g, bits, weights) if channels == 3 else oracle.lut_build(g, bits)
    np.testing.assert_array_equal(st.lut.cpu().numpy().view(np.uint32), want)


@pytest.mark.parametrize("nlabels,flat", [(8, False), (9, False), (13, True)])
def test_label_tables(sb, nlabels, flat):
    """Pixels of a value in runs and apart, their labels mixed: with up to eight
    labels only those that may lower an entry write it."""
    rng = np.random.default_rng(nlabels)
    sh, sw = 70, 61
    g = rng.integers(0, 3 if flat else 12, (sh, sw, 2)).astype(np.uint8) * 20
    labels = np.repeat(rng.integers(0, nlabels - 1, (sh, (sw + 2) // 3)), 3, 1)[:, :sw]
    labels = np.ascontiguousarray(labels.astype(np.uint8))  # the last label is absent
    print(f"[gpu-case] tables of {nlabels} labels flat={flat}", flush=True)
    st = sb.Style(np.zeros((sh, sw, 3), np.uint8), g, 6, labels=labels, nlabels=nlabels)
    np.testing.assert_array_equal(st.label_luts.cpu().numpy().view(np.uint32),
                                  oracle.lut_build_labels(g, labels, nlabels, 6))


def test_cost_of_many_labels(sb):
    """Sixteen tables of a 2048 x 2048 guide take less than four times as long as
    two (2.8 times; each pass waiting for entries it seldom lowers, 5.2)."""
    import torch

    gen = torch.Generator(device="cuda")
    gen.manual_seed(16)
    size = 2048
    g = torch.randint(0, 256, (size, size, 2), generator=gen, device="cuda").byte()
    rgb = torch.zeros(size, size, 3, dtype=torch.uint8, device="cuda")
    y, x = torch.meshgrid(*[torch.arange(size, device="cuda")] * 2, indexing="ij")

    def ms(n):
        labels = (((x // 300) + 5 * (y // 300)) % n).byte()
        best = float("inf")
        for _ in range(5):
            t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            torch.cuda.synchronize()
            t[0].record()
            for _ in range(3):
                sb.Style(rgb, g, 8, labels=labels, nlabels=n)
            t[1].record()
            t[1].synchronize()
            best = min(best, t[0].elapsed_time(t[1]))
        return best

    print("[gpu-case] cost of many labels", flush=True)
    assert ms(16) < 4 * ms(2)
