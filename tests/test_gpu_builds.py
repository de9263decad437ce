"""Style registration on the GPU (lookup tables and search trees) at the sizes
where the build kernels change their split, against the oracle.  Tolerance 0:
every entry is a source coordinate."""
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


# sides around one scan block (4^6 buckets from 128 x 128 pixels on), several
# blocks, fewer pixels than a wave, and a last wave with one pixel
@pytest.mark.parametrize("sw,sh,bits,spread", [(1, 1, 3, "noise"), (13, 5, 8, "noise"),
                                               (129, 127, 8, "smooth"), (130, 131, 9, "runs"),
                                               (256, 256, 9, "noise"), (301, 260, 11, "smooth"),
                                               (256, 257, 4, "one")])
def test_16bit_table(sb, sw, sh, bits, spread):
    """The bucket sort behind a 16-bit table: runs of equal buckets within and
    across waves, every pixel in one bucket, and a label no pixel holds."""
    rng = np.random.default_rng(sw * 1000 + sh)
    if spread == "smooth":  # neighbours share buckets, as in texture coordinates
        y, x = np.mgrid[0:sh, 0:sw]
        g = np.stack([x * 65536 // sw, y * 65536 // sh], -1)
    elif spread == "runs":
        g = np.repeat(rng.integers(0, 65536, (sh, (sw + 9) // 10, 2)), 10, 1)[:, :sw]
    else:
        g = rng.integers(0, 65536 if spread == "noise" else 1, (sh, sw, 2)) + (spread == "one") * 777
    g = np.ascontiguousarray(g.astype(np.uint16))
    rgb = rng.integers(0, 256, (sh, sw, 3)).astype(np.uint8)
    labels = rng.integers(0, 2, (sh, sw)).astype(np.uint8)  # label 2 is absent
    print(f"[gpu-case] 16-bit table {sw}x{sh} bits={bits} {spread}", flush=True)
    st = sb.Style(rgb, g, bits, labels=labels, nlabels=3)
    np.testing.assert_array_equal(st.lut.cpu().numpy().view(np.uint32), oracle.lut_build(g, bits))
    np.testing.assert_array_equal(st.label_luts.cpu().numpy().view(np.uint32),
                                  oracle.lut_build_labels(g, labels, 3, bits))
