"""Hash codes where few, many and all projections are recomputed in binary64, in
both forms, around the sizes of a block (256 descriptors in the plain form, 64 in
the batched one), against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1805_08995_amd import binding, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mode", ["plain", "batched"])
@pytest.mark.parametrize("margin", [1e-3, 1e-1, 1e3])
@pytest.mark.parametrize("sizes", [[1], [15, 0, 17], [255], [256], [257], [40, 300, 0, 4097, 64]])
def test_codes_at_any_margin(mode, margin, sizes):
    print(f"codes mode={mode} margin={margin} sizes={sizes}", flush=True)
    rng = np.random.default_rng(sum(sizes))
    images = [synth.desc(rng, n) for n in sizes]
    if sizes[-1] > 1:
        images[-1][0] = 0    # a descriptor of zeros and one of the largest bytes
        images[-1][1] = 255
    mats = synth.projection_matrices()
    oc, ok = oracle.build_codes(images, *mats)
    m = binding.Matcher(*mats, mode=mode, margin_coef=margin)
    dev = [torch.from_numpy(im).cuda() for im in images]
    for _ in range(2):
        codes, keys, st = m.build_codes(dev)
        for i in range(len(sizes)):
            assert np.array_equal(codes[i].cpu().numpy().view(np.uint64).reshape(-1, 2), oc[i]), i
            assert np.array_equal(keys[i].cpu().numpy(), ok[i]), i
        if margin == 1e3:  # every projection, but those of the zero descriptor (its margin is the constant part)
            assert st["near_margin_recomputes"] == 176 * (sum(sizes) - (sizes[-1] > 1))
    m.close()
