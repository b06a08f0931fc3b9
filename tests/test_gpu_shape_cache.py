"""Launch shapes kept in a file: a line written with or without the class of the
call's size is used, also where CASHASH_AUTOTUNE=0 keeps new lines from being
written, and every shape gives the same outputs."""
import json

import numpy as np
import pytest

from paper_1805_08995_amd import binding, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("size_class", ["", "/q13"])
@pytest.mark.parametrize("autotune", ["0", "1"])
@pytest.mark.parametrize("qt,bpc", [(8, 6), (32, 4)])
def test_shape_of_a_file_is_used(tmp_path, monkeypatch, size_class, autotune, qt, bpc):
    w = synth.scene_set(seed=15, n_images=4, n_feat=1400, n_scenes=2)
    images = [torch.from_numpy(im).cuda() for im in w.images]
    monkeypatch.setenv("CASHASH_AUTOTUNE", "0")
    monkeypatch.delenv("CASHASH_AUTOTUNE_CACHE", raising=False)
    plain = binding.Matcher()
    codes, keys, _ = plain.build_codes(images)
    ref, _ = plain.match_pairs(images, codes, keys, w.pairs)
    # 6 pairs of 1400 points: classes 10 (size) and 13 (8400 queries)
    line = json.dumps({"key": f"gfx950/batched/plain/k10/nt10/nq10{size_class}", "qt": qt, "bpc": bpc})
    cache = tmp_path / "shapes.jsonl"
    cache.write_text(line + "\n")
    monkeypatch.setenv("CASHASH_AUTOTUNE_CACHE", str(cache))
    monkeypatch.setenv("CASHASH_AUTOTUNE", autotune)
    m = binding.Matcher()
    got, st = m.match_pairs(images, codes, keys, w.pairs)
    assert (st["tile_queries"], st["blocks_per_cu"]) == (qt, bpc)
    assert cache.read_text() == line + "\n"
    for a, b in zip(got, ref):
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
