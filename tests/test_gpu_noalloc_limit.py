"""The allocation-free entry point close to its scratch limit: a call that fits
with the largest query tiles runs, whatever tiles a call of its size would
otherwise take, and one that needs more is refused."""
import numpy as np
import pytest

from paper_1805_08995_amd import binding, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _say(msg):
    print(msg, flush=True)


def scratch_bytes(n_feat, pairs, tile):
    """Bytes a call takes (pieces rounded up to 256) at `tile` queries per work item."""
    up = lambda n: (n + 255) & ~255  # noqa: E731
    train = sorted(set(int(t) for _, t in pairs))
    tables = sum(up(6 * 257 * 4) + up(144 * n_feat[t]) for t in train)
    views = up(up(56 * len(n_feat)) + up(16 * len(n_feat)) + 4 * len(train))
    items = sum(-(-n_feat[q] // tile) for q, _ in pairs)
    return tables + views + up(up(88 * len(pairs)) + 8 * len(pairs)) + up(16 * items) + up(2048)


@pytest.mark.parametrize("k,largest", [(10, 32), (64, 6)])
def test_largest_tiles_decide_what_fits(k, largest):
    rng = np.random.default_rng(k)
    n_feat = [900] + [57500] * 4
    pairs = np.array([(0, t) for t in range(1, 5)], np.int32)
    # the last image as large as the limit allows at the largest tiles
    while scratch_bytes(n_feat, pairs, largest) + 512 > binding.NOALLOC_SCRATCH_BYTES:
        n_feat[1] -= 1000
    while scratch_bytes(n_feat, pairs, largest) + 512 <= binding.NOALLOC_SCRATCH_BYTES:
        n_feat[4] += 1
    n_feat[4] -= 1
    assert n_feat[4] <= 65535
    # 3600 queries: a call of this size would take 4 queries per item
    assert scratch_bytes(n_feat, pairs, 4) > binding.NOALLOC_SCRATCH_BYTES
    _say(f"noalloc at the scratch limit: k={k} images of {n_feat} points")
    base = torch.from_numpy(synth.desc(rng, max(n_feat))).cuda()
    images = [base[torch.randperm(n, device="cuda")].contiguous() for n in n_feat]
    m = binding.Matcher(k=k)
    codes, keys, _ = m.build_codes(images)
    outs = lambda: tuple(torch.full((4 * n_feat[0],), -7, dtype=torch.int32, device="cuda") for _ in range(3))  # noqa: E731
    got, _ = m.match_pairs_noalloc(images, codes, keys, pairs, out=outs())
    ref, _ = m.match_pairs(images, codes, keys, pairs, out=outs())
    for a, b in zip(got, ref):
        assert torch.equal(a, b)
    # eight points more do not fit even so
    over = torch.cat([images[4], base[:8]])
    images[4] = over
    codes, keys, _ = m.build_codes(images)
    with pytest.raises(binding.CashashError) as e:
        m.match_pairs_noalloc(images, codes, keys, pairs, out=outs())
    assert e.value.code == binding.E_LIMIT
    m.close()
