"""Contexts of several threads at once: calls large enough to make and replay
graphs of their launches, beside synchronous copies and contexts that come and
go, give what the same calls give alone."""
import threading

import numpy as np
import pytest

from paper_1805_08995_amd import binding, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

THREADS, CALLS = 6, 8


@pytest.mark.parametrize("own_streams", [False, True])
def test_threads_with_graphs_and_copies(own_streams):
    print(f"threads with graphs and copies, own_streams={own_streams}", flush=True)
    rng = np.random.default_rng(51)
    base = synth.desc(rng, 2500)
    images = [torch.from_numpy(synth.noisy(rng, base[rng.permutation(2500)[:n]])).cuda() for n in (2000, 1500, 2500, 900)]
    pairs = synth.exhaustive_pairs(4)
    pairs = np.concatenate([pairs, pairs[:, ::-1]])  # 20700 queries
    ref_m = binding.Matcher()
    codes, keys, _ = ref_m.build_codes(images)
    ref = [x.cpu().numpy() for x in ref_m.match_pairs(images, codes, keys, pairs)[0]]
    n = len(ref[0])
    streams = [torch.cuda.Stream() for _ in range(THREADS)]
    torch.cuda.synchronize()
    errors = []

    def work(i):
        try:
            with torch.cuda.stream(streams[i]):
                m = binding.Matcher(stream=streams[i].cuda_stream if own_streams else None)
                for call in range(CALLS):
                    # outputs not seen before: another graph
                    out = tuple(torch.full((n,), -7, dtype=torch.int32, device="cuda") for _ in range(3))
                    streams[i].synchronize()
                    got, _ = m.match_pairs(images, codes, keys, pairs, out=out)
                    for g, r, name in zip(got, ref, ("match_idx", "d1sq", "d2sq")):
                        if not np.array_equal(g.cpu().numpy(), r):
                            errors.append(f"thread {i} call {call}: {name}")
                    binding.Matcher(k=5).close()  # synchronous uploads
                m.close()
        except Exception as e:
            errors.append(f"thread {i}: {e!r}")

    threads = [threading.Thread(target=work, args=(i,)) for i in range(THREADS)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
