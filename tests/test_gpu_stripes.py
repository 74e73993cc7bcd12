"""GPU: Ids of tensors whose chunk counts lie around the edges of what a wave folds.

A wave folds its stripe of 64 chunks to nodes of the tensor's tree; the levels
above are folded by the launches that follow. Chunk counts around one, two, four
and thirty-two stripes' edges, a last chunk of one row, and a tensor long enough
for a launch between the stripes and the top (over 16 MiB), against the oracle's
BLAKE3: the hash alone, and inside the whole path (dense and paged)."""

import pytest
import torch

import oracle
import synth
import paper_2607_01308_amd as cm

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    yield
    torch.cuda.synchronize()


def _ids(caches):
    return [oracle.fragment_id(oracle.Fragment(*synth.to_numpy_cache(c))) for c in caches]


# rows of 256 bytes: four per chunk, and one head, so T = 4 c + r is c chunks and r rows
@pytest.mark.parametrize("chunks", [1, 2, 16, 17, 32, 33, 63, 64, 65, 96, 127, 128, 129, 191, 255,
                                    257, 2047, 2049])
def test_ids_around_stripe_edges(chunks):
    w = synth.custom("edges", L=2, H=1, d=128, lengths=(4 * chunks, 4 * chunks + 1, 7),
                     seed=chunks)
    frags = synth.make_fragments(w, device="cuda")
    want = _ids(frags)
    assert cm.fragment_ids(frags) == want
    assert cm.render_deliveries(frags, 1, 1e6).digests == want
    pool, lengths, lists, free = synth.make_paged(frags, 16, 2 * (sum(w.lengths) // 16 + 2))
    r = cm.render_paged_set(cm.PagedSet(pool, lengths, lists), 1, 1e6, free)
    torch.cuda.synchronize()
    assert [bytes(x) for x in r.digests_dev.cpu().numpy()] == want


def test_ids_of_tensors_beyond_the_top_launch():
    w = synth.custom("long", L=1, H=1, d=128, lengths=(4 * 64 * 600 + 3, 5), seed=3)
    frags = synth.make_fragments(w, device="cuda")
    want = _ids(frags)
    assert cm.fragment_ids(frags) == want
    assert cm.render_deliveries(frags, 0, 1e6).digests == want


# 2 x 512 stripes: a chunk grid of a wave per SIMD of 256 compute units, and one of more
@pytest.mark.parametrize("T", [131072, 131073])
def test_ids_around_one_wave_per_simd(T):
    w = synth.custom("grid", L=1, H=1, d=128, lengths=(T,), seed=T)
    frags = synth.make_fragments(w, device="cuda")
    want = _ids(frags)
    assert cm.fragment_ids(frags) == want
    pool, lengths, lists, free = synth.make_paged(frags, 64, 2 * (T // 64 + 2))
    r = cm.render_paged_set(cm.PagedSet(pool, lengths, lists), 0, 1e6, free, fused=False)
    torch.cuda.synchronize()
    assert [bytes(x) for x in r.digests_dev.cpu().numpy()] == want
