"""GPU: re-deliveries known by their bytes inside the one-call path.

From 256 MiB of deliveries on, the one-call path compares deliveries of equal
score and length instead of hashing each of them first. Groups where every form
meets: copies, a damaged copy (one bit, in the last bytes of the last tensor), equal
K with another V (with copies of their own, which are no copies of the group's
first), and an equal score at another length. The result must be the serial
pipeline's, which hashes every delivery and never compares, bit for bit: Ids, plan,
merged cache; also replayed from a graph. With a non-finite score in the set nothing
is rendered, and the Ids of the deliveries with an equal score are written all the
same."""

import numpy as np
import pytest
import torch

import synth
import paper_2607_01308_amd as cm
from paper_2607_01308_amd import _cabi as C

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    yield
    torch.cuda.synchronize()


def _clone(c):
    return tuple((k.clone(), v.clone()) for k, v in c)


def _groups(dtype, T):
    d = 128 if dtype == "bfloat16" else 64
    w = synth.custom("copies", L=8, H=8, d=d, dtype=dtype, lengths=(T, T, T + 100, T + 13),
                     shared_k=((0, 1),), seed=T)
    a, b, e, z = synth.make_fragments(w, device="cuda")
    for (ka, _), (ke, _) in zip(a, e):
        ke[:, :, -T:] = ka                       # a's score, another length
    flipped = _clone(a)
    flipped[-1][1].view(torch.int32).view(-1)[-1] ^= 1
    return [a, b, _clone(a), flipped, _clone(b), _clone(a), e, _clone(e), _clone(flipped), z]


@pytest.mark.parametrize("dtype,T,seed", [("bfloat16", 1201, 0), ("bfloat16", 1201, 1),
                                          ("bfloat16", 1280, 2), ("float32", 1203, 3)])
def test_copies_against_the_serial_pipeline(dtype, T, seed):
    dl = _groups(dtype, T)
    dl = [dl[i] for i in np.random.default_rng(seed).permutation(len(dl))]
    batch = cm.FragmentBatch(dl)
    assert sum(batch.fragment_bytes(i) for i in range(batch.n)) > 256 << 20
    want = cm.render_deliveries(batch, 3, 1e6, pipeline="serial")
    got = cm.render_deliveries(batch, 3, 1e6)
    graph = cm.RenderGraph(batch, 3, 1e6)
    for r in (got, graph.replay(), graph.replay()):
        assert r.digests == want.digests
        assert r.n_unique == 5
        assert np.array_equal(r.plan, want.plan)
        assert torch.equal(r.merged.view(torch.int16), want.merged.view(torch.int16))
    graph.close()


@pytest.mark.parametrize("L,lengths", [(8, (3000, 2999)), (1, (20000, 17))])
def test_only_copies(L, lengths):
    """Every delivery of a key is the same fragment: no digest is read before the order.
    Tensors of 6 MB, and of 41 MB beside 35 KB, whose trees take a launch more, which
    passes over the deliveries that were not hashed."""
    w = synth.custom("same", L=L, H=8, d=128, lengths=lengths, seed=5)
    a, b = synth.make_fragments(w, device="cuda")
    batch = cm.FragmentBatch([b, a, _clone(a), _clone(b), _clone(a), _clone(a)])
    assert sum(batch.fragment_bytes(i) for i in range(batch.n)) > 256 << 20
    want = cm.render_deliveries(batch, L // 2, 1e6, pipeline="serial")
    got = cm.render_deliveries(batch, L // 2, 1e6)
    assert got.digests == want.digests and np.array_equal(got.plan, want.plan)
    assert torch.equal(got.merged.view(torch.int16), want.merged.view(torch.int16))


@pytest.mark.parametrize("n", [12, 100])
def test_colliding_ids_are_written_beside_a_non_finite_score(n):
    if n == 12:
        dl = _groups("bfloat16", 1201)
        dl.append(_clone(dl[-1]))                # the only copies among those that collide
    else:
        dl = _many(n, 70, 800, seed=8)[1:]
    layer = len(dl[0]) // 2
    bad = tuple((k + 0, v + 0) for k, v in dl[1])
    bad[layer][0][0, 0, -1, 0] = float("nan")
    dl.insert(4, bad)
    batch = cm.FragmentBatch(dl)
    assert batch.n == n and sum(batch.fragment_bytes(i) for i in range(n)) > 256 << 20
    T = sum(batch.lengths)
    keys = torch.empty(n, dtype=torch.float64, device="cuda")
    mask = torch.empty(n, dtype=torch.uint8, device="cuda")
    digests = torch.full((n, 32), 0xCD, dtype=torch.uint8, device="cuda")
    plan = torch.empty(cm.plan_elems(n), dtype=torch.int64, device="cuda")
    out = torch.full((batch.L * 2 * batch.H * T * batch.d,), 7.0, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(cm.workspace_size(batch), dtype=torch.uint8, device="cuda")
    cm.render_deliveries_async(batch, layer, min(batch.lengths), 1e6, "half", keys, mask, digests,
                               plan, out, T, ws)
    assert int(plan[C.PLAN_STATUS]) == C.CM_ENONFINITE
    ids = cm.fragment_ids(dl)
    got = [bytes(r) for r in digests.cpu().numpy()]
    collide = mask.cpu().tolist()
    scores = keys.cpu().tolist()
    assert collide == [int(scores.count(k) > 1) for k in scores] and collide[4] == 0
    assert sum(collide) >= n // 2
    assert got == [f if c else b"\xcd" * 32 for f, c in zip(ids, collide)]
    assert bool((out == 7.0).all())


def _many(n, copies, T, seed, L=2):
    """n deliveries of L x H = 8 x T x d = 64, `copies` of them drawn from the others."""
    w = synth.custom("many", L=L, H=8, d=64, lengths=(T,) * (n - copies), routing_layer=1, seed=seed)
    base = list(synth.make_fragments(w, device="cuda"))
    rng = np.random.default_rng(seed)
    dl = base + [_clone(base[int(i)]) for i in rng.integers(0, len(base), copies)]
    return [dl[i] for i in rng.permutation(n)]


@pytest.mark.parametrize("n,T,compares", [(1024, 8, 0), (128, 512, 1), (127, 512, 0)])
def test_deliveries_are_compared_from_256_mib_on(n, T, compares):
    """4096 stripes of little (33 MB) and of 64 KiB (256 MiB), and one delivery less."""
    batch = cm.FragmentBatch(_many(n, 3, T, seed=n))
    assert (sum(batch.fragment_bytes(i) for i in range(n)) >= 256 << 20) == bool(compares)
    cm.timing_reset()
    cm.timing_enable(True)
    try:
        res = cm.render_deliveries(batch, 1, 1e6)
        torch.cuda.synchronize()
        launches = cm.timing_query("key_mask")[1]
    finally:
        cm.timing_enable(False)
        cm.timing_reset()
    assert launches == 1 + compares
    assert res.n_unique == n - 3


@pytest.mark.parametrize("n,copies,T", [(300, 120, 257), (1024, 1000, 256), (65, 40, 2100)])
def test_many_deliveries_against_the_serial_pipeline(n, copies, T):
    """More deliveries than a wave has lanes: copies, damaged copies (the first, a
    middle and the last bytes), a pair with equal K and copies of one of it."""
    dl = _many(n, copies, T, seed=n)
    rng = np.random.default_rng(n)
    for k, i in enumerate(rng.choice(n, size=9, replace=False)):
        dl[i] = _clone(dl[i])
        x = dl[i][(0, 1, -1)[k % 3]][1].view(torch.int32).view(-1)
        x[(0, x.numel() // 2, -1)[k % 3]] ^= 1 << k
    a, b, c = (int(i) for i in rng.choice(n, size=3, replace=False))
    dl[b] = tuple((k.clone(), v.flip(2).contiguous()) for k, v in dl[a])
    dl[c] = _clone(dl[b])
    batch = cm.FragmentBatch(dl)
    assert sum(batch.fragment_bytes(i) for i in range(n)) >= 256 << 20
    want = cm.render_deliveries(batch, 1, 1e6, pipeline="serial")
    got = cm.render_deliveries(batch, 1, 1e6)
    assert got.digests == want.digests
    assert np.array_equal(got.plan, want.plan)
    assert torch.equal(got.merged.view(torch.int16), want.merged.view(torch.int16))


def test_many_small_copies_take_no_longer_than_hashing_them():
    """1000 copies of 1 MiB, 16 stripes each: compared by the whole chip (they took
    fifteen times as long with each delivery's stripes on the same few waves)."""
    batch = cm.FragmentBatch(_many(1024, 1000, 256, seed=2))
    time = {}
    for pipeline in ("fused", "serial") * 2:
        cm.render_deliveries(batch, 1, 1e6, pipeline=pipeline).plan
        t = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            cm.render_deliveries(batch, 1, 1e6, pipeline=pipeline).plan
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        time[pipeline] = min(t)
    assert time["fused"] < 2 * time["serial"], time


def test_order_is_no_slower_where_copies_are_looked_for():
    """The order of 1024 distinct deliveries, with re-deliveries known by their bytes
    (1 GiB) and without (128 MiB): no delivery is walked for another one's copies (that
    took 1.8 times as long)."""
    best = {}
    for T in (32, 256):
        batch = cm.FragmentBatch(_many(1024, 0, T, seed=3))
        for _ in range(5):
            cm.timing_reset()
            cm.timing_enable(True)
            try:
                cm.render_deliveries(batch, 1, 1e6).plan
                torch.cuda.synchronize()
                ms, launches = cm.timing_query("order")
            finally:
                cm.timing_enable(False)
                cm.timing_reset()
            assert launches == 1
            best[T] = min(best.get(T, 1e9), ms)
    assert best[256] < 1.4 * best[32], best
