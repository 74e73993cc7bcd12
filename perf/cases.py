"""The work this library is used for, as cases that can be prepared, run, checked
and timed: the CanonicalMerge render of sets of KV-cache fragments through the
public entry points, from two fragments of a few tokens (latency) to the 39 GB
Qwen3-4B-shaped set (throughput).

A case is a dict of plain values:
  call      which entry point (see run())
  L, H, d   layers, KV heads, head dimension
  dtype     "bfloat16" | "float32"
  style     RoPE pairing, "half" | "interleaved"
  base      RoPE base
  lengths   tokens of each distinct fragment, as text "512,768"
  arrivals  deliveries in order of arrival, indices of distinct fragments, as
            text "0,1,1": an index that comes again is a byte copy in other memory
  equal     "a,b": fragment b has the K of fragment a and another V, so their
            scores are equal and their contents differ; "" for none
  block     tokens per page (paged storage only)
The routing layer is the middle one, L // 2.
"""

import math

import numpy as np
import torch

import paper_2607_01308_amd as cm

_DT = {"bfloat16": torch.bfloat16, "float32": torch.float32}

# The Qwen3-1.7B N=5 set: 256 to 2048 tokens, each fragment delivered one to
# three times, shuffled.
_N5_LENGTHS = "416,1643,1429,1042,1032"
_N5_ARRIVALS = "3,0,1,0,1,2,3,0,4,3,4"

# The Qwen3-4B large set: 31 fragments of 2048 to 16384 tokens, 264 thousand in
# all, one of them delivered twice and one pair with equal scores.
_LARGE_LENGTHS = ("2657,7250,14259,10552,2713,7667,9497,10989,14981,11450,10579,2242,8918,13178,"
                  "6430,16324,2174,7384,4372,3648,5678,14845,2894,11024,2588,7384,12967,12351,"
                  "5403,15431,6352")
_LARGE_ARRIVALS = ("9,16,17,0,14,12,3,30,11,27,8,29,19,26,28,13,22,23,15,24,5,0,4,18,2,25,10,7,"
                   "6,1,21,20")


def listed():
    qwen_17b = dict(L=28, H=8, d=128, dtype="bfloat16", style="half", base=1e6)
    qwen_4b = dict(L=36, H=8, d=128, dtype="bfloat16", style="half", base=1e6)
    tiny = dict(L=2, H=2, d=64, dtype="float32", style="half", base=1e4)

    def case(name, call, shape, lengths, arrivals="", equal="", block=0):
        arrivals = arrivals or ",".join(str(i) for i in range(len(lengths.split(","))))
        return dict(name=name, call=call, lengths=lengths, arrivals=arrivals, equal=equal,
                    block=block, **shape)

    return [
        # the smallest merge, two fragments of a few tokens: all launches and latency. A serving
        # loop that keeps its buffers and calls the library once per merge, steps 1-5.
        case("tiny-deliveries", "deliveries-into", tiny, "16,24"),
        # the same set rendered again after its Ids are known (steps 2-5)
        case("tiny-set", "set-into", tiny, "16,24"),
        # two agents' thoughts of some hundred tokens, 1.7B model: the ordinary merge
        case("1.7b-n2-deliveries", "deliveries-into", qwen_17b, "512,768"),
        # its render on every decode after the set has been ingested
        case("1.7b-n2-set", "set-into", qwen_17b, "512,768"),
        # five agents over an at-least-once transport: most fragments arrive again and are absorbed
        case("1.7b-n5-redelivered", "deliveries", qwen_17b, _N5_LENGTHS, _N5_ARRIVALS),
        # one fragment of odd length arrives and is ingested: its content address only
        case("1.7b-ingest", "ids", qwen_17b, "1531"),
        # ragged fragments that live on pages of 16 tokens, merged inside the pool
        case("1.7b-n5-paged", "paged", qwen_17b, _N5_LENGTHS, block=16),
        # float32 caches, interleaved pairs, lengths that fit nothing
        case("fp32-interleaved-ragged", "deliveries",
             dict(L=12, H=4, d=128, dtype="float32", style="interleaved", base=1e4),
             "333,1021,77,500,1,219"),
        # four long thoughts of a 4B model, steps 1-5
        case("4b-n4-deliveries", "deliveries", qwen_4b, "4096,4096,4096,4096"),
        # and steps 2-5 of the ingested set: streaming
        case("4b-n4-set", "set", qwen_4b, "4096,4096,4096,4096"),
        # the largest: 39 GB delivered, 39 GB merged
        case("4b-large-deliveries", "deliveries", qwen_4b, _LARGE_LENGTHS, _LARGE_ARRIVALS,
             equal="25,17"),
    ]


def draw(rng):
    """One more case: any call, shape, type and pairing of the listed ranges, 100 KB to 5 GB
    delivered, one to twelve fragments of one token and up, odd lengths, with or without
    re-deliveries and a pair of equal scores."""
    call = rng.choice(["deliveries", "deliveries", "deliveries-into", "set", "set-into", "ids",
                       "paged"])
    dtype = rng.choice(["bfloat16", "bfloat16", "float32"])
    d = rng.choice([64, 128, 128, 256])
    H = rng.choice([1, 2, 4, 8])
    L = rng.randint(2, 36)
    n = rng.randint(1, 12)
    token = 2 * L * H * d * (2 if dtype == "bfloat16" else 4)
    tokens = math.exp(rng.uniform(math.log(1e5), math.log(5e9))) / token
    parts = [math.exp(rng.uniform(0.0, math.log(8.0))) for _ in range(n)]
    lengths = [max(1, int(tokens * p / sum(parts))) for p in parts]
    arrivals, equal = list(range(n)), ""
    if call.startswith("deliveries"):
        if rng.random() < 0.4:
            arrivals += [rng.randrange(n) for _ in range(rng.randint(1, n))]
        if n >= 2 and rng.random() < 0.25:
            a, b = rng.sample(range(n), 2)
            lengths[b] = lengths[a]
            equal = "%d,%d" % (a, b)
        rng.shuffle(arrivals)
    return dict(call=call, L=L, H=H, d=d, dtype=dtype, style=rng.choice(["half", "interleaved"]),
                base=rng.choice([1e4, 1e6]), lengths=",".join(map(str, lengths)),
                arrivals=",".join(map(str, arrivals)), equal=equal,
                block=16 if call == "paged" else 0)


def _ints(text):
    return [int(x) for x in text.split(",") if x]


def _fragments(case, seed):
    """The distinct fragments, legacy caches (tuples over layers of (K, V), each [1, H, T, d]):
    K ~ N(0, s_i^2) with log-normal s_i, V ~ N(0, 1)."""
    lengths, equal = _ints(case["lengths"]), _ints(case["equal"])
    g = torch.Generator(device="cuda")
    g.manual_seed(1_000_003 * int(seed) + 17)
    z = np.random.default_rng(int(seed)).standard_normal(len(lengths))
    # scores apart by at least a percent, as different thoughts' are
    scale = np.exp(0.3 * z + 0.01 * np.argsort(np.argsort(z)))
    frags = []
    for i, T in enumerate(lengths):
        layers = []
        for _ in range(case["L"]):
            x = torch.randn((2, 1, case["H"], T, case["d"]), generator=g, device="cuda")
            x[0].mul_(float(scale[i]))
            x = x.to(_DT[case["dtype"]])
            layers.append((x[0], x[1]))
        frags.append(tuple(layers))
    if equal:
        a, b = equal
        frags[b] = tuple((ka.clone(), vb) for (ka, _), (_, vb) in zip(frags[a], frags[b]))
    return frags


def _deliveries(case, frags):
    seen, out = set(), []
    for i in _ints(case["arrivals"]):
        out.append(tuple((k.clone(), v.clone()) for k, v in frags[i]) if i in seen else frags[i])
        seen.add(i)
    return out


def _pages(case, frags, seed):
    """The fragments on pages of `block` tokens at random places of one pool [L, 2, P, H, B, d]
    with as many free pages as a merge can need; rows past a fragment's end are zero."""
    B = case["block"]
    lengths = [f[0][0].shape[2] for f in frags]
    need = [-(-T // B) for T in lengths]
    spare = 2 * -(-sum(lengths) // B)
    P = sum(need) + spare
    perm = np.random.default_rng(int(seed) + 1).permutation(P)
    pool = torch.zeros((case["L"], 2, P, case["H"], B, case["d"]), dtype=_DT[case["dtype"]],
                       device="cuda")
    lists, at = [], 0
    for f, T, nb in zip(frags, lengths, need):
        ids = perm[at:at + nb]
        at += nb
        lists.append([int(q) for q in ids])
        where = torch.as_tensor(ids, device="cuda")
        for l, kv in enumerate(f):
            for w, x in enumerate(kv):
                rows = torch.zeros((case["H"], nb * B, case["d"]), dtype=x.dtype, device="cuda")
                rows[:, :T] = x[0]
                pool[l, w, where] = rows.view(case["H"], nb, B, case["d"]).transpose(0, 1)
    return pool, lengths, lists, [int(q) for q in perm[at:]]


def prepare(case, seed):
    s = dict(case=case, layer=case["L"] // 2)
    frags = _fragments(case, seed)
    call = case["call"]
    if call == "ids":
        s["caches"] = frags
        return s
    if call == "paged":
        pool, lengths, lists, free = _pages(case, frags, seed)
        s["pages"] = cm.PagedSet(pool, lengths, lists)
        s["free"] = np.array(free, dtype=np.int32)
        return s
    if call in ("set", "set-into"):
        fset = cm.LatentFragmentSet()
        ids = fset.ingest_many(frags)
        if call == "set":
            s["set"] = fset
            return s
        s["ids"] = torch.tensor(np.frombuffer(b"".join(ids), dtype=np.uint8).reshape(-1, 32),
                                device="cuda")
        deliveries = frags
    else:
        deliveries = _deliveries(case, frags)
    b = s["batch"] = cm.FragmentBatch(deliveries)
    if call in ("deliveries-into", "set-into"):
        # the buffers of a program that merges in a loop
        T = sum(b.lengths)
        s["out"] = torch.empty((b.L, 2, 1, b.H, T, b.d), dtype=b.torch_dtype, device="cuda")
        s["keys"] = torch.empty(b.n, dtype=torch.float64, device="cuda")
        s["mask"] = torch.empty(b.n, dtype=torch.uint8, device="cuda")
        s["digests"] = torch.empty((b.n, 32), dtype=torch.uint8, device="cuda")
        s["plan"] = torch.empty(cm.plan_elems(b.n), dtype=torch.int64, device="cuda")
        s["ws"] = torch.empty(max(cm.workspace_size(b), 256), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    case, call = s["case"], s["case"]["call"]
    if call == "ids":
        return np.frombuffer(b"".join(cm.fragment_ids(s["caches"])), dtype=np.uint8)
    if call == "paged":
        p = s["pages"]
        r = cm.render_paged_set(p, s["layer"], case["base"], s["free"], style=case["style"])
        return dict(pool=p.pool, k_table=r.k_table, v_table=r.v_table, digests=r.digests_dev,
                    keys=r.keys_dev)
    if call == "set":
        r = s["set"].render(s["layer"], case["base"], style=case["style"])
        return dict(merged=_layers(r.merged), keys=r.keys_dev, plan=r.plan_dev)
    if call == "deliveries":
        r = cm.render_deliveries(s["batch"], s["layer"], case["base"], style=case["style"])
        return dict(merged=_layers(r.merged), digests=r.digests_dev, keys=r.keys_dev,
                    plan=r.plan_dev)
    b = s["batch"]
    T = sum(b.lengths)
    if call == "set-into":
        cm.render_set(b, s["ids"], s["layer"], min(b.lengths), case["base"], case["style"],
                      s["keys"], s["plan"], s["out"], T, s["ws"])
        return dict(merged=s["out"], keys=s["keys"], plan=s["plan"])
    cm.render_deliveries_async(b, s["layer"], min(b.lengths), case["base"], case["style"],
                               s["keys"], s["mask"], s["digests"], s["plan"], s["out"], T, s["ws"])
    # the merged rows lie at the buffer's start; with nothing absorbed they fill it
    whole = len(set(_ints(case["arrivals"]))) == b.n
    return dict(merged=s["out"] if whole else s["out"].view(-1)[:_merged_elements(case)],
                digests=s["digests"], keys=s["keys"], plan=s["plan"], mask=s["mask"])


def _layers(merged):
    """The merged cache layer by layer, as a model takes it."""
    return [merged[l] for l in range(merged.shape[0])]


def _merged_elements(case):
    return 2 * case["L"] * case["H"] * case["d"] * sum(_ints(case["lengths"]))


def _bytes(case, lengths):
    e = 2 if case["dtype"] == "bfloat16" else 4
    return 2 * case["L"] * case["H"] * case["d"] * e * sum(lengths)


def work(case):
    """bytes: every delivery (set calls: every member) read once, the merged cache written once.
    flops: the rotation of the merged K, two products and a sum per element. The content address
    costs 672 integer operations per 64 delivered bytes besides."""
    lengths = _ints(case["lengths"])
    arrived = [lengths[i] for i in _ints(case["arrivals"])]
    if case["call"] == "ids":
        return {"bytes": _bytes(case, lengths), "flops": 0}
    if case["call"] == "paged":
        # every fragment page is read (its Id); V of a page-aligned slot stays where it is, here
        # counted as written like the rest, since lengths are ragged
        return {"bytes": 2 * _bytes(case, lengths), "flops": 3 * _merged_elements(case) // 2}
    read = lengths if case["call"].startswith("set") else arrived
    return {"bytes": _bytes(case, read) + _bytes(case, lengths),
            "flops": 3 * _merged_elements(case) // 2}


def tolerance(case):
    """Merged K is rounded once from a result of 64 bits and V is copied, so another correct
    implementation differs in a last bit here and there: by at most one unit of it, 2^-7 of the
    value in bfloat16 and 2^-23 in float32, on few elements. Ids, plans, masks and tables are the
    same."""
    if case["dtype"] == "bfloat16":
        return {"rel": 4e-4, "max": 8e-3, "differ": 0.0}
    return {"rel": 1e-7, "max": 1e-6, "differ": 0.0}


# ------------------------------------------------------------------ the same in 64 bits

def _rotated(x, off, base, style):
    """[.., T, d] rows of K re-encoded by offset off, in 64 bits."""
    x = x.double()
    if off == 0:
        return x
    d = x.shape[-1]
    j = torch.arange(d // 2, dtype=torch.float64, device=x.device)
    phi = off * torch.pow(torch.tensor(base, dtype=torch.float64, device=x.device), -2 * j / d)
    c, sn = torch.cos(phi), torch.sin(phi)
    y = torch.empty_like(x)
    if style == "half":
        a, b = x[..., :d // 2], x[..., d // 2:]
        y[..., :d // 2], y[..., d // 2:] = a * c - b * sn, b * c + a * sn
    else:
        a, b = x[..., 0::2], x[..., 1::2]
        y[..., 0::2], y[..., 1::2] = a * c - b * sn, b * c + a * sn
    return y


def exact(case, seed):
    if case["call"] == "ids" or _bytes(case, _ints(case["lengths"])) > 12e9:
        return None
    if case["call"] == "paged" and sum(_ints(case["lengths"])) > 200_000:
        return None     # a loop over the merged blocks
    if case["equal"]:
        return None     # the order of the pair falls to its content addresses
    frags = _fragments(case, seed)
    lengths, layer = _ints(case["lengths"]), case["L"] // 2
    tail = min(lengths)
    key = [float(f[layer][0][0, :, T - tail:].double().norm(dim=-1).sum())
           for f, T in zip(frags, lengths)]
    order = sorted(range(len(frags)), key=lambda i: -key[i])
    offs, at = {}, 0
    for i in order:
        offs[i] = at
        at += lengths[i]
    merged = torch.empty((case["L"], 2, 1, case["H"], at, case["d"]), dtype=torch.float64,
                         device="cuda")
    for i in order:
        rows = slice(offs[i], offs[i] + lengths[i])
        for l, (k, v) in enumerate(frags[i]):
            merged[l, 0, :, :, rows] = _rotated(k, offs[i], case["base"], case["style"])
            merged[l, 1, :, :, rows] = v.double()
    arrivals = _ints(case["arrivals"])
    keys = torch.tensor([key[i] for i in (arrivals if case["call"].startswith("deliveries")
                                          else range(len(frags)))], dtype=torch.float64)
    if case["call"] == "paged":
        return dict(pool=_paged_exact(case, frags, seed, order, offs, merged), k_table=None,
                    v_table=None, digests=None, keys=keys)
    if case["call"] in ("set", "deliveries"):
        out = dict(merged=_layers(merged), keys=keys, plan=None)
    else:
        whole = case["call"] == "set-into" or len(set(arrivals)) == len(arrivals)
        out = dict(merged=merged if whole else merged.view(-1), keys=keys, plan=None)
    if case["call"].startswith("deliveries"):
        out["digests"] = None
    if case["call"] == "deliveries-into":
        out["mask"] = None
    return out


def _paged_exact(case, frags, seed, order, offs, merged):
    """The pool after the merge: block j of the merged cache keeps a fragment's page where all its
    rows are one page of one fragment (V; K only at offset 0), every other takes the next free
    page, K before V."""
    pool, lengths, lists, free = _pages(case, frags, seed)
    pool, B, T_out = pool.double(), case["block"], merged.shape[4]
    taken = 0
    for j in range(-(-T_out // B)):
        r0, r1 = j * B, min(j * B + B, T_out)
        i = max((i for i in order if offs[i] <= r0), key=lambda i: offs[i])
        whole = r1 <= offs[i] + lengths[i] and (r0 - offs[i]) % B == 0
        for kv in (0, 1):
            if whole and (kv == 1 or offs[i] == 0):
                continue
            pool[:, kv, free[taken], :, :r1 - r0] = merged[:, kv, 0, :, r0:r1]
            taken += 1
    return pool
