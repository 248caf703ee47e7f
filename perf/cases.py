"""What a user of the library has it do, as cases whose time can be measured: decodes of a batch of
requests (draft levels plus verification), stand-alone verification of tuples, and the build of an
item set.

Inputs are made on the GPU from a seed: hidden states N(0, 1), weights and code embeddings
N(0, 0.02), catalogs whose first level follows a capped Zipf law, planted with most of the tuples
the head ranks highest, so that about 30 % of the best unverified beams are not items."""
import math

import numpy as np
import torch

import paper_2511_18793_amd as nz

CODE_STD = 0.02
RNN_CODE_STD = 0.5      # embeddings of the recurrent Transition: large enough that tanh bends


def _decode(name, B, radices, K, d, e, items, **more):
    c = {"name": name, "kind": "decode", "B": B, "radices": radices, "K": K, "d": d, "e": e,
         "items": items, "zipf": 1.1, "dtype": "bf16", "call": "plan", "transition": "add",
         "prefix_sets": False}
    c.update(more)
    return c


def listed():
    return [
        # one user waiting for recommendations: the smallest call, all latency
        _decode("one_request", 1, "512,512,512", 10, 1024, 128, 33_614, zipf=0.0),
        # the public-dataset setting in small batches; new tensors on every call, so no kept plan
        _decode("paper_batch", 64, "512,512,512", 10, 1024, 128, 57_288, zipf=0.0, call="decode"),
        # an online server's batch at its usual fill
        _decode("serving", 256, "256,256,256", 20, 512, 128, 1_000_000),
        # the same server with the recurrent Transition and a prefix filter at every level
        _decode("serving_rnn_prefix", 200, "256,256,256", 20, 512, 128, 1_000_000,
                transition="rnn", prefix_sets=True),
        # codebooks of unequal, odd sizes, a batch that fills no tile, a state of unusual width
        _decode("ragged", 333, "1008,656,2032", 37, 736, 96, 3_000_000),
        # four levels, a thousand requests
        _decode("wide", 1024, "1024,1024,1024,1024", 50, 1024, 128, 10_000_000),
        # offline batch scoring at the largest configuration
        _decode("large", 4096, "4096,4096,4096", 100, 2048, 128, 50_000_000),
        # retrieval: few requests, a beam of hundreds
        _decode("recall", 64, "4096,4096,4096", 512, 1024, 128, 20_000_000),
        # a head kept in float32, as a model under evaluation is
        _decode("float32", 48, "256,256,256", 8, 512, 64, 100_000, dtype="f32", call="decode"),
        # drafts of one server batch, checked on their own
        {"name": "verify_batch", "kind": "verify", "n": 5_120, "radices": "256,256,256",
         "items": 1_000_000},
        # a bulk check against the largest catalog
        {"name": "verify_bulk", "kind": "verify", "n": 4_000_000, "radices": "4096,4096,4096",
         "items": 100_000_000},
        # the catalog's daily refresh, from host memory
        {"name": "build", "kind": "build", "radices": "1024,1024,1024,1024", "items": 10_000_000,
         "on_device": False},
    ]


def _log_between(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _radix(rng, lo, hi):
    return max(lo, min(hi, 16 * int(round(_log_between(rng, lo, hi) / 16))))


def draw(rng):
    kind = rng.choices(("decode", "retrieve", "float32", "verify", "build"), (12, 2, 1, 2, 1))[0]
    if kind == "verify":
        V = _radix(rng, 256, 4096)
        return {"kind": "verify", "n": _log_between(rng, 1_000, 4_000_000),
                "radices": ",".join([str(V)] * 3),
                "items": min(_log_between(rng, 10_000, 100_000_000), V ** 3 // 8)}
    if kind == "build":
        V = _radix(rng, 256, 4096)
        return {"kind": "build", "radices": ",".join([str(V)] * rng.choice((3, 4))),
                "items": min(_log_between(rng, 10_000, 10_000_000), V ** 3 // 8),
                "on_device": rng.random() < 0.4}
    L = rng.choice((3, 3, 3, 4))
    if kind == "retrieve":
        # codebooks no smaller than the beam, which is wider than 128
        radices = [_radix(rng, 1024, 4096) for _ in range(L)]
        K = _log_between(rng, 129, 1000)
        d, e = 32 * _log_between(rng, 8, 32), rng.choice((64, 128))
        B = _log_between(rng, 1, 64)
        most = 64 * 512 * 4096 * 2
    elif kind == "float32":
        radices = [_radix(rng, 128, 512)] * 3
        K = _log_between(rng, 4, 20)
        d, e = _log_between(rng, 64, 512), rng.choice((32, 64, 128))
        B = _log_between(rng, 1, 48)
        most = 48 * 8 * 256 * 2
    else:
        if rng.random() < 0.25:
            radices = [_radix(rng, 256, 4096) for _ in range(L)]
        else:
            radices = [_radix(rng, 256, 4096)] * L
        K = _log_between(rng, 5, 128)
        d, e = 32 * _log_between(rng, 8, 64), rng.choice((32, 64, 64, 96, 128, 128, 128, 256))
        B = _log_between(rng, 1, 4096)
        # a state width that is no power of two costs more for each logit
        most = 4096 * 100 * 4096 * 2 // (8 if e == 96 else 2 if e == 256 else 1)
    B = max(1, min(B, most // (K * sum(radices[1:]))))
    size = 1
    for r in radices:
        size *= r
    c = _decode("", B, ",".join(map(str, radices)), K, d, e,
                min(_log_between(rng, 10_000, 50_000_000), size // 8),
                zipf=rng.choice((0.0, 1.1, 1.2)), dtype="f32" if kind == "float32" else "bf16",
                call="decode" if kind == "float32" or rng.random() < 0.3 else "plan",
                transition="rnn" if kind == "decode" and rng.random() < 0.15 else "add",
                prefix_sets=kind == "decode" and rng.random() < 0.15)
    del c["name"]
    return c


def _radices(case):
    return [int(r) for r in case["radices"].split(",")]


def _first_level(V, zipf, items, below):
    """Popularity of the first-level codes: Zipf by rank, but at most half of the tuples that exist
    under a code."""
    p = np.arange(1, V + 1, dtype=np.float64) ** -zipf
    p /= p.sum()
    cap = max(1.0 / V, 0.5 * below / items)
    for _ in range(V):
        over = p >= cap
        if not (p > cap).any():
            break
        p[over] = cap
        p[~over] *= (1.0 - cap * over.sum()) / p[~over].sum()
    return p


def _catalog(radices, items, zipf, gen):
    """int32 [items, L] on the GPU; the few tuples that come twice are stored once by the set."""
    below = 1
    for r in radices[1:]:
        below *= r
    p = torch.from_numpy(_first_level(radices[0], zipf, items, below)).cuda()
    rank = torch.searchsorted(p.cumsum(0), torch.rand(items, generator=gen, device="cuda",
                                                      dtype=torch.float64))
    order = torch.randperm(radices[0], generator=gen, device="cuda").to(torch.int32)
    out = torch.empty((items, len(radices)), dtype=torch.int32, device="cuda")
    out[:, 0] = order[rank.clamp_(max=radices[0] - 1)]
    for l in range(1, len(radices)):
        out[:, l] = torch.randint(radices[l], (items,), generator=gen, device="cuda",
                                  dtype=torch.int32)
    return out


def _likely(H, W, d, K, gen):
    """70 % of the tuples that the head ranks highest for each request, by the part of the logits
    that the state has no share in: int32 [n, L]."""
    B, L = H.shape[:2]
    keep = 2 * K + 16
    score, codes = None, None
    for l in range(L):
        logp = torch.log_softmax(H[:, l].float() @ W[l][:d].float(), dim=1)
        top, code = logp.topk(min(max(K, 16), logp.shape[1]), dim=1)
        if score is None:
            score, codes = top, code.unsqueeze(2)
            continue
        m = top.shape[1]
        both = (score.unsqueeze(2) + top.unsqueeze(1)).reshape(B, -1)
        score, at = both.topk(min(keep, both.shape[1]), dim=1)
        before = torch.div(at, m, rounding_mode="floor")
        codes = torch.cat([codes.gather(1, before.unsqueeze(2).expand(-1, -1, l)),
                           code.gather(1, at % m).unsqueeze(2)], dim=2)
    codes = codes.reshape(-1, L)
    coin = torch.rand(codes.shape[0], generator=gen, device="cuda") < 0.7
    return codes[coin].to(torch.int32)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    radices = _radices(case)
    if case["kind"] == "verify":
        n, items = case["n"], case["items"]
        catalog = _catalog(radices, items, 0.0, gen)
        itemset = nz.build_itemset(catalog, radices)
        # 30 % of the tuples are drawn from the whole space, 70 % are items, popular ones more often
        u = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
        rank = ((u * math.log(items + 1.0)).exp().long() - 1).clamp_(0, items - 1)
        codes = catalog[rank]
        absent = torch.rand(n, generator=gen, device="cuda") < 0.3
        for l, r in enumerate(radices):
            other = torch.randint(r, (n,), generator=gen, device="cuda", dtype=torch.int32)
            codes[:, l] = torch.where(absent, other, codes[:, l])
        return {"kind": "verify", "set": itemset, "codes": codes,
                "mask": torch.zeros(n, dtype=torch.uint8, device="cuda"),
                "index": torch.zeros(n, dtype=torch.int64, device="cuda"),
                "count": torch.zeros(1, dtype=torch.int64, device="cuda"),
                "workspace": torch.empty(max(16, nz.verify_workspace(n)), dtype=torch.uint8,
                                         device="cuda")}
    if case["kind"] == "build":
        catalog = _catalog(radices, case["items"], 1.1, gen)
        queries = _catalog(radices, 65_536, 1.1, gen)
        known = torch.rand(65_536, generator=gen, device="cuda") < 0.5
        some = torch.randint(case["items"], (65_536,), generator=gen, device="cuda")
        queries = torch.where(known.unsqueeze(1), catalog[some], queries)
        return {"kind": "build", "radices": radices, "queries": queries, "set": None,
                "catalog": catalog if case["on_device"] else catalog.cpu().numpy()}

    B, K, d, e, L = case["B"], case["K"], case["d"], case["e"], len(radices)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    rnn = case["transition"] == "rnn"

    def normal(std, *shape):
        return (torch.randn(*shape, generator=gen, device="cuda") * std).to(dt)

    H = normal(1.0, B, L, d)
    W = [normal(0.02, d + e, r) for r in radices]
    E = [normal(RNN_CODE_STD if rnn else CODE_STD, r, e) for r in radices[:-1]]
    U = [normal(1.0 / math.sqrt(e), e, e) for _ in radices[:-1]] if rnn else None
    catalog = _catalog(radices, case["items"], case["zipf"], gen)
    plant = _likely(H, W, d, K, gen)
    n = min(plant.shape[0], case["items"] // 2)
    catalog[:n] = plant[torch.randperm(plant.shape[0], generator=gen, device="cuda")[:n]]
    itemset = nz.build_itemset(catalog, radices)
    prefix_sets = None
    if case["prefix_sets"]:
        prefix_sets = [nz.build_itemset(catalog[:, :l].contiguous(), radices[:l])
                       for l in range(1, L)]
    buffers = nz.DraftBuffers(B, L, K, d, e, radices, dt, torch.device("cuda"))
    if dt == torch.bfloat16:
        W = [nz.pack_weights(l + 1, L, radices, W[l], d) for l in range(L)]
    if case["call"] == "plan":
        return {"kind": "plan", "plan": nz.DecodePlan(H, W, E, radices, K, itemset, buffers=buffers,
                                                      U=U, prefix_sets=prefix_sets)}
    return {"kind": "decode", "args": (H, W, E, radices, K, itemset),
            "more": {"buffers": buffers, "U": U, "prefix_sets": prefix_sets}}


def run(state):
    kind = state["kind"]
    if kind == "verify":
        mask, index, count = nz.verify_tuples(state["set"], state["codes"], state["mask"],
                                              state["index"], state["count"], state["workspace"])
        return {"mask": mask, "index": index, "count": count}
    if kind == "build":
        # the new set replaces the one before it, whose users' work the build has waited for
        fresh = nz.build_itemset(state["catalog"], state["radices"])
        state["set"] = fresh
        info = fresh.info()
        mask, index, count = nz.verify_tuples(fresh, state["queries"], want_index=False)
        return {"mask": mask, "n_distinct": info["n_distinct"], "n_slots": info["n_slots"]}
    if kind == "plan":
        outs = state["plan"].run()
    else:
        outs = nz.decode(*state["args"], **state["more"])
    # every level's beams.  The states between the levels are sums of code embeddings along
    # (parent, code), which come out here; two beams of equal score may stand in either order, which
    # no tolerance on the states themselves could allow for.
    return [{k: o[k] for k in ("key", "score", "parent", "code", "count")} for o in outs]


def work(case):
    radices = _radices(case)
    L = len(radices)
    if case["kind"] == "verify":
        # codes, one key of the table for each tuple, mask, the accepted 70 % of the indices
        return {"bytes": case["n"] * (4 * L + 8 + 1 + 0.7 * 8), "flops": 0}
    if case["kind"] == "build":
        # the tuples once, the keys at load factor 0.5, the prefilter's four bytes per item
        return {"bytes": case["items"] * (4 * L + 16 + 4), "flops": 0}
    B, K, d, e = case["B"], case["K"], case["d"], case["e"]
    size = 2 if case["dtype"] == "bf16" else 4
    total = 0
    flops = 0
    for l, r in enumerate(radices):
        total += B * d * size + (d + e) * r * size + B * K * 20 + B * 4
        flops += 2 * B * d * r
        if l > 0:
            flops += 2 * B * K * e * r
        if l < L - 1:
            total += min(r, B * K) * e * size + B * K * e * size
            if case["transition"] == "rnn":
                total += e * e * size
                flops += 2 * B * K * e * e
        if l == L - 1 or case["prefix_sets"]:
            total += min(16 * case["items"], 8 * B * (K if l > 0 else 1) * K)
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["kind"] != "decode":
        return "exact"
    # float32 scores of magnitude 10 from float32 sums of at most 2176 terms; where two scores agree
    # to that precision the beams may change places, and so do the parents of what comes after them
    return {"rel": 1e-5, "max": 1e-4, "differ": 4e-3}
