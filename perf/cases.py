"""Performance cases of the HiSparse decode path: what a serving program asks of the library.

Three kinds of case:
  attention  one sparse decode attention call over a resident record pool
             (hisparse_sparse_decode_pool), latent (MLA) or grouped-query (GQA) records
  tables     the metadata phases of one layer's resolve (hisparse_resolve_tables)
  step       one layer's decode step on a live cache: write-through of the new record, resolve
             with the miss fetch from the host pool, attention (hisparse_append,
             hisparse_resolve, hisparse_sparse_decode or its workspace-free form); with
             layers > 1 the layers of one share group, each attention launch carrying the
             replay of the anchor's miss plan into the next layer's cache

A step's state is a decode loop in progress: its selections drift over a cycle of STEPS steps
(about 14% of each step's entries miss a cache of twice the selection's size), and every pass
takes the next step of the cycle.
"""
import math

import torch

from paper_2608_07009_amd import HiSparseCache, hisparse as hs

STEPS = 32      # selections of a state's cycle
WINDOW = 16     # newest positions that every step of the cycle selects
MISS = 0.14     # the share of a step's entries that miss, about (for work() alone)

MLA = {"d_qk": 576, "d_v": 512, "v_offset": 0, "elems": 576, "scale": 1.0 / math.sqrt(192.0)}
GQA = {"d_qk": 128, "d_v": 128, "v_offset": 128, "elems": 256, "scale": 1.0 / math.sqrt(128.0)}


def _attention(name, form, units, heads, k, records, tokens=1, pad=0):
    """pad: trailing entries of each unit's selection that are padding (shorter contexts)."""
    return {"name": name, "kind": "attention", "form": form, "units": units, "heads": heads,
            "k": k, "records": records, "tokens": tokens, "pad": pad}


def _step(name, units, heads, k, capacity, context, layers=1, workspace=True):
    return {"name": name, "kind": "step", "form": "mla", "units": units, "heads": heads, "k": k,
            "capacity": capacity, "context": context, "tokens": 1, "layers": layers,
            "workspace": workspace}


def _tables(name, units, k, capacity, context):
    return {"name": name, "kind": "tables", "form": "mla", "units": units, "heads": 1, "k": k,
            "capacity": capacity, "context": context, "tokens": 1}


def listed():
    return [
        # The smallest decode step: one short request on a small model, all launches and latency.
        _step("tiny_step", 1, 16, 128, 512, 4096, workspace=False),
        # The DSA/MLA layer step of a full batch: 32 requests at 32K context, top-2048 tokens.
        _step("layer_step", 32, 128, 2048, 4096, 32768),
        # Long contexts whose layers share one indexer's selection in groups of four.
        _step("share_group_step", 2, 128, 2048, 4096, 131072, layers=4),
        # The resolve's table work alone, as a scheduler that splits resolve and fetch calls it.
        _tables("resolve_tables", 16, 2048, 4096, 32768),
        # Latent attention of one request (single-user decoding), 128 heads over top-2048.
        _attention("mla_one_request", "mla", 1, 128, 2048, 4096),
        # A micro-batch of 16 requests: half of the full batch.
        _attention("mla_micro_batch", "mla", 16, 128, 2048, 4096),
        # A large decode batch: the largest latent call.
        _attention("mla_large_batch", "mla", 96, 128, 2048, 4096),
        # One rank of eight-way tensor parallelism: 16 of the 128 heads, all 64 requests.
        _attention("mla_head_shard", "mla", 64, 16, 2048, 4096),
        # Odd everything: 5 requests, 72 heads, a selection that no tile divides, padded.
        _attention("mla_ragged", "mla", 5, 72, 1337, 3000, pad=61),
        # NSA-style block selection: 16 requests x 4 kv heads, 24 blocks of 64 tokens.
        _attention("gqa_blocks", "gqa", 64, 16, 24, 48, tokens=64),
        # Quest page selection: 8 requests x 8 kv heads, 256 pages of 16 tokens.
        _attention("gqa_pages", "gqa", 64, 4, 256, 384, tokens=16),
        # A few units of token-level grouped-query records, ragged and padded.
        _attention("gqa_ragged", "gqa", 11, 7, 501, 900, pad=37),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("mla", "mla", "mla", "gqa", "gqa", "gqa", "step", "step", "group", "tables"))
    if kind == "mla":
        units, heads = _log(rng, 1, 96), rng.choice((16, 32, 64, 128, rng.randint(5, 128)))
        k = _log(rng, 128, 2048)
        pad = rng.choice((0, 0, rng.randint(1, k // 8)))
        c = _attention("", "mla", units, heads, k, 2 * k, pad=pad)
    elif kind == "gqa":
        tokens = rng.choice((1, 16, 64))
        units, heads = _log(rng, 1, 64), rng.choice((4, 8, 16, rng.randint(1, 32)))
        k = max(4, _log(rng, 128, 4096) // tokens)
        pad = rng.choice((0, 0, rng.randint(1, max(1, k // 8))))
        c = _attention("", "gqa", units, heads, k, k + k // 2, tokens=tokens, pad=pad)
    elif kind == "step":
        units, k = _log(rng, 1, 32), _log(rng, 128, 2048)
        c = _step("", units, rng.choice((16, 64, 128, rng.randint(5, 128))), k, 2 * k,
                  rng.choice((16, 20)) * k)
    elif kind == "group":
        units, k = rng.randint(1, 3), _log(rng, 512, 2048)
        c = _step("", units, rng.choice((16, 64, 128)), k, 2 * k, 32 * k, layers=4)
    else:
        k = _log(rng, 24, 2048)
        c = _tables("", _log(rng, 1, 64), k, 2 * k, 16 * k)
    del c["name"]
    return c


def _form(case):
    return MLA if case["form"] == "mla" else GQA


def _randn(seed, salt, shape):
    g = torch.Generator(device="cuda").manual_seed(seed * 64 + salt)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def _record_elems(case):
    return _form(case)["elems"] * case["tokens"]


def _query(case, seed):
    layers = case.get("layers", 1)
    return _randn(seed, 1, (layers * case["units"], case["heads"], _form(case)["d_qk"]))


def _desc(case, flags=0):
    f = _form(case)
    return hs.AttnDesc(case["heads"], f["d_qk"], f["d_v"], f["v_offset"], case["tokens"], 0,
                       f["scale"], flags)


# -- attention over a resident pool ---------------------------------------------------------

def _pool(case, seed):
    return _randn(seed, 2, (case["units"], case["records"], _record_elems(case)))


def _indices(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed * 64 + 3)
    u = torch.rand((case["units"], case["records"]), generator=g, device="cuda")
    idx = torch.sort(u, dim=1, stable=True)[1][:, :case["k"]].to(torch.int32).contiguous()
    if case["pad"]:
        idx[:, case["k"] - case["pad"]:] = -1
    return idx


# -- a live cache ---------------------------------------------------------------------------

def _host_records(case, seed, layer):
    return _randn(seed, 8 + layer, (case["units"], case["context"], _record_elems(case)))


def _new_records(case, seed):
    """The record that each step of the cycle appends, per layer and unit."""
    return _randn(seed, 4, (STEPS, case["layers"], case["units"], _record_elems(case)))


def _positions():
    """The position that each step appends, counted from the end of the context."""
    return [t - STEPS for t in range(STEPS)]


def _selections(case, seed):
    """int32 [STEPS][units][k]: the top k of scores that drift around a cycle (a static part and
    a rotating one), the newest WINDOW positions always among them, none beyond the newest."""
    U, L, k = case["units"], case["context"], case["k"]
    g = torch.Generator(device="cuda").manual_seed(seed * 64 + 5)
    static, x, y = (torch.randn((U, L), generator=g, device="cuda") for _ in range(3))
    out = torch.empty((STEPS, U, k), dtype=torch.int32, device="cuda")
    for t in range(STEPS):
        a = 2.0 * math.pi * t / STEPS
        s = 0.5 * static + math.cos(a) * x + math.sin(a) * y
        end = L + _positions()[t] + 1
        s[:, max(0, end - WINDOW):end] += 100.0
        s[:, end:] = -1000.0
        out[t] = torch.sort(s, dim=1, descending=True, stable=True)[1][:, :k]
    return out


class _Device:
    """Device memory that the library owns, for torch.as_tensor."""

    def __init__(self, ptr, shape):
        self.__cuda_array_interface__ = {"shape": shape, "typestr": "<i4", "data": (ptr, False),
                                         "strides": None, "version": 2}


def _cache_view(cache, layer, shape):
    """A tensor view of a layer's GPU cache; it keeps the cache alive."""
    view = torch.as_tensor(_Device(cache.layer_cache(layer)[0], shape), device="cuda")
    view.owner = cache
    return view


def _cache(case):
    layers = case.get("layers", 1)
    return HiSparseCache(num_requests=case["units"], num_layers=layers, units_per_request=1,
                         capacity=case["capacity"], num_records=case["context"],
                         top_k=case["k"], record_bytes=2 * _record_elems(case),
                         share_group=layers)


def prepare(case, seed):
    dev, U, k = "cuda", case["units"], case["k"]
    f = _form(case)
    s = {"case": case, "t": 0}
    if case["kind"] == "attention":
        s["q"], s["pool"], s["idx"] = _query(case, seed), _pool(case, seed), _indices(case, seed)
        s["desc"] = _desc(case)
        s["out"] = torch.empty((U, case["heads"], f["d_v"]), dtype=torch.float32, device=dev)
        s["ws"] = torch.empty(hs.hisparse_decode_workspace_bytes(
            U, k, 2 * _record_elems(case), s["desc"]), dtype=torch.uint8, device=dev)
        return s
    s["cache"] = cache = _cache(case)
    stream = torch.cuda.current_stream()
    s["sel"] = _selections(case, seed)
    s["slots"] = torch.empty((U, k), dtype=torch.int32, device=dev)
    s["counts"] = torch.empty((U, 2), dtype=torch.int32, device=dev)
    if case["kind"] == "tables":
        for t in range(STEPS):  # a loop in progress: the cache holds the last steps' records
            hs.hisparse_resolve_tables(cache.handle, 0, s["sel"][t], s["slots"], s["counts"],
                                       stream)
        return s
    layers = case["layers"]
    for l in range(layers):
        kv = _host_records(case, seed, l)
        hs.hisparse_stage(cache.handle, l, 1, 0, U, 0, case["context"], kv, 0, stream)
        torch.cuda.synchronize()
        del kv
    s["q"] = _query(case, seed).view(layers, U, case["heads"], f["d_qk"])
    s["out"] = torch.empty((layers, U, case["heads"], f["d_v"]), dtype=torch.float32, device=dev)
    s["new"] = _new_records(case, seed)
    s["pos"] = [torch.full((U,), case["context"] + p, dtype=torch.int32, device=dev)
                for p in _positions()]
    s["new_slots"] = torch.empty((1, U), dtype=torch.int32, device=dev)
    s["desc"] = _desc(case)
    s["carry"] = _desc(case, hs.HISPARSE_ATTN_CARRIES_REPLAY)
    if case["workspace"]:
        n = max(hs.hisparse_decode_workspace_bytes(U, k, cache.R, d)
                for d in (s["desc"], s["carry"]))
        s["ws"] = torch.empty(n, dtype=torch.uint8, device=dev)
    s["records"] = [_cache_view(cache, l, (U, case["capacity"], cache.R // 4))
                    for l in range(layers)]
    for t in range(STEPS):  # a loop in progress: the cache holds the last steps' records
        hs.hisparse_resolve(cache.handle, 0, s["sel"][t], s["slots"], s["counts"], stream)
        if layers > 1:
            hs.hisparse_prefetch_layers(cache.handle, 0, 1, layers - 1, stream)
    return s


def run(s):
    case, stream = s["case"], torch.cuda.current_stream()
    if case["kind"] == "attention":
        hs.hisparse_sparse_decode_pool(s["pool"], case["records"], 2 * _record_elems(case),
                                       case["units"], case["k"], s["q"], s["idx"], s["out"],
                                       s["desc"], s["ws"], s["ws"].numel(), stream)
        return {"out": s["out"]}
    t = s["t"]
    s["t"] = (t + 1) % STEPS
    h = s["cache"].handle
    if case["kind"] == "tables":
        hs.hisparse_resolve_tables(h, 0, s["sel"][t], s["slots"], s["counts"], stream)
        return {"slots": s["slots"], "counts": s["counts"]}
    layers = case["layers"]
    hs.hisparse_append(h, 0, layers, s["pos"][t], s["new"][t], s["new_slots"], stream)
    hs.hisparse_resolve(h, 0, s["sel"][t], s["slots"], s["counts"], stream)
    if not case["workspace"]:
        hs.hisparse_sparse_decode_noalloc(h, 0, s["q"][0], s["slots"], s["out"][0], s["desc"],
                                          stream)
    else:
        ws, n = s["ws"], s["ws"].numel()
        for l in range(layers - 1):
            hs.hisparse_sparse_decode_prefetch(h, l, s["q"][l], s["slots"], s["out"][l],
                                               s["carry"], ws, n, 0, l + 1, 1, stream)
        hs.hisparse_sparse_decode(h, layers - 1, s["q"][layers - 1], s["slots"],
                                  s["out"][layers - 1], s["desc"], ws, n, stream)
    return {"new_slots": s["new_slots"], "slots": s["slots"], "counts": s["counts"],
            "out": s["out"], "records": s["records"]}


def work(case):
    f, U, k = _form(case), case["units"], case["k"]
    R, layers = 2 * _record_elems(case), case.get("layers", 1)
    tables = U * (8 * k + 8 + 8 * case.get("capacity", 0))  # selection, slots, recency index
    if case["kind"] == "tables":
        return {"bytes": tables, "flops": 0}
    n = k - case.get("pad", 0)
    attn = U * (n * R + 4 * k + case["heads"] * (2 * f["d_qk"] + 4 * f["d_v"]))
    flops = 2 * U * case["heads"] * n * case["tokens"] * (f["d_qk"] + f["d_v"])
    if case["kind"] == "attention":
        return {"bytes": attn, "flops": flops}
    # misses: read from the host pool, written to the cache; the new record: read, written twice
    moved = U * R * (2 * MISS * k + 3)
    return {"bytes": tables + layers * (attn + moved), "flops": layers * flops}


def tolerance(case):
    if case["kind"] == "tables":
        return "exact"
    # attention: weights rounded to bf16, sums in fp32 (about four times the distance from
    # exact(), 0.0008 to 0.0016 over these shapes); tables and records are whole numbers
    return {"rel": 0.006}


def _softmax_attention(case, q, kv):
    """float64 attention of one unit: q [heads][d_qk], kv [tokens][elems]."""
    f = _form(case)
    kv = kv.double()
    keys = kv[:, :f["d_qk"]].t().contiguous()
    values = kv[:, f["v_offset"]:f["v_offset"] + f["d_v"]].contiguous()
    p = torch.softmax(q.double() @ keys * f["scale"], dim=1)
    return p @ values


def exact(case, seed):
    if case["kind"] == "tables":
        return None
    f, U, E = _form(case), case["units"], _form(case)["elems"]
    q = _query(case, seed)
    if case["kind"] == "attention":
        pool, idx = _pool(case, seed), _indices(case, seed)
        out = [_softmax_attention(case, q[u], pool[u, idx[u, :case["k"] - case["pad"]].long()]
                                  .reshape(-1, E)) for u in range(U)]
        return {"out": torch.stack(out)}
    layers = case["layers"]
    sel, new = _selections(case, seed)[0].long(), _new_records(case, seed)[0]
    out = torch.empty((layers, U, case["heads"], f["d_v"]), dtype=torch.float64, device="cuda")
    for l in range(layers):
        kv = _host_records(case, seed, l)
        kv[:, case["context"] + _positions()[0]] = new[l]
        for u in range(U):
            out[l, u] = _softmax_attention(case, q[l * U + u], kv[u, sel[u]].reshape(-1, E))
        del kv
    return {"new_slots": None, "slots": None, "counts": None, "out": out,
            "records": [None] * layers}
