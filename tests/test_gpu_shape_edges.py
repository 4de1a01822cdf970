"""GPU parity at the edges where the kernels change shape: attention's token rounds, head blocks,
split cap and single-split output against the float64 oracle, and the tables' recency index read
16 bytes at a time or entry by entry against the canonical LRU.

Attention tolerance: weights rounded to bf16 (relative step 2^-9, one rounding per weight) and
fp32 sums, as for every attention test here: max-abs 1e-2, relative L2 5e-3.
"""
import zlib

import numpy as np
import pytest
import torch

import oracle
import workload as W
from hs_harness import attn_desc, log
from paper_2608_07009_amd import HiSparseCache, hisparse as hs

pytestmark = pytest.mark.gpu

MAX_ABS, REL_L2 = 1e-2, 5e-3
BESIDE = hs.HISPARSE_ATTN_BESIDE_FETCH
CARRY = hs.HISPARSE_ATTN_CARRIES_REPLAY
DEFER = hs.HISPARSE_ATTN_DEFER_MERGE


@pytest.mark.parametrize("kind,H,k,tpr,splits,units,flags", [
    # latent, one round of four 16-head waves (up to 128 tokens) and its far side, one to 16 head
    # blocks, and more of them than CUs left (the tiled kernels, in one split and in two)
    ("mla", 16, 128, 1, 0, 2, 0), ("mla", 1, 127, 1, 0, 1, 0), ("mla", 15, 31, 4, 0, 3, 0),
    ("mla", 16, 32, 4, 0, 2, 0), ("mla", 16, 129, 1, 0, 2, 0), ("mla", 17, 128, 1, 0, 2, 0),
    ("mla", 16, 1, 1, 0, 1, 0), ("mla", 16, 33, 4, 0, 2, 0),
    ("mla", 20, 64, 1, 0, 2, 0), ("mla", 32, 65, 1, 1, 2, 0), ("mla", 33, 63, 1, 0, 2, 0),
    ("mla", 128, 50, 1, 0, 9, BESIDE), ("mla", 72, 64, 1, 1, 2, 0), ("mla", 256, 128, 1, 0, 2, 0),
    ("mla", 241, 32, 4, 0, 15, 0), ("mla", 241, 64, 1, 0, 16, 0), ("mla", 241, 128, 1, 0, 16, 0),
    # latent, a unit of one split: one head wave, two, and two with the query after the first chunk;
    # the same kernels with splits to merge
    ("mla", 20, 129, 1, 1, 2, 0), ("mla", 32, 193, 1, 1, 2, 0), ("mla", 33, 150, 1, 1, 2, 0),
    ("mla", 72, 192, 1, 1, 2, 0), ("mla", 128, 140, 1, 1, 9, BESIDE), ("mla", 128, 200, 1, 0, 9, BESIDE),
    # latent, both sides of four rounds and of eight below 16 workgroup columns, with the replay hint
    ("mla", 32, 256, 1, 0, 5, 0), ("mla", 32, 257, 1, 0, 5, 0), ("mla", 32, 512, 1, 0, 5, 0),
    ("mla", 32, 513, 1, 0, 5, 0), ("mla", 72, 200, 1, 0, 2, 0), ("mla", 100, 1030, 1, 0, 2, CARRY),
    ("mla", 100, 900, 1, 0, 2, CARRY),
    # latent, both sides of the 2048-record split cap, and of the 1024-record one of few columns
    ("mla", 256, 2048, 1, 0, 33, 0), ("mla", 256, 2049, 1, 0, 33, 0), ("mla", 20, 2048, 1, 1, 129, 0),
    ("mla", 20, 2049, 1, 0, 129, 0),
    ("mla", 40, 2048, 1, 1, 1, 0), ("mla", 40, 2049, 1, 1, 1, 0), ("mla", 20, 2048, 1, 1, 1, 0),
    ("mla", 72, 1024, 1, 1, 2, 0), ("mla", 20, 1025, 1, 1, 2, 0),
    # grouped-query, one, two and four head waves: one split (five rounds), and one more
    ("gqa", 4, 640, 1, 0, 2, 0), ("gqa", 4, 641, 1, 0, 2, 0), ("gqa", 16, 40, 16, 0, 2, 0),
    ("gqa", 17, 320, 1, 0, 2, 0), ("gqa", 32, 321, 1, 0, 2, 0), ("gqa", 33, 160, 1, 0, 2, 0),
    ("gqa", 64, 161, 1, 0, 2, 0), ("gqa", 70, 3, 64, 0, 2, 0), ("gqa", 5, 1, 1, 0, 2, 0),
    # grouped-query beside a fetch, six rounds per split: up to five, one split of more, two splits
    ("gqa", 4, 640, 1, 0, 2, BESIDE), ("gqa", 4, 1535, 1, 0, 2, BESIDE), ("gqa", 4, 96, 16, 0, 2, BESIDE),
    ("gqa", 4, 1537, 1, 0, 2, BESIDE), ("gqa", 24, 767, 1, 0, 2, BESIDE), ("gqa", 24, 769, 1, 0, 2, BESIDE),
    ("gqa", 40, 383, 1, 0, 2, BESIDE), ("gqa", 40, 385, 1, 0, 2, BESIDE), ("gqa", 40, 6, 64, 3, 2, BESIDE),
    # grouped-query with the replay hint: three quarters of the CUs, and more
    ("gqa", 4, 2048, 1, 0, 24, CARRY), ("gqa", 4, 2048, 1, 0, 32, CARRY), ("gqa", 16, 1024, 1, 0, 64, CARRY),
    ("gqa", 8, 2048, 1, 1, 1, 0), ("gqa", 8, 2049, 1, 1, 1, 0), ("gqa", 8, 1024, 1, 1, 1, 0),
    ("gqa", 256, 2048, 1, 0, 65, 0), ("gqa", 256, 2049, 1, 0, 65, 0),
])
def test_attention_shape_edges(kind, H, k, tpr, splits, units, flags):
    """Against the oracle, with padding entries and (from two units on) a unit with nothing
    selected; the deferred call and its merge give the same bits as the call by itself."""
    rng = np.random.default_rng(zlib.crc32(f"edge-{kind}-{H}-{k}-{tpr}-{splits}".encode()))
    if kind == "mla":
        d_qk, d_v, voff, te, scale = 576, 512, 0, 576, 1 / np.sqrt(192)
    else:
        d_qk, d_v, voff, te, scale = 128, 128, 128, 256, 1 / np.sqrt(128)
    many = units > 20  # a small pool, records repeated; three of the units against the oracle
    n_rec, R = 300 if many else k + 19, te * tpr * 2
    w = W.workload(1 if kind == "mla" else 3, q_heads=H, k=k, d_qk=d_qk, d_v=d_v, v_offset=voff,
                   tokens_per_record=tpr, record_bytes=R, scale=float(scale))
    bf16 = lambda shape: torch.from_numpy(rng.standard_normal(shape).astype(np.float32)) \
        .to(torch.bfloat16).view(torch.int16)
    pool, q = bf16((units, n_rec, te * tpr)), bf16((units, H, d_qk))
    idx = np.stack([rng.choice(n_rec, size=k, replace=many) for _ in range(units)]).astype(np.int32)
    if k > 4:
        idx[0, k // 3::7] = -1
    if units > 1:
        idx[1, :] = -1
    log(f"test_attention_shape_edges {kind} H={H} k={k} tpr={tpr} splits={splits} units={units}")
    dev = torch.device("cuda:0")
    pool_d, q_d, idx_d = pool.to(dev), q.to(dev), torch.from_numpy(idx).to(dev)
    ad = attn_desc(w, splits, flags)
    n = hs.hisparse_decode_workspace_bytes(units, k, R, ad)
    ws = torch.full((n,), 0xFF, dtype=torch.uint8, device=dev)  # partials never read unwritten
    s = torch.cuda.current_stream()
    out = torch.full((units, H, d_v), float("nan"), dtype=torch.float32, device=dev)
    hs.hisparse_sparse_decode_pool(pool_d, n_rec, R, units, k, q_d, idx_d, out, ad, ws, n, s)
    late = torch.full_like(out, float("nan"))
    add = attn_desc(w, splits, flags | DEFER)
    hs.hisparse_sparse_decode_pool(pool_d, n_rec, R, units, k, q_d, idx_d, late, add, ws, n, s)
    hs.hisparse_attention_merge(units, k, R, add, late, ws, n, s)
    o, l = out.cpu().numpy(), late.cpu().numpy()
    assert o.tobytes() == l.tobytes()
    for u in (0, 1, units - 1) if many else range(units):
        if u == 1:
            assert (o[u] == 0).all()
            continue
        ref = oracle.sparse_decode(q[u].numpy().view(np.uint16), pool[u].numpy().view(np.uint16),
                                   idx[u], d_qk=d_qk, d_v=d_v, v_off=voff, token_elems=te,
                                   tokens_per_record=tpr, scale=w.scale)
        assert np.abs(o[u] - ref).max() <= MAX_ABS
        assert np.linalg.norm(o[u] - ref) <= REL_L2 * np.linalg.norm(ref)


@pytest.mark.parametrize("B,k", [(1, 1), (3, 2), (4, 4), (7, 5), (63, 31), (64, 64), (66, 40),
                                 (255, 100), (256, 128), (257, 60), (260, 256), (1000, 513),
                                 (1023, 700), (1024, 512), (1025, 300), (4094, 2048),
                                 (4096, 4096), (4097, 1500), (4100, 2000), (8191, 3000),
                                 (16384, 4096)])
def test_tables_recency_index_edges(B, k):
    """Resolves of drifting selections and one-position admissions in turn, at capacities on both
    sides of every change in how the recency index is read (16 bytes or one entry at a time, 4 or
    16 entries per thread, one or several admission batches): slots, counts, state and recency
    index as the canonical LRU gives them, for three units."""
    U, G, L = 3, 2, 3 * B + k + 40
    rng = np.random.default_rng(B * 7 + k)
    log(f"test_tables_recency_index_edges B={B} k={k}")
    cache = HiSparseCache(num_requests=U, num_layers=G, units_per_request=1, capacity=B,
                          num_records=L, top_k=k, record_bytes=48, share_group=G)
    try:
        dev = torch.device("cuda:0")
        for layer in range(G):
            cache.host_view(layer)[:] = 0
        slots = torch.empty((U, k), dtype=torch.int32, device=dev)
        counts = torch.empty((U, 2), dtype=torch.int32, device=dev)
        new_slots = torch.empty((1, U), dtype=torch.int32, device=dev)
        orc = oracle.OracleCache(U, L, B, k)
        s = torch.cuda.current_stream()
        sel = np.stack([rng.choice(L, size=k, replace=False) for _ in range(U)]).astype(np.int32)
        for t in range(6):
            for u in range(U):  # a fifth of the entries change; unit 2 pads its tail
                fresh = np.setdiff1d(np.arange(L), sel[u])
                at = rng.choice(k, size=max(1, k // 5), replace=False)
                sel[u, at] = rng.choice(fresh, size=len(at), replace=False)
            step = sel.copy()
            step[2, k - k // 4:] = -1
            hs.hisparse_resolve(cache.handle, 0, torch.from_numpy(step).to(dev), slots, counts, s)
            e_slots, e_counts, _, _, bad = orc.resolve(step)
            assert bad == 0
            assert (slots.cpu().numpy() == e_slots).all(), f"slots, step {t}"
            assert (counts.cpu().numpy() == e_counts).all(), f"counts, step {t}"
            # a resident position, a new one, and none
            pos = np.array([step[0, 0], rng.integers(L), -1], dtype=np.int32)
            rec = torch.full((G, U, 24), t + 1, dtype=torch.int16, device=dev)
            hs.hisparse_append(cache.handle, 0, G, torch.from_numpy(pos).to(dev), rec, new_slots, s)
            got = new_slots.cpu().numpy()[0]
            for u in range(2):
                rc, slot, _ = orc.admit_unit(u, int(pos[u]))
                assert rc == oracle.OK and got[u] == slot, f"admission, step {t} unit {u}"
                for layer in range(G):
                    host = cache.host_view(layer)[u, pos[u]].view(np.int16)
                    assert (host == t + 1).all(), f"write-through, step {t} unit {u} layer {layer}"
            assert got[2] == -1
            orc.clock[2] += 1
        st = cache.read_state(0)
        assert (st["slot_pos"] == orc.slot_pos).all() and (st["slot_ts"] == orc.slot_ts).all()
        assert (st["clock"] == orc.clock).all() and (st["page_table"] == orc.pt).all()
        order = np.stack([np.lexsort((np.arange(B), ts)) for ts in orc.slot_ts])
        assert (st["order"] == order).all()
        assert cache.check_errors()[0] == hs.HISPARSE_OK
    finally:
        torch.cuda.synchronize()
        cache.close()


def _score_case(kind, H, k, units, rng, key, query):
    """Inputs whose scores are products of two bf16 numbers, exact in fp32: one key dimension (of
    latent records one outside the values) holds key [units][k], the query there query [H]."""
    mla = kind == "mla"
    d_qk, d_v, voff, te = (576, 512, 0, 576) if mla else (128, 128, 128, 256)
    R, scale = te * 2, float(1 / np.sqrt(192 if mla else 128))
    w = W.workload(1 if mla else 3, q_heads=H, k=k, d_qk=d_qk, d_v=d_v, v_offset=voff,
                   tokens_per_record=1, record_bytes=R, scale=scale)
    pool = rng.standard_normal((units, k, te)).astype(np.float32)
    q = np.zeros((units, H, d_qk), np.float32)
    pool[:, :, d_qk - 1], q[:, :, d_qk - 1] = key, query
    bf16 = lambda a: torch.from_numpy(a).to(torch.bfloat16).view(torch.int16)
    idx = np.stack([rng.permutation(k) for _ in range(units)]).astype(np.int32)
    return w, bf16(pool), bf16(q), idx


def _pool_call(w, pool, q, idx, splits, flags, units):
    dev = torch.device("cuda:0")
    ad = attn_desc(w, splits, flags)
    n = hs.hisparse_decode_workspace_bytes(units, w.k, w.record_bytes, ad)
    ws = torch.full((n,), 0xFF, dtype=torch.uint8, device=dev)
    out = torch.full((units, w.q_heads, w.d_v), 7.0, dtype=torch.float32, device=dev)
    hs.hisparse_sparse_decode_pool(pool.to(dev), pool.shape[1], w.record_bytes, units, w.k,
                                   q.to(dev), torch.from_numpy(idx).to(dev), out, ad, ws, n,
                                   torch.cuda.current_stream())
    return out.cpu().numpy()


@pytest.mark.parametrize("kind,H,k,splits,units,flags,level", [
    # no later chunk beats its token group's first: 16-head kernel, one and two head waves written
    # directly, merged, and with the query after the first chunk
    ("mla", 16, 128, 0, 2, 0, True), ("mla", 100, 128, 0, 2, 0, True), ("mla", 20, 200, 1, 2, 0, True),
    ("mla", 72, 200, 1, 2, 0, True), ("mla", 24, 300, 2, 2, 0, True), ("mla", 72, 300, 2, 2, 0, True),
    ("mla", 128, 140, 1, 9, BESIDE, True), ("mla", 128, 270, 2, 9, BESIDE, True),
    # scores outgrow the reference (exact fallback; the moving reference)
    ("mla", 20, 200, 1, 2, 0, False), ("mla", 72, 300, 2, 2, 0, False), ("gqa", 4, 600, 1, 2, 0, False),
    ("gqa", 24, 300, 2, 2, 0, False), ("gqa", 64, 200, 0, 2, 0, False),
])
def test_attention_huge_scores(kind, H, k, splits, units, flags, level):
    """Scores of 2^34 and more (in powers of two), 2^27 and more apart: the softmax is one
    record. fp32 holds such a score to about 2^10, so a weight taken from an unrounded product
    against a rounded reference would be 0 or infinite; every value out is that record's, exactly."""
    rng = np.random.default_rng(zlib.crc32(f"huge-{kind}-{H}-{k}-{splits}".encode()))
    log(f"test_attention_huge_scores {kind} H={H} k={k} splits={splits} units={units} level={level}")
    # k distinct bf16 numbers, neighbours 2^14 apart or more
    steps = np.concatenate([np.arange(1, 257), *(np.arange(130, 257, 2) * 2.0 ** e for e in range(7))])
    key = np.stack([rng.permutation(np.unique(steps)[:k]) for _ in range(units)]) * 2.0 ** 14
    query = rng.integers(128, 256, H) * 2.0 ** 10 * rng.choice((-1, 1), H)
    w, pool, q, idx = _score_case(kind, H, k, units, rng, key, query)
    assert len(np.unique(pool[0, :, w.d_qk - 1])) == k
    if level:  # each group's extreme records first: its chunks are every other 32 of its split
        split = -(-(-(-k // max(splits, 1))) // 64) * 64
        for u in range(units):
            for tokens in (np.arange(k)[(np.arange(k) // split == s) & (np.arange(k) // 32 % 2 == g)]
                           for s in range(-(-k // split)) for g in (0, 1)):
                for place, extreme in enumerate((np.argmax, np.argmin)[:len(tokens)]):
                    rest = tokens[place:]
                    at = rest[extreme(key[u, idx[u, rest]])]
                    idx[u, [rest[0], at]] = idx[u, [at, rest[0]]]
    out = _pool_call(w, pool, q, idx, splits, flags, units)
    v = pool.view(torch.bfloat16).float().numpy()[:, :, w.v_offset:w.v_offset + w.d_v]
    for u in range(units):
        best = np.where(query > 0, key[u].argmax(), key[u].argmin())
        assert (out[u] == v[u, best]).all(), f"unit {u}"


@pytest.mark.parametrize("kind,H,k,splits,units,flags", [
    ("mla", 16, 100, 0, 1, 0), ("mla", 20, 150, 1, 2, 0), ("mla", 24, 300, 0, 2, 0),
    ("mla", 72, 200, 0, 2, 0), ("mla", 72, 150, 1, 2, 0), ("mla", 128, 140, 1, 9, BESIDE),
    ("gqa", 24, 300, 2, 2, 0),
])
@pytest.mark.parametrize("offset", [1, 4])
def test_attention_query_at_any_element(kind, H, k, splits, units, flags, offset):
    """A query that starts 2 or 8 bytes off a 16-byte boundary gives the bits of an aligned one."""
    rng = np.random.default_rng(zlib.crc32(f"offset-{kind}-{H}-{k}".encode()))
    log(f"test_attention_query_at_any_element {kind} H={H} k={k} units={units} offset={offset}")
    key, query = rng.standard_normal((units, k)), rng.standard_normal(H)
    w, pool, q, idx = _score_case(kind, H, k, units, rng, key, query)
    q = torch.from_numpy(rng.standard_normal(tuple(q.shape)).astype(np.float32)) \
        .to(torch.bfloat16).view(torch.int16).to("cuda:0")
    room = torch.zeros(q.numel() + 8, dtype=torch.int16, device="cuda:0")
    moved = room[offset:offset + q.numel()].view(q.shape).copy_(q)
    assert q.data_ptr() % 16 == 0 and moved.data_ptr() % 16 == 2 * offset
    aligned = _pool_call(w, pool, q, idx, splits, flags, units)
    assert np.isfinite(aligned).all() and np.abs(aligned).max() > 0
    assert _pool_call(w, pool, moved, idx, splits, flags, units).tobytes() == aligned.tobytes()


@pytest.mark.parametrize("kind,H,k,most,units", [("mla", 65, 448, 3, 2), ("mla", 128, 300, 90, 60),
                                                 ("gqa", 4, 1712, 95, 47)])
def test_attention_workspace_of_a_larger_batch(kind, H, k, most, units):
    """A workspace sized for `most` units serves `units`, whose own need is larger."""
    rng = np.random.default_rng(zlib.crc32(f"workspace-{kind}-{H}-{k}".encode()))
    log(f"test_attention_workspace_of_a_larger_batch {kind} H={H} k={k} {most} -> {units}")
    key, query = rng.standard_normal((units, k)), rng.standard_normal(H)
    w, pool, q, idx = _score_case(kind, H, k, units, rng, key, query)
    ad, dev = attn_desc(w), torch.device("cuda:0")
    n = hs.hisparse_decode_workspace_bytes(most, k, w.record_bytes, ad)
    ws = torch.full((n + 256,), 0xFF, dtype=torch.uint8, device=dev)
    out = torch.empty((units, H, w.d_v), dtype=torch.float32, device=dev)
    hs.hisparse_sparse_decode_pool(pool.to(dev), k, w.record_bytes, units, k, q.to(dev),
                                   torch.from_numpy(idx).to(dev), out, ad, ws, n,
                                   torch.cuda.current_stream())
    assert out.cpu().numpy().tobytes() == _pool_call(w, pool, q, idx, 0, 0, units).tobytes()
    assert (ws[n:] == 0xFF).all()
