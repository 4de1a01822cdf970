"""GPU parity of sparse decode attention.

* Placement independence (Section 3.1): attention over the GPU cache through the resolve
  step's slots is bit-identical to the same kernel over a fully resident copy of the KV
  addressed by positions.
* Accuracy: within max-abs 1e-2 and relative-L2 5e-3 of the oracle's float64 attention.
  The kernel rounds q, K, V to bf16 inputs exactly as given (they are bf16 already) and rounds
  the softmax weights P to bf16 before the PV contraction; everything else accumulates in
  fp32, so errors stay near bf16's 2^-9 relative step on P.
"""
import zlib

import numpy as np
import pytest
import torch

import oracle
import workload as W
from hs_harness import Run, attn_desc, log
from paper_2608_07009_amd import hisparse as hs

pytestmark = pytest.mark.gpu

MAX_ABS, REL_L2 = 1e-2, 5e-3


def rel_l2(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


def decode(run, layer, q_dev, slots, ws, flags=0):
    w = run.w
    out = torch.empty((w.units, w.q_heads, w.d_v), dtype=torch.float32, device=run.dev)
    hs.hisparse_sparse_decode(run.cache.handle, layer, q_dev, slots, out,
                              attn_desc(w, 0, flags), ws, ws.numel(), run.stream)
    return out


def decode_pool(pool_dev, rec_per_unit, w, q_dev, idx_dev, ws, num_splits=0, units=None,
                flags=0):
    units = w.units if units is None else units
    out = torch.empty((units, w.q_heads, w.d_v), dtype=torch.float32, device=pool_dev.device)
    hs.hisparse_sparse_decode_pool(pool_dev, rec_per_unit, w.record_bytes, units, w.k, q_dev,
                                   idx_dev, out, attn_desc(w, num_splits, flags), ws, ws.numel(),
                                   torch.cuda.current_stream())
    return out


def oracle_unit(w, q_host_u, pool_u_u16, idx):
    return oracle.sparse_decode(q_host_u, pool_u_u16, idx, d_qk=w.d_qk, d_v=w.d_v,
                                v_off=w.v_offset, token_elems=w.token_elems,
                                tokens_per_record=w.tokens_per_record, scale=w.scale)


SAMPLE_UNITS = {1: [0], 2: [0, 17, 31], 3: [0, 29, 63], 4: [0, 40, 63], 5: [0]}
STEPS = {1: 12, 2: 3, 3: 6, 4: 4, 5: 3}


BESIDE = hs.HISPARSE_ATTN_BESIDE_FETCH
CARRY = hs.HISPARSE_ATTN_CARRIES_REPLAY


@pytest.mark.parametrize("cfg,flags", [(1, 0), (2, 0), (2, BESIDE), (3, 0), (3, BESIDE), (4, 0),
                                       (4, BESIDE), (5, 0), (5, BESIDE), (5, CARRY)])
def test_attention_cache_vs_resident_vs_oracle(cfg, flags):
    """The default plan, the beside-fetch hint's (latent: half the workgroups; grouped-query: six
    rounds per split) and, for one request, the carries-replay hint's (4-chunk splits)."""
    steps = STEPS[cfg]
    w = W.fit_pinned(W.workload(cfg))
    layer = w.anchors[-1]
    log(f"test_attention cfg={cfg} flags={flags} {w.name} layer={layer} steps={steps}")
    run = Run(w, steps, layers_to_fill=[layer])
    try:
        host = run.cache.host_view(layer)                   # [U][L][R] pinned
        resident = torch.from_numpy(host.reshape(-1)).to(run.dev)  # full KV on the device
        ws_bytes = hs.hisparse_decode_workspace_bytes(w.units, w.k, w.record_bytes,
                                                      attn_desc(w, 0, flags))
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device=run.dev)
        a = layer // w.share_group
        for t in range(steps):
            run.resolve_step(t)
            q_host = W.queries(w, t, layer)
            q_dev = torch.from_numpy(q_host.view(np.int16)).to(run.dev)
            sel_dev = run.sel[t, a * w.units:(a + 1) * w.units]
            out_cache = decode(run, layer, q_dev, run.slots[layer], ws, flags)
            out_res = decode_pool(resident, w.L, w, q_dev, sel_dev, ws, flags=flags)
            torch.cuda.synchronize()
            assert torch.equal(out_cache, out_res), f"placement changed the output at step {t}"
            if t in (0, steps - 1):
                o = out_cache.cpu().numpy()
                for u in SAMPLE_UNITS[cfg]:
                    pool_u = host[u].view(np.uint16).reshape(w.L, -1)
                    ref = oracle_unit(w, q_host[u], pool_u, run.sel_host[t, a * w.units + u])
                    err = np.abs(o[u] - ref).max()
                    rl2 = rel_l2(o[u], ref)
                    log(f"  step {t} unit {u}: max-abs {err:.2e} rel-L2 {rl2:.2e}")
                    assert err <= MAX_ABS and rl2 <= REL_L2
    finally:
        run.close()


def _bf16(rng, shape):
    t = torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(torch.bfloat16)
    return t.view(torch.int16).numpy().view(np.uint16)


@pytest.mark.parametrize("kind,H,k,tpr,splits,units", [
    ("mla", 16, 37, 1, 0, 3), ("mla", 128, 77, 1, 3, 3), ("mla", 40, 300, 1, 0, 3),
    ("mla", 1, 5, 1, 0, 3),
    # latent, 16 or more workgroup columns
    ("mla", 128, 301, 1, 0, 8), ("mla", 200, 97, 1, 3, 6), ("mla", 128, 64, 1, 0, 9),
    ("gqa", 4, 9, 16, 0, 3), ("gqa", 16, 3, 64, 2, 3), ("gqa", 24, 50, 1, 0, 3),
    ("gqa", 64, 13, 4, 1, 3),
])
def test_attention_ragged_and_padding(kind, H, k, tpr, splits, units):
    """Ragged token counts (not multiples of the 32-token chunk), padding entries, a unit with
    no valid record, head counts that are not multiples of 16, explicit split counts."""
    rng = np.random.default_rng(zlib.crc32(f"{kind}-{H}-{k}-{tpr}".encode()))
    if kind == "mla":
        d_qk, d_v, voff, te, scale = 576, 512, 0, 576, 1 / np.sqrt(192)
    else:
        d_qk, d_v, voff, te, scale = 128, 128, 128, 256, 1 / np.sqrt(128)
    n_rec = max(97, k + 40)
    R = te * tpr * 2
    w = W.workload(1 if kind == "mla" else 3, q_heads=H, k=k, d_qk=d_qk, d_v=d_v, v_offset=voff,
                   tokens_per_record=tpr, record_bytes=R, scale=float(scale))
    pool = _bf16(rng, (units, n_rec, te * tpr))
    q = _bf16(rng, (units, H, d_qk))
    idx = np.stack([rng.choice(n_rec, size=k, replace=False) for _ in range(units)]).astype(np.int32)
    idx[0, ::3] = -1          # padding entries
    idx[2, :] = -1            # a unit with nothing selected
    dev = torch.device("cuda:0")
    pool_d = torch.from_numpy(pool.view(np.int16)).to(dev)
    q_d = torch.from_numpy(q.view(np.int16)).to(dev)
    idx_d = torch.from_numpy(idx).to(dev)
    ad = attn_desc(w, splits)
    ws = torch.empty(hs.hisparse_decode_workspace_bytes(units, k, R, ad), dtype=torch.uint8,
                     device=dev)
    out = decode_pool(pool_d, n_rec, w, q_d, idx_d, ws, splits, units=units).cpu().numpy()
    for u in range(units):
        ref = oracle_unit(w, q[u], pool[u], idx[u])
        if u == 2:
            assert (out[u] == 0).all()
            continue
        assert np.abs(out[u] - ref).max() <= MAX_ABS and rel_l2(out[u], ref) <= REL_L2
    # a permuted placement of the same records gives the identical bits
    perm = rng.permutation(n_rec)
    inv = np.argsort(perm)
    pool_p = np.ascontiguousarray(pool[:, perm])
    idx_p = np.where(idx >= 0, inv[np.maximum(idx, 0)], -1).astype(np.int32)
    out_p = decode_pool(torch.from_numpy(pool_p.view(np.int16)).to(dev), n_rec, w, q_d,
                        torch.from_numpy(idx_p).to(dev), ws, splits, units=units).cpu().numpy()
    assert out.tobytes() == out_p.tobytes()


@pytest.mark.parametrize("kind,H,splits,units,flags", [
    # latent, the exact fallback's partial results and outputs: two head waves per token group, one,
    # and two with the query after the first chunk (more than 16 workgroup columns beside a fetch)
    ("mla", 128, 1, 2, 0), ("mla", 128, 2, 2, 0), ("mla", 20, 2, 2, 0), ("mla", 20, 1, 2, 0),
    ("mla", 128, 1, 8, 0), ("mla", 128, 1, 9, BESIDE), ("mla", 128, 2, 9, BESIDE),
    ("gqa", 16, 1, 2, 0), ("gqa", 64, 0, 2, 0), ("gqa", 64, 0, 2, BESIDE),
])
def test_attention_wide_score_range(kind, H, splits, units, flags):
    """Scores that keep growing along the selection (by far more than the kernels' reference
    slack within one split) exercise the rescale / exact-fallback paths: still within the oracle's
    tolerance, still independent of placement."""
    rng = np.random.default_rng(zlib.crc32(f"wide-{kind}-{H}-{splits}".encode()))
    if kind == "mla":
        d_qk, d_v, voff, te, scale, tpr, k = 576, 512, 0, 576, 1 / np.sqrt(192), 1, 256
        growth = slice(512, 576)      # the rope dims carry the growth; values stay N(0,1)
    else:
        d_qk, d_v, voff, te, scale, tpr, k = 128, 128, 128, 256, 1 / np.sqrt(128), 16, 16
        growth = slice(0, 128)        # keys grow, values (dims 128..255) stay N(0,1)
    n_rec = k + 21
    R = te * tpr * 2
    w = W.workload(1 if kind == "mla" else 3, q_heads=H, k=k, d_qk=d_qk, d_v=d_v, v_offset=voff,
                   tokens_per_record=tpr, record_bytes=R, scale=float(scale))
    pool_f = rng.standard_normal((units, n_rec, tpr, te)).astype(np.float32)
    q_f = (0.1 * rng.standard_normal((units, H, d_qk))).astype(np.float32)
    q_f[:, :, growth] = 1.0
    idx = np.stack([rng.choice(n_rec, size=k, replace=False) for _ in range(units)]).astype(np.int32)
    n_tok = k * tpr
    rate = 60.0 if kind == "mla" else 25.0
    for u in range(units):
        for i in range(k):
            t = i * tpr + np.arange(tpr)                    # selection-order token numbers
            pool_f[u, idx[u, i], :, growth] = (t * (rate / n_tok))[:, None]
    to_bf16 = lambda a: torch.from_numpy(a).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
    pool = to_bf16(pool_f.reshape(units, n_rec, tpr * te))
    q = to_bf16(q_f)
    # The scores really do leave the kernels' reference slack (so the rescale / exact-fallback
    # path runs): the float64 scores in log2 units, in selection order, of the bf16 inputs.
    widen = lambda a: (a.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    keys = widen(pool).reshape(units, n_rec, tpr, te)[..., :d_qk]
    sc = np.stack([np.einsum("hd,itd->hit", widen(q[u]), keys[u][idx[u]]).reshape(H, n_tok)
                   for u in range(units)]) * (scale * np.log2(np.e))
    if kind == "mla":
        # latent kernel: explicit splits of whole 64-token rounds, whose 32-token chunks go to two
        # token groups in turn; a group's reference is the max of its first chunk, and a score
        # more than 64 above it sends the whole split to the fallback. In every split of every
        # unit some head of one group goes well beyond.
        assert n_tok > 128  # not the one-round kernel
        per = -(-n_tok // splits)
        st = -(-per // 64) * 64
        chunks = sc.reshape(units, H, n_tok // 32, 32).max(axis=3)
        for b in range(0, n_tok // 32, st // 32):
            own = chunks[:, :, b:b + st // 32]
            over = np.max([(own[:, :, g::2].max(axis=2) - own[:, :, g]).max(axis=1)
                           for g in (0, 1)], axis=0)
            assert over.min() > 80.0, over
    else:
        # grouped-query kernel: the running max moves (a rescale) when a later 32-token chunk
        # outgrows it by more than 8; every chunk outgrows the previous one by more than that,
        # and each part holds at least two chunks
        cmax = sc.reshape(units, H, n_tok // 32, 32).max(axis=3)
        assert (cmax[:, :, 1:] - cmax[:, :, :-1]).min() > 8.0
        assert n_tok >= 2 * 32 * 4
    dev = torch.device("cuda:0")
    ad = attn_desc(w, splits, flags)
    ws = torch.empty(hs.hisparse_decode_workspace_bytes(units, k, R, ad), dtype=torch.uint8,
                     device=dev)
    q_d = torch.from_numpy(q.view(np.int16)).to(dev)
    out = decode_pool(torch.from_numpy(pool.view(np.int16)).to(dev), n_rec, w, q_d,
                      torch.from_numpy(idx).to(dev), ws, splits, units=units,
                      flags=flags).cpu().numpy()
    for u in range(units):
        ref = oracle_unit(w, q[u], pool[u], idx[u])
        err, rl2 = np.abs(out[u] - ref).max(), rel_l2(out[u], ref)
        log(f"  {kind} H={H} unit {u}: max-abs {err:.2e} rel-L2 {rl2:.2e}")
        assert err <= MAX_ABS and rl2 <= REL_L2
    perm = rng.permutation(n_rec)
    inv = np.argsort(perm)
    idx_p = inv[idx].astype(np.int32)
    out_p = decode_pool(torch.from_numpy(np.ascontiguousarray(pool[:, perm]).view(np.int16)).to(dev),
                        n_rec, w, q_d, torch.from_numpy(idx_p).to(dev), ws, splits,
                        units=units, flags=flags).cpu().numpy()
    assert out.tobytes() == out_p.tobytes()
