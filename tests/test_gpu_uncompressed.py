"""The uncompressed bf16 cache at the edges of its tiles: frames of one row, around one query block and around one key
tile, forced key-range splits, logits far apart; against Eq. 1 in 64 bits (through the C ABI).  Probabilities and
values are rounded to 11 bits on the way (2^-12 each, relative), everything else is exact or fp32, so an output of unit
RMS is off by a few 2^-12: the bars of parity_util (2e-2 largest, 2e-3 mean) leave room for peaked rows only."""
import numpy as np
import pytest

from tests import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,splits,k_scale", [(1, 0, 1.0), (31, 3, 1.0), (33, 0, 4.0), (64, 2, 1.0), (65, 16, 4.0), (385, 0, 1.0)])
def test_tile_edges(n, splits, k_scale):
    import torch
    import paper_2601_01204_amd as kvx
    H, d, frames = 3, 64, 5
    rng = np.random.default_rng(60 + n)
    h = kvx.KvHandle(n_heads=H, tokens_per_frame=n, n_special=0, budget_tokens=frames * n, mode=kvx.KV_UNCOMPRESSED_BF16, max_frames=frames,
                     out_dtype=kvx.KV_F32)
    if splits:
        h.set_option("attention_splits", splits)
    keys, values = [], []
    for t in range(frames):
        q, k, v = (torch.from_numpy(rng.standard_normal((n, H, d)).astype(np.float32) * s).to("cuda:0").to(torch.bfloat16)
                   for s in (1.0, k_scale, 1.0))
        out = torch.empty((n, H, d), dtype=torch.float32, device="cuda:0")
        h.step(q, k, v, out)
        torch.cuda.synchronize()
        keys.append(k.double().cpu().numpy())
        values.append(v.double().cpu().numpy())
        K, V, Q = np.concatenate(keys), np.concatenate(values), q.double().cpu().numpy()
        s = np.einsum("qhd,khd->hqk", Q, K) / np.sqrt(d)
        p = np.exp(s - s.max(-1, keepdims=True))
        ref = np.einsum("hqk,khd->qhd", p / p.sum(-1, keepdims=True), V)
        pu.check_output(out.cpu().numpy(), ref, f"n {n} frame {t}")
    h.close()


def test_logits_near_the_top_of_fp32():
    """Products of queries and keys beyond fp32's range whose scaled logits (times log2 e / 8) are inside it: rows are one-hot."""
    import torch
    import paper_2601_01204_amd as kvx
    n, H, d, frames = 70, 2, 64, 3
    rng = np.random.default_rng(77)
    h = kvx.KvHandle(n_heads=H, tokens_per_frame=n, n_special=0, budget_tokens=frames * n, mode=kvx.KV_UNCOMPRESSED_BF16, max_frames=frames,
                     out_dtype=kvx.KV_F32)
    keys, values, overflowed = [], [], 0
    for t in range(frames):
        q, k, v = (torch.from_numpy((rng.standard_normal((n, H, d)) * s).astype(np.float32)).to("cuda:0").to(torch.bfloat16)
                   for s in (2.0 ** 63, 2.0 ** 61, 1.0))
        out = torch.empty((n, H, d), dtype=torch.float32, device="cuda:0")
        h.step(q, k, v, out)
        torch.cuda.synchronize()
        keys.append(k.double().cpu().numpy())
        values.append(v.double().cpu().numpy())
        s = np.einsum("qhd,khd->hqk", q.double().cpu().numpy(), np.concatenate(keys))
        overflowed += int((s.max(-1) > np.finfo(np.float32).max).sum())
        best = s.argmax(-1)                                       # [H, n]
        ref = np.stack([np.concatenate(values)[best[i], i] for i in range(H)], axis=1)
        pu.check_output(out.cpu().numpy(), ref, f"frame {t}")
    assert overflowed > n
    h.close()


def test_several_caches_in_one_call():
    """Two and three caches of one handle in a call, at different fill levels and one of them restarted."""
    import torch
    import paper_2601_01204_amd as kvx
    n, H, d, frames = 67, 3, 64, 6
    rng = np.random.default_rng(78)
    h = kvx.KvHandle(n_streams=3, n_layers=1, n_heads=H, tokens_per_frame=n, n_special=0, budget_tokens=frames * n, mode=kvx.KV_UNCOMPRESSED_BF16,
                     max_frames=frames, out_dtype=kvx.KV_F32)
    past = {0: [], 1: [], 2: []}

    def step(streams):
        items, refs = [], []
        for s in streams:
            q, k, v = (torch.from_numpy(rng.standard_normal((n, H, d)).astype(np.float32)).to("cuda:0").to(torch.bfloat16) for _ in range(3))
            items.append((s, 0, q, k, v, torch.empty((n, H, d), dtype=torch.float32, device="cuda:0")))
            past[s].append((k.double().cpu().numpy(), v.double().cpu().numpy()))
            K, V = (np.concatenate([kv[i] for kv in past[s]]) for i in (0, 1))
            p = np.einsum("qhd,khd->hqk", q.double().cpu().numpy(), K) / np.sqrt(d)
            p = np.exp(p - p.max(-1, keepdims=True))
            refs.append(np.einsum("hqk,khd->qhd", p / p.sum(-1, keepdims=True), V))
        h.step_batched(items)
        torch.cuda.synchronize()
        for it, ref in zip(items, refs):
            pu.check_output(it[5].cpu().numpy(), ref, f"stream {it[0]} after {len(past[it[0]])} frames")

    for streams in ((0,), (0, 1), (2, 0, 1), (1, 2)):
        step(streams)
    h.reset(0, 0)
    past[0].clear()
    for streams in ((0, 1, 2), (0, 2)):
        step(streams)
    h.close()
