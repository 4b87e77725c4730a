"""The attention kernels at the edges of their tiling, against the oracle: one to twelve query blocks a workgroup (waves
with no, one and two blocks), a last block of one row, cache ends on and off a tile, key ranges that begin and end in the
cache, at its ragged last tile and in the frame's own keys, and logits that outgrow the softmax reference of earlier keys."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import xstream_oracle as xo
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


def run(w, frames, splits, meta16, grow=1.0, dtype="bf16"):
    import torch
    h = pu.make_handle(w, meta_format=1 if meta16 else 0)
    h.set_option("attention_splits", splits)
    cache = xo.OracleCache(pu.oracle_cfg(w, meta16))
    sigma = si.key_channel_scales(w, 0, 0)
    for t in range(frames):
        q, k, v = si.frame_qkv(w, t, 0, 0, sigma)
        k = (k * np.float32(grow ** t)).astype(np.float32)        # a power of two: still bf16 values
        ref = cache.step(q, k, v)
        tq, tk, tv = (pu.to_device(a, w) for a in (q, k, v))
        out = torch.empty(tq.shape, dtype=torch.float32, device=tq.device)
        h.step(tq, tk, tv, out)
        torch.cuda.synchronize()
        pu.check_output(out.cpu().numpy(), ref, f"n {w.tokens_per_frame} splits {splits} frame {t}")
    h.close()


@pytest.mark.parametrize("meta16", [True, False])
@pytest.mark.parametrize("n,budget", [(1, 5), (31, 64), (33, 70), (64, 192), (128, 320), (129, 390), (225, 512), (256, 513), (257, 640),
                                      (289, 600), (352, 1000), (384, 768), (385, 800)])
@pytest.mark.parametrize("splits", [1, 5])
def test_query_blocks_and_key_ranges(n, budget, splits, meta16):
    w = si.Workload("tiles", 2, 64, n, min(1, n - 1), 16, budget, 4, 1, 1, 4, 64, 4, 64, "bf16", 61)
    run(w, 4, splits, meta16)


@pytest.mark.parametrize("meta16", [True, False])
@pytest.mark.parametrize("n,budget,splits", [(70, 300, 1), (300, 1300, 1), (300, 1300, 2)])
def test_logits_outgrow_the_reference(n, budget, splits, meta16):
    """Keys eight times those of the frame before: a later tile's logits exceed the first tile's by far more than the 16 log2
    units that half-precision probabilities hold, in cached tiles and in the frame's own (every path that raises the reference)."""
    w = si.Workload("grow", 2, 64, n, 1, 16, budget, 4, 1, 1, 4, 64, 4, 64, "bf16", 62)
    run(w, 4, splits, meta16, grow=8.0)


@pytest.mark.parametrize("k_bits,k_group,v_bits,v_group", [(4, 32, 2, 32), (2, 64, 8, 64), (2, 32, 8, 32), (4, 64, 8, 32)])
def test_code_widths(k_bits, k_group, v_bits, v_group):
    w = si.Workload("widths", 3, 64, 290, 2, 16, 1111, 5, 1, 1, k_bits, k_group, v_bits, v_group, "bf16", 63)
    run(w, 5, 2, True)


@pytest.mark.parametrize("mode", ["meta16", "meta32", "uncompressed"])
def test_a_tiny_logit_factor_averages_the_values(mode):
    """A logit factor of 1e-30 makes every logit 0 to all accuracy: each value weighs the same.  The bound: values in halves
    (2^-11 of |v| < 8 at most), nothing else rounds in a plain mean."""
    import paper_2601_01204_amd as kvx
    import torch
    n, H = 192, 2
    w = si.Workload("equal", H, 64, n, 1, 16, 8 * n, 1, 1, 1, 4, 64, 4, 64, "bf16", 64)
    extra = dict(mode=kvx.KV_UNCOMPRESSED_BF16, max_frames=2) if mode == "uncompressed" else dict(meta_format=1 if mode == "meta16" else 0)
    h = pu.make_handle(w, softmax_scale=1e-30, **extra)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(6)
    v = torch.randn((n, H, 64), generator=gen, device="cuda:0").to(torch.bfloat16)
    q, k = torch.full_like(v, 1.0), torch.full_like(v, 1.0)
    for splits in (1, 2):
        h.reset()
        h.set_option("attention_splits", splits)
        out = torch.empty(v.shape, dtype=torch.float32, device="cuda:0")
        h.step(q, k, v, out)
        torch.cuda.synchronize()
        err = (out.double() - v.double().mean(0, keepdim=True)).abs().max().item()
        assert err <= 8 * 2.0 ** -11, f"splits {splits}: {err}"
    h.close()


@pytest.mark.parametrize("mode", ["meta16", "meta32", "uncompressed"])
@pytest.mark.parametrize("n,frames,splits", [(70, 1, 1), (70, 2, 1), (300, 2, 1), (300, 2, 3)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_bad_query_row_stays_alone(mode, n, frames, splits, bad):
    """A query row that is not finite spoils its own output row and no other: the rest equals the outputs of the same frames
    with that row finite.  Sums of a unit's probabilities may be added in another order for its neighbours: 32 terms of 2^-24
    relative each, over values below 8."""
    import paper_2601_01204_amd as kvx
    import torch
    H = 2
    w = si.Workload("bad", H, 64, n, 1, 16, 8 * n, frames, 1, 1, 4, 64, 4, 64, "bf16", 65)
    extra = dict(mode=kvx.KV_UNCOMPRESSED_BF16, max_frames=frames) if mode == "uncompressed" else dict(meta_format=1 if mode == "meta16" else 0)
    hs = [pu.make_handle(w, **extra) for _ in range(2)]
    rows = [3, 21, 40, n - 1]
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(7)
    for h in hs:
        h.set_option("attention_splits", splits)
    for t in range(frames):
        q, k, v = (torch.randn((n, H, 64), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(3))
        spoilt = q.clone()
        spoilt[rows, 0, 5] = bad
        outs = [torch.empty(q.shape, dtype=torch.float32, device="cuda:0") for _ in hs]
        hs[0].step(q, k, v, outs[0])
        hs[1].step(spoilt, k, v, outs[1])
        torch.cuda.synchronize()
        assert torch.isfinite(outs[0]).all()
        keep = torch.ones((n, H), dtype=torch.bool, device="cuda:0")
        keep[rows, 0] = False
        err = (outs[1][keep] - outs[0][keep]).abs().max().item()
        assert err <= 8 * 32 * 2.0 ** -24, f"frame {t}: rows beside a bad one differ by {err}"
    for h in hs:
        h.close()


@pytest.mark.parametrize("mode", ["meta16", "meta32", "uncompressed"])
@pytest.mark.parametrize("n,frames,splits", [(50, 1, 1), (50, 2, 1), (64, 2, 1), (150, 1, 1), (192, 3, 1), (192, 3, 4)])
def test_the_order_of_a_tile_does_not_matter(mode, n, frames, splits):
    """The softmax reference is the largest logit of a range's first 64 keys, so that the roundings of the probabilities do not
    depend on their order within a tile of 64 (nor does a key group's quantisation): keys and values reversed inside every tile
    give the same outputs but for the order of fp32 sums, 2^-24 sqrt(32 terms) of values below 8 in up to 24 of them (another
    reference rounds every probability anew: 2^-12 each)."""
    import paper_2601_01204_amd as kvx
    import torch
    H = 2
    w = si.Workload("order", H, 64, n, 1, 16, 8 * n, frames, 1, 1, 4, 64, 4, 64, "bf16", 66)
    extra = dict(mode=kvx.KV_UNCOMPRESSED_BF16, max_frames=frames) if mode == "uncompressed" else dict(meta_format=1 if mode == "meta16" else 0)
    hs = [pu.make_handle(w, **extra) for _ in range(2)]
    order = torch.cat([torch.arange(min(a + 64, n) - 1, a - 1, -1) for a in range(0, n, 64)]).to("cuda:0")
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(8)
    for h in hs:
        h.set_option("attention_splits", splits)
    for t in range(frames):
        q, k, v = (torch.randn((n, H, 64), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(3))
        outs = [torch.empty(q.shape, dtype=torch.float32, device="cuda:0") for _ in hs]
        hs[0].step(q, k, v, outs[0])
        hs[1].step(q, k[order].contiguous(), v[order].contiguous(), outs[1])
        torch.cuda.synchronize()
        err = (outs[1] - outs[0]).abs().max().item()
        assert err <= 24 ** 0.5 * 32 ** 0.5 * 8 * 2.0 ** -24, f"frame {t}: {err}"
    for h in hs:
        h.close()


@pytest.mark.parametrize("meta16", [True, False])
@pytest.mark.parametrize("n,splits", [(40, 1), (192, 1), (192, 3)])
def test_logits_far_beyond_the_exponent_range(n, splits, meta16):
    """Logits of 1e9, in the frame's own tiles and in cached ones: a sum that starts from the reference is rounded elsewhere than
    the reference was, by more than 2^-p covers.  Every row is one of its values (its largest key's, up to the few whose logits
    fp32 cannot tell apart), never lost: finite and no further from zero than the largest value."""
    import torch
    H = 2
    w = si.Workload("far", H, 64, n, 1, 16, 8 * n, 3, 1, 1, 4, 64, 4, 64, "bf16", 67)
    h = pu.make_handle(w, meta_format=1 if meta16 else 0)
    h.set_option("attention_splits", splits)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(9)
    for t in range(3):
        q, k, v = (torch.randn((n, H, 64), generator=gen, device="cuda:0") for _ in range(3))
        q, k, v = (16384 * q).clamp(-60000, 60000).to(torch.bfloat16), (16384 * k).clamp(-60000, 60000).to(torch.bfloat16), v.to(torch.bfloat16)
        out = torch.empty(q.shape, dtype=torch.float32, device="cuda:0")
        h.step(q, k, v, out)
        torch.cuda.synchronize()
        assert torch.isfinite(out).all(), f"frame {t}"
        assert out.abs().max().item() <= 1.25 * 6.0, f"frame {t}"       # values up to 6, their codes' error up to half a step of 12 / 15
        if t == 0:
            s = torch.einsum("qhd,khd->hqk", q.double().cpu(), k.double().cpu())
            best = s.argmax(-1)
            gap = s.topk(2, -1).values
            clear = (gap[..., 0] - gap[..., 1]) * 0.18 > 2.0 ** -20 * s.abs().amax(-1) + 32
            for hh in range(H):
                want = v.double().cpu()[best[hh], hh]
                err = (out.double().cpu()[:, hh] - want)[clear[hh]].abs().max().item()
                assert err <= 8 * 2.0 ** -11, f"head {hh}: {err}"
            assert clear.double().mean().item() > 0.9
    h.close()
