"""GPU parity of the update chain where its launches change shape: heads shared out over a block's waves,
launches of more blocks than compute units, frames that end inside a block of 64 positions.  Scores, keep lists,
codes and metadata are compared bit-for-bit with the oracle (through the C ABI)."""
import pytest

import synth_inputs as si
from oracle import xstream_oracle as xo
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,pool_group", [(129, 1), (128, 1), (200, 2)])
def test_pooled_rows_around_one_lds_load(n, pool_group):
    """129, 128 and 101 pooled rows: the row mean in a launch of its own, and in the scoring blocks up to 128 rows."""
    w = si.Workload("rows", 2, 64, n, 2, pool_group, 3 * n + 5, 6, 1, 1, 4, 64, 4, 64, "bf16", 52)
    pu.run_stream(w, 6)


@pytest.mark.parametrize("n_heads,n,budget,k_bits,k_group,meta16,slots", [
    (11, 37, 513, 4, 32, True, False), (17, 64, 513, 2, 64, False, True), (3, 65, 513, 8, 32, False, False),
    (1, 50, 513, 4, 64, True, False), (19, 40, 513, 8, 64, False, False), (5, 200, 2300, 4, 64, True, True)])
def test_wide_launches(n_heads, n, budget, k_bits, k_group, meta16, slots):
    """48 caches in one call: more score blocks than compute units on every pruning frame (and, at 2300 positions, as
    many as six times the units), so the row mean has a launch of its own and a block's waves take turns over the heads."""
    import torch
    streams, frames = 48, budget // n + 3
    units = torch.cuda.get_device_properties(0).multi_processor_count
    w = si.Workload("wide", n_heads, 64, n, 3, 8, budget, frames, 1, streams, k_bits, k_group, 4, 32, "bf16", 51)
    h = pu.make_handle(w, n_streams=streams, meta_format=1 if meta16 else 0, layout=1 if slots else 0)
    checked = (0, 21, 47)
    caches = {s: xo.OracleCache(pu.oracle_cfg(w, meta16, slots)) for s in checked}
    sigmas = {s: si.key_channel_scales(w, s, 0) for s in checked}
    wide = 0
    for t in range(frames):
        t_c = caches[0].cache_len
        if t_c + n > budget:
            assert streams * (-(-t_c // 64) - n // 64) > units
            wide += 1
        refs, dev = {}, {}
        for s in checked:
            q, k, v = si.frame_qkv(w, t, s, 0, sigmas[s])
            refs[s] = caches[s].step(q, k, v)
            dev[s] = tuple(pu.to_device(a, w) for a in (q, k, v))
        # the other caches take the frames of a checked one
        outs = [torch.empty(dev[0][0].shape, dtype=torch.float32, device="cuda:0") for _ in range(streams)]
        h.step_batched([(s, 0, *dev[s if s in dev else 0], outs[s]) for s in range(streams)])
        torch.cuda.synchronize()
        for s in checked:
            pu.check_output(outs[s].cpu().numpy(), refs[s], f"stream {s} frame {t}")
            pu.check_state(h.export(s, 0), caches[s], f"stream {s} frame {t}")
    assert wide >= 2
    h.close()


@pytest.mark.parametrize("slots", [False, True])
@pytest.mark.parametrize("k_bits,v_bits,meta16", [(k, v, m) for k in (2, 4, 8) for v in (2, 4, 8) for m in ((False, True) if k != 8 else (False,))])
def test_key_and_value_rebuild_apart(k_bits, v_bits, meta16, slots):
    """Key and value rebuild as launches of their own, which a call takes while either is timed (and above 32768
    blocks), on one and on two caches a call, for every combination of code widths."""
    import torch
    k_group, v_group = (32, 64) if (k_bits + v_bits) % 4 else (64, 32)
    w = si.Workload("apart", 3, 64, 45, 3, 8, 230, 8, 1, 2, k_bits, k_group, v_bits, v_group, "bf16", 53)
    h = pu.make_handle(w, n_streams=2, meta_format=1 if meta16 else 0, layout=1 if slots else 0)
    h.set_option("timing_every", 1)
    h.set_timing(1 << 5)                      # the key rebuild
    caches = [xo.OracleCache(pu.oracle_cfg(w, meta16, slots)) for _ in range(2)]
    sigmas = [si.key_channel_scales(w, s, 0) for s in range(2)]
    launches = 0
    for t in range(w.frames):
        items, refs = [], []
        for s in range(2) if t != 2 else range(1):          # one cache alone once, so that the two lengths differ
            q, k, v = si.frame_qkv(w, t, s, 0, sigmas[s])
            refs.append((s, caches[s].step(q, k, v)))
            dev = tuple(pu.to_device(a, w) for a in (q, k, v))
            items.append((s, 0, *dev, torch.empty(dev[0].shape, dtype=torch.float32, device="cuda:0")))
        h.step_batched(items)
        torch.cuda.synchronize()
        for (s, ref), it in zip(refs, items):
            pu.check_output(it[5].cpu().numpy(), ref, f"stream {s} frame {t}")
            pu.check_state(h.export(s, 0), caches[s], f"stream {s} frame {t}")
        launches += 1
    assert h.read_timing()["rebuild_k"][1] == launches
    h.close()
