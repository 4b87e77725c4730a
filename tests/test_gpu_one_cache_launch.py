"""Calls on one cache whose attention launch carries the scoring and the selection (more than 16 workgroup columns, bf16
inputs): every piece of state bit for bit against the oracle and the output against it, over the numbers of scoring blocks,
code widths, metadata formats, layouts and pooled rows, step after step, and against the launches of their own
("overlap_update" 0) on the same stream."""
import numpy as np
import pytest

import synth_inputs as si
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [False, True])
@pytest.mark.parametrize("heads,n,special,pool,budget,frames,k_bits,k_group,meta16", [
    (17, 3, 1, 2, 40, 20, 4, 64, True),          # one scoring block
    (20, 60, 5, 16, 130, 6, 2, 32, True),        # three, much of them outside the middle
    (64, 40, 0, 1, 200, 9, 4, 32, False),        # 64 heads
    (17, 129, 129, 16, 1100, 12, 8, 64, False),  # 129 pooled rows: two rounds of the row mean; 16 blocks
    (18, 130, 1, 1, 1230, 13, 4, 64, True),      # 130 pooled rows, 18 blocks shared by 16
    (17, 64, 2, 16, 2304, 38, 2, 64, True),      # 36 blocks
])
def test_scoring_and_selection_in_the_attention_launch(heads, n, special, pool, budget, frames, k_bits, k_group, meta16, slots):
    w = si.Workload("inside", heads, 64, n, special, pool, budget, frames, 1, 1, k_bits, k_group, 4, 64, "bf16", 71)
    pu.run_stream(w, frames, check_every=max(1, frames // 3), meta16=meta16, slots=slots, log=lambda *a, **k: None)


def test_the_largest_selection_and_launches_of_their_own():
    """32768 tokens, the most the selection's LDS holds: the same bits from the attention launch and from separate launches."""
    import torch
    w = si.Workload("inside_max", 17, 64, 900, 5, 16, 32768, 40, 1, 1, 4, 64, 4, 64, "bf16", 72)
    hs = [pu.make_handle(w, meta_format=1) for _ in range(2)]
    hs[1].set_option("overlap_update", 0)
    for h in hs:
        h.set_option("attention_splits", 4)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    for t in range(39):
        q, k, v = (torch.randn((900, 17, 64), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(3))
        outs = [torch.empty((900, 17, 64), dtype=torch.float32, device="cuda:0") for _ in hs]
        for h, o in zip(hs, outs):
            h.step(q, k, v, o)
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1]), t
    a, b = (h.export() for h in hs)
    for key in ("ids", "k_codes", "k_scale", "k_zero", "v_codes", "v_scale", "v_zero", "last_keep", "last_scores"):
        assert np.array_equal(a[key], b[key]), key


def test_three_caches_of_different_lengths():
    """Three caches a call, one of them not full yet: scoring blocks of their own each, against single calls without them."""
    import torch
    w = si.Workload("inside_three", 8, 64, 70, 3, 16, 1100, 30, 3, 1, 4, 64, 4, 64, "bf16", 73)
    a = pu.make_handle(w, n_streams=3, meta_format=1)
    b = pu.make_handle(w, n_streams=3, meta_format=1)
    b.set_option("overlap_update", 0)
    for h in (a, b):
        h.set_option("attention_splits", 1)      # (a call's ranges go by its shortest cache)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(6)
    for t in range(24):
        streams = [s for s in range(3) if t >= (0, 2, 12)[s]]
        f = {s: [torch.randn((70, 8, 64), generator=gen, device="cuda:0").to(torch.bfloat16) for _ in range(3)] for s in streams}
        outs = [{s: torch.empty((70, 8, 64), dtype=torch.float32, device="cuda:0") for s in streams} for _ in range(2)]
        a.step_batched([(s, 0, *f[s], outs[0][s]) for s in streams])
        for s in streams:
            b.step(*f[s], outs[1][s], stream=s)
        torch.cuda.synchronize()
        for s in streams:
            assert torch.equal(outs[0][s], outs[1][s]), (t, s)
    for s in range(3):
        x, y = a.export(s, 0), b.export(s, 0)
        for key in ("ids", "k_codes", "k_scale", "k_zero", "v_codes", "v_scale", "v_zero"):
            assert np.array_equal(x[key], y[key]), (s, key)
