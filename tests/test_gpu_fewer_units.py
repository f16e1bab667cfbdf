"""Decode launches cut into fewer units than the plan's table lists, against the oracle.

The default plan of a small or middling batch launches one or two units per CU.  The cases
sit where the choice changes: as many rows as units, more rows than one per CU, an empty row,
an uneven batch (two per CU but not one), 14 heads on one KV head, and batches that keep the
table's units because they cannot be balanced (short rows, an empty one among them).  The
planner's choice for each is asserted by a host test.  The static-scratch call runs the same
form, so its outputs are the same bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_03077_amd import libra
from paper_2606_03077_amd import workloads as wl

import gpu_harness as H

pytestmark = pytest.mark.gpu

# (KV lengths, query heads, KV heads, CUs, decode units launched)
CASES = [
    ([4096], 8, 2, 8, 8),
    ([1000, 1030, 990, 1010], 8, 2, 8, 8),            # rows = units of one per CU
    ([1000, 1030, 2000, 2010, 1020, 990], 8, 2, 8, 16),  # more rows: two per CU
    ([1000, 1030, 0, 990, 1010, 1020, 980, 1040], 8, 2, 8, 16),  # an empty row among them
    ([3000, 600, 500, 700, 650, 620, 580, 640], 4, 1, 8, 16),
    ([600, 640, 580, 620], 14, 1, 2, 4),
    ([5000, 4900, 5100], 16, 4, 32, 64),
    ([1000, 1030, 990, 1010, 1020], 8, 2, 8, 24),     # one row too many for an even cut
    ([17, 0, 300, 1, 15, 16, 900], 14, 1, 4, 11),     # too short to fill a wave
]


@pytest.mark.parametrize("lens,hq,hkv,cus,launched", CASES)
def test_fewer_units(lens, hq, hkv, cus, launched):
    H.say(f"[case] fewer units lens={lens} heads={hq}/{hkv} cus={cus}")
    b = wl.custom_batch(lens, num_q_heads=hq, num_kv_heads=hkv, seed=11, append=False)
    o, lse, cache, raw = H.run(b, plan_params=dict(num_cus=cus), repeat=2)
    plan = H.plan_for(b, num_cus=cus)
    out = torch.full((len(lens), hq, 128), H.BF16_NAN_I16, dtype=torch.int16, device="cuda")
    libra.libra_decode_attn_noalloc(cache.layout, plan, H.u16_to_dev(b.q), cache.bt,
                                    cache.bt_stride, len(lens), hq, b.scale, out)
    torch.cuda.synchronize()
    ro, rl = oracle.decode_ref(b.q, b.k_pages, b.v_pages, b.block_table, b.seq_lens, b.scale)
    units = libra.libra_plan_get_units(plan)           # the table is the rule's all the same
    ref, _ = oracle.plan_ref(lens, None, hkv, hq // hkv, oracle.PlanParams(num_cus=cus))
    assert np.array_equal(units, np.array(ref, dtype=np.int32).reshape(-1, 12))
    cache.close()
    libra.libra_plan_destroy(plan)
    H.assert_parity(o, lse, ro, rl, label=f"fewer units {lens}")
    assert np.array_equal(H.dev_to_u16(out), raw)
