"""Append tiles cut by rows and keys: the forms of the chunk launch against the oracle.

Few chunk tiles run as 128-row workgroups whose keys may be split, with the partials merged
("tiles"); short or half-filled ones in many waves as halves of their units ("halves", or
"listed" where only some units have two); many long full ones, or those beside decode rows that fill the chip, as whole 256-row tiles
("units").  The cases sit at the edges: rows of one head group at and beside 128 and 256, key
counts at and beside the 32-key step and the smallest piece, rows that see no key of a split,
one-token tails, more pages than the staged block-table row holds, and the workspace that is
too small for the partials (the same results, unsplit).  The planner's form for each, and the
most key ranges of a tile, are asserted by a host test."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_03077_amd import libra
from paper_2606_03077_amd import workloads as wl

import gpu_harness as H

pytestmark = pytest.mark.gpu

# (KV lengths after the append, new tokens, query heads, KV heads, CUs, form, key ranges)
CASES = [
    ([33], [2], 4, 1, 256, "tiles", 1),               # two tokens, one step past a boundary
    ([1056, 1025], [32, 32], 4, 1, 256, "tiles", 5),  # 128 rows exactly; 33 and 32.03 steps
    ([1500], [33], 4, 1, 256, "tiles", 6),            # 132 rows: a second tile of four rows
    ([2100], [2], 16, 1, 256, "tiles", 9),            # 32 rows, pieces of the minimum size
    ([4000, 17, 900], [51, 17, 40], 10, 2, 64, "tiles", 16),  # 255 rows; a prefill; short tiles
    ([2700, 300, 3064], [300, 1, 64], 14, 2, 256, "tiles", 12),  # a decode row beside chunk tiles
    ([700, 3000, 64], [300, 1, 64], 14, 2, 64, "tiles", 1),   # where the host sets the time
    ([1700, 20000, 64], [300, 1, 64], 14, 2, 16, "units", 1),  # and one that fills the chip
    ([900], [850], 8, 8, 256, "tiles", 4),            # rows that see no key of the later splits
    ([6000], [10], 16, 1, 8, "tiles", 8),             # 16-head groups, few slots
    ([6000], [90], 16, 1, 8, "units", 1),             # and enough tiles of them for whole units
    ([128] * 12, [128] * 12, 8, 1, 2, "halves", 1),   # more full tiles than slots
    ([130] * 12, [130] * 12, 8, 1, 2, "listed", 1),   # and a few half-filled ones among them
    ([400] * 9, [20] * 9, 8, 2, 4, "halves", 1),      # many waves of half-filled tiles
    ([700] * 5, [37] * 5, 14, 2, 4, "listed", 1),     # and of second halves of few rows
    ([3000] * 6, [256] * 6, 4, 1, 2, "units", 1),     # many waves of long full tiles
    ([66000], [40], 4, 1, 256, "tiles", 230),         # past the staged block-table row if unsplit
    ([66002] * 3, [2] * 3, 4, 1, 1, "halves", 1),     # past it in one 128-row workgroup
    ([140000], [8], 4, 1, 1, "tiles", 2),             # past it in each key range
]


@pytest.mark.parametrize("lens,new,hq,hkv,cus,form,parts", CASES)
@pytest.mark.parametrize("small_ws", [False, True])
def test_fine_tiles(lens, new, hq, hkv, cus, form, parts, small_ws):
    H.say(f"[case] fine tiles lens={lens} new={new} heads={hq}/{hkv} cus={cus} {form} small={small_ws}")
    b = wl.custom_batch(lens, q_lens=new, num_q_heads=hq, num_kv_heads=hkv, seed=7, append=True)
    cache = H.DeviceCache(b)
    plan = H.plan_for(b, num_cus=cus)
    ws = libra.alloc_workspace(plan)
    if small_ws:                                  # what a plan of whole tiles needs
        need = H.plain_workspace(plan, hq // hkv)
        assert need <= ws.numel()
        ws = ws[:need]
    rows = b.q.shape[0]
    out = torch.full((rows, hq, 128), H.BF16_NAN_I16, dtype=torch.int16, device="cuda")
    lse = torch.full((rows, hq), float("nan"), dtype=torch.float32, device="cuda")
    for _ in range(2):                            # the second call finds its tables uploaded
        libra.libra_append_attn(cache.layout, plan, H.u16_to_dev(b.q), H.u16_to_dev(b.k_new),
                                H.u16_to_dev(b.v_new), cache.bt, cache.bt_stride, len(lens), hq,
                                b.scale, ws, out, lse)
    torch.cuda.synchronize()
    o = wl.bf16_bits_to_f32(H.dev_to_u16(out)).astype(np.float64)
    ro, rl, _, _ = oracle.append_ref(b.q, b.k_new, b.v_new, b.k_pages, b.v_pages, b.block_table,
                                     b.seq_lens, b.q_lens, b.scale)
    cache.close()
    libra.libra_plan_destroy(plan)
    H.assert_parity(o, lse.cpu().numpy().astype(np.float64), ro, rl, label=f"fine {lens}/{new}")
