"""Append tiles cut by rows and keys: the forms of the chunk launch against the oracle.

Few chunk tiles run as 128-row workgroups whose keys may be split, with the partials merged;
many full ones as whole 256-row tiles.  The cases sit at the edges: rows of one head group at
and beside 128 and 256, key counts at and beside the 32-key step and the smallest piece, rows
that see no key of a split, one-token tails, and the workspace that is too small for the
partials (the same results, unsplit)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_03077_amd import libra
from paper_2606_03077_amd import workloads as wl

import gpu_harness as H

pytestmark = pytest.mark.gpu

# (KV lengths after the append, new tokens, query heads, KV heads, CUs)
CASES = [
    ([33], [2], 4, 1, 256),                       # two tokens, one step past a boundary
    ([1056, 1025], [32, 32], 4, 1, 256),          # 128 rows exactly; 33 and 32.03 steps
    ([1500], [33], 4, 1, 256),                    # 132 rows: a second tile of four rows
    ([2100], [2], 16, 1, 256),                    # 32 rows, many pieces of the minimum size
    ([4000, 17, 900], [51, 17, 40], 10, 2, 64),   # 255 rows; a prefill; a short tile
    ([700, 3000, 64], [300, 1, 64], 14, 2, 64),   # decode rows beside chunk tiles
    ([900], [850], 8, 8, 256),                    # rows that see no key of the later splits
    ([6000], [90], 16, 1, 8),                     # 16-head groups, few slots
    ([130] * 12, [130] * 12, 8, 1, 2),            # more full tiles than slots: whole tiles
    ([400] * 9, [20] * 9, 8, 2, 4),               # many waves of half-filled tiles
    ([66000], [40], 4, 1, 256),                   # past the staged block-table row
]


@pytest.mark.parametrize("lens,new,hq,hkv,cus", CASES)
@pytest.mark.parametrize("small_ws", [False, True])
def test_fine_tiles(lens, new, hq, hkv, cus, small_ws):
    H.say(f"[case] fine tiles lens={lens} new={new} heads={hq}/{hkv} cus={cus} small={small_ws}")
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
