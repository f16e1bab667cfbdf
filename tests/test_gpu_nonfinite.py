"""NaN and infinity in the inputs of an append whose chunk tiles are cut into key ranges.

A row that sees a NaN score or value has no finite result, whatever its keys were cut into:
its output is NaN and its LSE -inf, with the partials merged (full workspace) and unsplit (a
workspace too small for them) alike.  Rows that do not see it keep the oracle's results."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_03077_amd import libra
from paper_2606_03077_amd import workloads as wl

import gpu_harness as H

pytestmark = pytest.mark.gpu

HQ, HKV, NEW = 8, 2, 32        # one fine tile of 32 x 4 rows per KV head


def append(b, plan, ws):
    cache = H.DeviceCache(b)
    out = torch.zeros((b.q.shape[0], HQ, 128), dtype=torch.int16, device="cuda")
    lse = torch.zeros((b.q.shape[0], HQ), dtype=torch.float32, device="cuda")
    libra.libra_append_attn(cache.layout, plan, H.u16_to_dev(b.q), H.u16_to_dev(b.k_new),
                            H.u16_to_dev(b.v_new), cache.bt, cache.bt_stride, len(b.seq_lens), HQ,
                            b.scale, ws, out, lse)
    torch.cuda.synchronize()
    cache.close()
    return H.bf16_dev_to_f64(out), lse.cpu().numpy().astype(np.float64)


# (KV length, CUs, splits of the tile's keys)
@pytest.mark.parametrize("length,cus,splits", [(3072, 2, 2), (3072, 4, 4), (2304, 9, 9)])
@pytest.mark.parametrize("where", ["key", "new key", "value", "query"])
@pytest.mark.parametrize("small_ws", [False, True])
def test_nan_reaches_the_rows_that_see_it(length, cus, splits, where, small_ws):
    H.say(f"[case] NaN {where} length={length} cus={cus} splits={splits} small={small_ws}")
    b = wl.custom_batch([length], q_lens=[NEW], num_q_heads=HQ, num_kv_heads=HKV, seed=5)
    ro, rl, _, _ = oracle.append_ref(b.q, b.k_new, b.v_new, b.k_pages, b.v_pages, b.block_table,
                                     b.seq_lens, b.q_lens, b.scale)
    bad = np.zeros((NEW, HQ), bool)
    page = int(b.block_table[0, length // 32])              # half-way: in no split's first step
    if where == "key":
        b.k_pages[page, 0, 5, :] = wl.BF16_NAN
        bad[:, :4] = True
    elif where == "new key":                                # seen from token 20 on
        b.k_new[20, 0, 3] = wl.BF16_NAN
        bad[20:, :4] = True
    elif where == "value":
        b.v_pages[page, 0, 5, :] = wl.BF16_NAN
        bad[:, :4] = True
    else:
        b.q[7, 6, :] = wl.BF16_NAN
        bad[7, 6] = True
    plan = H.plan_for(b, num_cus=cus)
    assert H.chunk_partials(plan) == HKV * splits
    ws = libra.alloc_workspace(plan)
    if small_ws:
        ws = ws[:H.plain_workspace(plan)]
    o, lse = append(b, plan, ws)
    libra.libra_plan_destroy(plan)
    assert np.isnan(o[bad]).all()
    if where != "value":
        assert np.isneginf(lse[bad]).all()
    H.assert_parity(o[~bad][:, None], lse[~bad][:, None], ro[~bad][:, None], rl[~bad][:, None],
                    label=f"rows beside a NaN {where}, {splits} splits")


@pytest.mark.parametrize("cus,splits", [(2, 2), (4, 4)])
@pytest.mark.parametrize("at", ["start", "piece", "both"])
@pytest.mark.parametrize("small_ws", [False, True])
def test_keys_masked_by_infinity(cus, splits, at, small_ws):
    """Keys that a program masks with an infinite channel score -inf: whole first steps of a
    tile or of one of its key ranges give no maximum, which the steps after it then set."""
    length = 3072
    H.say(f"[case] -inf keys at {at} cus={cus} splits={splits} small={small_ws}")
    b = wl.custom_batch([length], q_lens=[NEW], num_q_heads=HQ, num_kv_heads=HKV, seed=6)
    b.q[:, :, 0] = wl.f32_to_bf16_bits(np.float32(1.0))
    starts = {"start": [0], "piece": [length // 2], "both": [0, length // 2]}[at]
    for s in starts:
        for p in range(s // 16, s // 16 + 4):               # a step of 64 keys
            b.k_pages[b.block_table[0, p], :, :, 0] = wl.f32_to_bf16_bits(np.float32(-np.inf))
    ro, rl, _, _ = oracle.append_ref(b.q, b.k_new, b.v_new, b.k_pages, b.v_pages, b.block_table,
                                     b.seq_lens, b.q_lens, b.scale)
    assert np.isfinite(ro).all() and np.isfinite(rl).all()
    plan = H.plan_for(b, num_cus=cus)
    assert H.chunk_partials(plan) == HKV * splits
    ws = libra.alloc_workspace(plan)
    if small_ws:
        ws = ws[:H.plain_workspace(plan)]
    o, lse = append(b, plan, ws)
    libra.libra_plan_destroy(plan)
    H.assert_parity(o, lse, ro, rl, label=f"-inf keys at {at}, {splits} splits")
