"""GPU parity of the HIP path (through the C-ABI) against the fp64 oracle.

Tolerances (bf16 inputs, float32 accumulation, bf16 outputs): max |gpu - oracle| <= 2e-2
over every output element, max over rows of ||gpu - oracle||_inf / ||oracle||_inf <= 1e-2,
and |lse_gpu - lse_oracle| <= 1e-3 (natural log).  Layout moves, block-table gathers and
cache writes are compared bit for bit.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle.attention import gather_tokens
from paper_2606_03077_amd import libra
from paper_2606_03077_amd import workloads as wl

import gpu_harness as H

pytestmark = pytest.mark.gpu


def _decode_oracle(batch, rows=None):
    return oracle.decode_ref(batch.q, batch.k_pages, batch.v_pages, batch.block_table,
                             batch.seq_lens, batch.scale, batch_rows=rows)


def _append_oracle(batch, rows=None):
    return oracle.append_ref(batch.q, batch.k_new, batch.v_new, batch.k_pages, batch.v_pages,
                             batch.block_table, batch.seq_lens, batch.q_lens, batch.scale,
                             batch_rows=rows)


def test_pack_unpack_and_gather_are_bit_exact():
    H.say("[case] pack/unpack/gather tiny")
    b = wl.make_batch("tiny")
    cache = H.DeviceCache(b)
    k2, v2 = cache.unpack()
    assert np.array_equal(k2, b.k_pages) and np.array_equal(v2, b.v_pages)
    lens = b.seq_lens.astype(np.int64)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    Hkv = b.workload.num_kv_heads
    ko = torch.empty((int(cu[-1]), Hkv, 128), dtype=torch.int16, device="cuda")
    vo = torch.empty_like(ko)
    max_pages = int((lens.max() + 15) // 16)
    libra.libra_kv_gather(cache.layout, cache.bt, cache.bt_stride, torch.from_numpy(cu).cuda(),
                          len(lens), max_pages, ko, vo)
    torch.cuda.synchronize()
    kg, vg = H.dev_to_u16(ko), H.dev_to_u16(vo)
    for s in range(len(lens)):
        for g in range(Hkv):
            ref_k = gather_tokens(b.k_pages, b.block_table[s], g, int(lens[s]))
            ref_v = gather_tokens(b.v_pages, b.block_table[s], g, int(lens[s]))
            assert np.array_equal(kg[cu[s]:cu[s + 1], g], ref_k)
            assert np.array_equal(vg[cu[s]:cu[s + 1], g], ref_v)
    cache.close()


def test_pack_unpack_round_trip_across_launch_chunks():
    """Whole-cache and offset page ranges larger than one pack / unpack launch (2^18
    tiles) round-trip bit for bit (device-generated bytes, compared on the device)."""
    H.say("[case] pack/unpack 70000 pages x 8 heads")
    P, Hkv = 70000, 8
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    k_log = torch.randint(-32768, 32767, (P * Hkv * 2048,), dtype=torch.int16, device="cuda",
                          generator=g)
    v_log = torch.randint(-32768, 32767, (P * Hkv * 2048,), dtype=torch.int16, device="cuda",
                          generator=g)
    k = torch.empty_like(k_log)
    v = torch.empty_like(v_log)
    lay = libra.libra_kv_layout_create(k, v, P, Hkv)
    libra.libra_kv_pack_pages(lay, k_log, v_log, 0, P)
    k2 = torch.empty_like(k_log)
    v2 = torch.empty_like(v_log)
    libra.libra_kv_unpack_pages(lay, k2, v2, 0, P)
    torch.cuda.synchronize()
    assert torch.equal(k2, k_log) and torch.equal(v2, v_log)
    # a sub-range that starts off a launch boundary: pages [first, first + n)
    first, n = 12345, 40000
    span = slice(first * Hkv * 2048, (first + n) * Hkv * 2048)
    k3 = torch.zeros(n * Hkv * 2048, dtype=torch.int16, device="cuda")
    v3 = torch.zeros_like(k3)
    libra.libra_kv_unpack_pages(lay, k3, v3, first, n)
    libra.libra_kv_pack_pages(lay, k3.flip(0), v3.flip(0), first, n)   # different bytes in
    libra.libra_kv_unpack_pages(lay, k2, v2, 0, P)
    torch.cuda.synchronize()
    assert torch.equal(k3, k_log[span]) and torch.equal(v3, v_log[span])
    assert torch.equal(k2[span], k_log[span].flip(0)) and torch.equal(v2[span], v_log[span].flip(0))
    assert torch.equal(k2[:span.start], k_log[:span.start])
    assert torch.equal(k2[span.stop:], k_log[span.stop:])
    libra.libra_kv_layout_destroy(lay)


def test_decode_tiny_full():
    H.say("[case] decode tiny (config 1) full")
    b = wl.make_batch("tiny")
    o, lse, cache, _ = H.run(b)
    ro, rl = _decode_oracle(b)
    H.assert_parity(o, lse, ro, rl, label="tiny")
    cache.close()


@pytest.mark.parametrize("hq,hkv", [(28, 4), (8, 2), (64, 8), (16, 16), (16, 1)])
def test_decode_ragged_with_splits(hq, hkv):
    lens = [1, 15, 16, 17, 31, 33, 100, 257, 1000, 2049, 5000]
    H.say(f"[case] decode ragged hq={hq} hkv={hkv} lens={lens}")
    b = wl.custom_batch(lens, num_q_heads=hq, num_kv_heads=hkv, seed=hq * 100 + hkv)
    for params in [dict(num_cus=4, units_per_cu=1, min_split_pages=2, max_splits=64),
                   dict(num_cus=256, units_per_cu=2, min_split_pages=32, max_splits=64),
                   dict(num_cus=8, units_per_cu=1, min_split_pages=1, max_splits=1)]:
        o, lse, cache, _ = H.run(b, plan_params=params)
        ro, rl = _decode_oracle(b)
        H.assert_parity(o, lse, ro, rl, label=f"ragged {hq}/{hkv} {params}")
        cache.close()


def test_decode_single_key_returns_v_bitwise():
    H.say("[case] decode L=1")
    b = wl.custom_batch([1, 1, 1], num_q_heads=8, num_kv_heads=2, seed=5)
    o, lse, cache, raw = H.run(b)
    G = 4
    for s in range(3):
        for h in range(8):
            v = b.v_pages[b.block_table[s, 0], h // G, 0]
            assert np.array_equal(raw[s, h], v)
    ro, rl = _decode_oracle(b)
    H.assert_parity(o, lse, ro, rl, label="L=1")
    cache.close()


def test_decode_empty_and_ragged_edges():
    H.say("[case] decode empty sequences")
    b = wl.custom_batch([0, 5, 0, 16, 17], num_q_heads=8, num_kv_heads=2, seed=6)
    o, lse, cache, _ = H.run(b)
    assert np.all(o[[0, 2]] == 0) and np.all(np.isneginf(lse[[0, 2]]))
    ro, rl = _decode_oracle(b)
    H.assert_parity(o, lse, ro, rl, label="empty")
    cache.close()


def test_decode_page_permutation_and_rerun_are_bitwise_identical():
    H.say("[case] page permutation / determinism")
    b = wl.custom_batch([700, 33, 4000, 1], num_q_heads=28, num_kv_heads=4, seed=7)
    params = dict(num_cus=4, units_per_cu=1, min_split_pages=4, max_splits=16)
    o1, l1, cache, raw1 = H.run(b, plan_params=params, repeat=2)
    o1b, l1b, _, raw1b = H.run(b, cache=cache, plan_params=params)
    assert np.array_equal(raw1, raw1b) and np.array_equal(l1, l1b)
    cache.close()
    perm = np.random.default_rng(1).permutation(b.num_pages)
    kp = np.empty_like(b.k_pages)
    vp = np.empty_like(b.v_pages)
    kp[perm] = b.k_pages
    vp[perm] = b.v_pages
    b2 = wl.Batch(b.workload, b.seq_lens, b.q_lens, b.cu_q_lens, perm[b.block_table].astype(np.int32),
                  kp, vp, b.q, None, None, b.scale)
    o2, l2, cache2, raw2 = H.run(b2, plan_params=params)
    assert np.array_equal(raw1, raw2) and np.array_equal(l1, l2)
    cache2.close()


_BENCH_WEIGHTS = []


def _bench_plan_params():
    """The plan parameters bench.py times with: defaults plus XCD read weights measured
    on this device (once per test session, on a 1 GiB buffer as bench.py's flush)."""
    if not _BENCH_WEIGHTS:
        buf = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
        _BENCH_WEIGHTS.append(libra.libra_xcd_read_weights(buf, reps=10))
        del buf
        H.say(f"[xcd] weights {_BENCH_WEIGHTS[0]}")
    return dict(xcd_weight=_BENCH_WEIGHTS[0])


@pytest.mark.parametrize("name", ["7b", "longtail", "straggler"])
def test_decode_full_config_every_row(name):
    """Configs 2-4 at full size, planned as bench.py plans them: every output row and
    LSE against the oracle (computed per (sequence, KV head) in host processes)."""
    H.say(f"[case] decode {name} full size, every row")
    b = wl.make_batch(name)
    o, lse, cache, _ = H.run(b, plan_params=_bench_plan_params())
    cache.close()
    ro, rl, secs, workers = H.oracle_whole_batch(b)
    H.say(f"[oracle] {name}: {len(b.seq_lens)} rows x {b.workload.num_q_heads} heads in "
          f"{secs:.1f} s on {workers} host processes")
    H.assert_parity(o, lse, ro, rl, label=f"{name} all {len(b.seq_lens)} rows")


@pytest.mark.parametrize("hq,hkv", [(32, 8), (28, 4), (8, 8), (16, 1), (40, 8)])
def test_append_mixed_chunks(hq, hkv):
    prior = [0, 7, 100, 1000, 33, 16, 5000, 250]
    chunk = [5, 1, 64, 300, 1, 16, 129, 1]
    lens = [p + c for p, c in zip(prior, chunk)]
    H.say(f"[case] append mixed hq={hq} hkv={hkv}")
    b = wl.custom_batch(lens, q_lens=chunk, num_q_heads=hq, num_kv_heads=hkv, seed=hq + hkv)
    o, lse, cache, _ = H.run(b, plan_params=dict(num_cus=4, units_per_cu=1, min_split_pages=2))
    ro, rl, k_after, v_after = _append_oracle(b)
    H.assert_parity(o, lse, ro, rl, label=f"append {hq}/{hkv}")
    k2, v2 = cache.unpack()
    assert np.array_equal(k2, k_after) and np.array_equal(v2, v_after)
    cache.close()


def test_append_one_token_rows_match_decode_bitwise():
    H.say("[case] append C=1 vs decode")
    lens = [40, 17, 3000, 1]
    b = wl.custom_batch(lens, q_lens=[1, 1, 1, 1], num_q_heads=28, num_kv_heads=4, seed=3,
                        append=True)
    oa, la, cache, rawa = H.run(b, plan_params=dict(num_cus=4, units_per_cu=1, min_split_pages=2))
    k_after, v_after = cache.unpack()
    cache.close()
    bd = wl.Batch(wl.dataclasses.replace(b.workload, append=False), b.seq_lens, b.q_lens,
                  b.cu_q_lens, b.block_table, k_after, v_after, b.q, None, None, b.scale)
    od, ld, cache2, rawd = H.run(bd, plan_params=dict(num_cus=4, units_per_cu=1, min_split_pages=2))
    cache2.close()
    assert np.array_equal(rawa, rawd) and np.array_equal(la, ld)


def test_append_full_config_every_row():
    """Config 5 at full size: every query row (chunk tokens and single tokens) and LSE
    against the oracle, and the cache write bit for bit."""
    H.say("[case] append (config 5) full size, every row")
    b = wl.make_batch("append")
    o, lse, cache, _ = H.run(b, plan_params=_bench_plan_params())
    k2, v2 = cache.unpack()
    cache.close()
    ro, rl, secs, workers = H.oracle_whole_batch(b)
    H.say(f"[oracle] append: {b.q.shape[0]} rows x {b.workload.num_q_heads} heads in "
          f"{secs:.1f} s on {workers} host processes")
    H.assert_parity(o, lse, ro, rl, label=f"append all {b.q.shape[0]} rows")
    k_after, v_after = oracle.write_new_tokens(b.k_pages, b.v_pages, b.k_new, b.v_new,
                                               b.block_table, b.seq_lens, b.q_lens)
    assert np.array_equal(k2, k_after) and np.array_equal(v2, v_after)


def test_split_merge_sees_fresh_partials_when_workspace_is_reused():
    """Same lengths, different values, one plan and one workspace: every call must merge
    its own partials (stale ones from the previous call would go unnoticed with equal
    inputs)."""
    lens = [3000, 17, 5000, 129, 2048]
    H.say(f"[case] workspace reuse lens={lens}")
    batches = [wl.custom_batch(lens, num_q_heads=28, num_kv_heads=4, seed=s) for s in (21, 22, 23)]
    w = batches[0].workload
    plan = libra.libra_splitkv_plan(libra.LIBRA_MODE_DECODE, len(lens), 28, 4, lens, None,
                                    num_cus=64, units_per_cu=1, min_split_pages=2)
    assert libra.libra_plan_get_info(plan)["n_partial_slots"] > 0
    ws = libra.alloc_workspace(plan)
    caches = [H.DeviceCache(b) for b in batches]
    qs = [H.u16_to_dev(b.q) for b in batches]
    refs = [_decode_oracle(b) for b in batches]
    out = torch.empty((len(lens), 28, 128), dtype=torch.int16, device="cuda")
    lse = torch.empty((len(lens), 28), dtype=torch.float32, device="cuda")
    for i in [0, 1, 2, 1, 0, 2, 2, 0]:
        libra.libra_decode_attn(caches[i].layout, plan, qs[i], caches[i].bt, caches[i].bt_stride,
                                len(lens), 28, batches[i].scale, ws, out, lse)
        torch.cuda.synchronize()
        o = H.bf16_dev_to_f64(out)
        H.assert_parity(o, lse.cpu().numpy().astype(np.float64), refs[i][0], refs[i][1],
                        label=f"reuse call batch {i}")
    for c in caches:
        c.close()
    libra.libra_plan_destroy(plan)


def test_two_plans_take_turns_on_one_workspace():
    """Two plans with different unit tables share one workspace without explicit uploads:
    each call must re-upload its own tables when the other plan wrote the workspace last.
    (Both batches have 5 rows and equally wide block tables padded with valid spare pages,
    so even a stale table would stay in bounds and show up as a parity failure.)"""
    lens_a = [3000, 17, 5000, 129, 2048]
    lens_b = [100, 2900, 40, 4999, 1000]
    H.say("[case] two plans, one workspace")
    ba = wl.custom_batch(lens_a, num_q_heads=28, num_kv_heads=4, seed=31)
    bb = wl.custom_batch(lens_b, num_q_heads=28, num_kv_heads=4, seed=32)
    assert ba.block_table.shape == bb.block_table.shape
    kw = dict(num_cus=64, units_per_cu=1, min_split_pages=2)
    pa = libra.libra_splitkv_plan(libra.LIBRA_MODE_DECODE, 5, 28, 4, lens_a, None, **kw)
    pb = libra.libra_splitkv_plan(libra.LIBRA_MODE_DECODE, 5, 28, 4, lens_b, None, **kw)
    assert not np.array_equal(libra.libra_plan_get_units(pa), libra.libra_plan_get_units(pb))
    n = max(libra.libra_plan_workspace_bytes(pa), libra.libra_plan_workspace_bytes(pb))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    assert ws.data_ptr() % 256 == 0
    cases = {"a": (ba, pa, H.DeviceCache(ba), _decode_oracle(ba)),
             "b": (bb, pb, H.DeviceCache(bb), _decode_oracle(bb))}
    out = torch.empty((5, 28, 128), dtype=torch.int16, device="cuda")
    lse = torch.empty((5, 28), dtype=torch.float32, device="cuda")
    for key in "abaabba":
        b, plan, cache, ref = cases[key]
        libra.libra_decode_attn(cache.layout, plan, H.u16_to_dev(b.q), cache.bt, cache.bt_stride,
                                5, 28, b.scale, ws, out, lse)
        torch.cuda.synchronize()
        H.assert_parity(H.bf16_dev_to_f64(out), lse.cpu().numpy().astype(np.float64), ref[0],
                        ref[1], label=f"plan {key}")
    for b, plan, cache, _ in cases.values():
        cache.close()
        libra.libra_plan_destroy(plan)


def test_append_prior_longer_than_staged_block_table():
    """A chunk whose keys span more pages than the chunk kernel stages in LDS (4096); with the
    default plan they are split into ranges that fit (test_gpu_fine_tiles.py runs workgroups
    that read past the staged ids)."""
    prior, chunk = 66000, 100
    H.say(f"[case] append long prior {prior} chunk {chunk}")
    b = wl.custom_batch([prior + chunk, 40], q_lens=[chunk, 1], num_q_heads=4, num_kv_heads=1,
                        seed=77)
    o, lse, cache, _ = H.run(b)
    ro, rl, _, _ = _append_oracle(b)
    H.assert_parity(o, lse, ro, rl, label="append long prior")
    cache.close()


@pytest.mark.parametrize("chunk", [1, 600, 2000])
def test_recompute_prefill_empty_prior(chunk):
    """Recompute of a migrated request's KV: an append with no prior context."""
    H.say(f"[case] prefill P=0 C={chunk}")
    b = wl.custom_batch([chunk], q_lens=[chunk], num_q_heads=40, num_kv_heads=8, seed=chunk,
                        append=True)
    o, lse, cache, _ = H.run(b)
    ro, rl, k_after, v_after = _append_oracle(b)
    H.assert_parity(o, lse, ro, rl, label=f"prefill C={chunk}")
    k2, v2 = cache.unpack()
    assert np.array_equal(k2, k_after) and np.array_equal(v2, v_after)
    cache.close()


@pytest.mark.parametrize("hq,hkv", [(28, 4), (16, 1), (48, 8), (96, 8), (24, 8)])
def test_recompute_prefill_head_shapes(hq, hkv):
    """Fewer than eight (sequence, KV head) groups, whose tiles the plan cuts into parts
    over all XCD queues, and groups G that do not divide 16 (query tiles of
    floor(256 / G) tokens whose column blocks span token boundaries)."""
    chunk = 1500
    from oracle.plan import plan_ref, PlanParams
    _, info = plan_ref([chunk], [chunk], hkv, hq // hkv, PlanParams())
    assert info["q_tile"] == 256 // (hq // hkv)
    if hkv < 8:
        assert all(n > 0 for n in info["xcd_queue_lens"])   # the groups were cut into parts
    H.say(f"[case] prefill P=0 C={chunk} hq={hq} hkv={hkv}")
    b = wl.custom_batch([chunk], q_lens=[chunk], num_q_heads=hq, num_kv_heads=hkv,
                        seed=hq * 100 + hkv, append=True)
    o, lse, cache, _ = H.run(b)
    ro, rl, k_after, v_after = _append_oracle(b)
    H.assert_parity(o, lse, ro, rl, label=f"prefill {hq}/{hkv}")
    k2, v2 = cache.unpack()
    assert np.array_equal(k2, k_after) and np.array_equal(v2, v_after)
    cache.close()


@pytest.mark.parametrize("hq,hkv", [(40, 8), (28, 4)])
def test_recompute_prefill_full_length_bands(hq, hkv):
    """The 40,960-token recompute at full size.  The oracle checks every head of whole
    bands of query rows: the first three query tiles, a band of 256 rows around the
    middle that spans tile boundaries, and the last 256 rows (query tiles are
    floor(256 / G) tokens: 51 at 40/8 heads, 36 at 28/4).  Every other row is checked
    for having been written (finite output and LSE)."""
    H.say(f"[case] prefill 40960 full size hq={hq} hkv={hkv}")
    b = wl.make_batch("prefill", num_q_heads=hq, num_kv_heads=hkv)
    o, lse, cache, _ = H.run(b)
    cache.close()
    assert np.isfinite(o).all() and np.isfinite(lse).all()
    T = 256 // (hq // hkv)
    k_all = b.k_new  # prior is empty: the new tokens are the whole context
    v_all = b.v_new
    from oracle.attention import attend, bf16_bits_to_f64
    G = hq // hkv
    L = b.q.shape[0]
    bands = [(0, 3 * T), (20480 - 128, 20480 + 128), (L - 256, L)]
    for r0, r1 in bands:
        visible = np.arange(r1)[None, :] <= np.arange(r0, r1)[:, None]
        for g in range(hkv):
            K = bf16_bits_to_f64(k_all[:r1, g])
            V = bf16_bits_to_f64(v_all[:r1, g])
            for h in range(g * G, (g + 1) * G):
                ro, rl = attend(bf16_bits_to_f64(b.q[r0:r1, h]), K, V, b.scale, visible)
                H.assert_parity(o[r0:r1, h], lse[r0:r1, h], ro, rl,
                                label=f"prefill rows [{r0},{r1}) head {h}")


def test_one_plan_shared_by_two_threads_and_streams():
    """Calls on two streams from two host threads share one plan (distinct workspaces and
    outputs): every result equals the single-stream one bit for bit."""
    import threading
    H.say("[case] plan shared by two threads / streams")
    b = wl.custom_batch([3000, 17, 900, 5000], num_q_heads=32, num_kv_heads=8, seed=21)
    cache = H.DeviceCache(b)
    plan = libra.libra_splitkv_plan(libra.LIBRA_MODE_DECODE, 4, 32, 8, b.seq_lens.tolist(), None,
                                    num_cus=64)
    q = H.u16_to_dev(b.q)
    ref = torch.empty((4, 32, 128), dtype=torch.int16, device="cuda")
    ws0 = libra.alloc_workspace(plan)
    libra.libra_decode_attn(cache.layout, plan, q, cache.bt, cache.bt_stride, 4, 32, b.scale, ws0,
                            ref)
    torch.cuda.synchronize()
    results, errors = {}, []

    def worker(t):
        try:
            stream = torch.cuda.Stream()
            ws = libra.alloc_workspace(plan)
            outs = [torch.empty_like(ref) for _ in range(10)]
            with torch.cuda.stream(stream):
                for o in outs:
                    libra.libra_decode_attn(cache.layout, plan, q, cache.bt, cache.bt_stride, 4,
                                            32, b.scale, ws, o, stream=stream)
            stream.synchronize()
            results[t] = outs
        except Exception as e:  # reported below
            errors.append(e)

    threads = [threading.Thread(target=worker, args=(t,)) for t in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    r = H.dev_to_u16(ref)
    for outs in results.values():
        for o in outs:
            assert np.array_equal(H.dev_to_u16(o), r)
    libra.libra_plan_destroy(plan)
    cache.close()


@pytest.mark.parametrize("group,hkv", [(1, 4), (3, 2), (5, 8), (7, 4), (16, 1)])
def test_merge_thread_groups_many_splits(group, hkv):
    """Rows cut into many splits (up to 64), into few and into none, at group sizes from one
    head to 16: the merge kernel takes a block per head, whose 16 groups of 16 threads share
    the splits; a row whose split count is not a multiple of the group count and one with
    fewer splits than groups."""
    lens = [16 * 64 * 5 + 7, 16 * 40 + 3, 16 * 3, 1000]
    H.say(f"[case] merge groups G={group} hkv={hkv} lens={lens}")
    b = wl.custom_batch(lens, num_q_heads=group * hkv, num_kv_heads=hkv, seed=60 + group)
    params = dict(num_cus=512, units_per_cu=1, min_split_pages=1, max_splits=64)
    plan = H.plan_for(b, **params)
    units = libra.libra_plan_get_units(plan)
    libra.libra_plan_destroy(plan)
    nsplit = {int(u[0]): int(u[7]) for u in units}
    assert max(nsplit.values()) >= 40 and min(nsplit.values()) <= 3, nsplit
    o, lse, cache, _ = H.run(b, plan_params=params)
    cache.close()
    ro, rl = _decode_oracle(b)
    H.assert_parity(o, lse, ro, rl, label=f"merge groups G={group} splits {nsplit}")
