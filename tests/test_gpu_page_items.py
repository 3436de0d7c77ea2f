"""Page writes whose pages are counted by tokens and found by search, and rotated
writes of several heads per workgroup: bit for bit the oracle's pools.

A call with single tokens beside long chunks finds each page's row by a search
over cu_new (one, two or three rounds of 64 probes here); rotated writes of many full
pages into bf16 pools take four KV heads per workgroup where four divide them, the fused
write two, so some KV head counts leave a remainder. Rows without tokens, page-aligned and unaligned starts and ends
are among the rows.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_18815_amd as ra
import synth
from tests.gpu_util import bits
from tests.test_gpu_rope import i32, rope_table

pytestmark = pytest.mark.gpu
KS, VS = 0.03, 0.02

ROWS = [
    ([1] * 70 + [500], 3),                                        # two search rounds
    ([0, 1, 15, 16, 17, 31, 33, 0, 600] + [1] * 40 + [0], 8),     # one round, edges of pages
    ([1] * 5000 + [900, 1000], 2),                                # three rounds
    ([1] * 1000 + [500, 500], 5),                                 # search, an odd number of heads
    ([300] * 60, 9),                                              # full grid, one head left of four
    ([300] * 60, 8),                                              # full grid, four heads when rotated (bf16)
    ([1] * 800 + [2000] * 4 + [1100] * 8, 8),                     # search, four heads when rotated (bf16)
]


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("n,Hkv", ROWS)
def test_page_write_items_bitexact(device, n, Hkv, fp8, rope):
    print(f"[gpu-test] page items rows={len(n)} Hkv={Hkv} fp8={fp8} rope={rope}", flush=True)
    rng = np.random.default_rng(41)
    start = rng.integers(0, 40, len(n)).astype(np.int32)
    lay = synth.make_layout(rng, start + np.asarray(n))
    gen = synth.value_generator(41, device)
    make = (lambda s: synth.randn_fp8_codes(s, gen, device, KS)) if fp8 else \
        (lambda s: synth.randn_bf16(s, gen, device))
    k, v = make((lay.num_pages, Hkv, 16, 128)), make((lay.num_pages, Hkv, 128, 16))
    kf, vf = k.clone(), v.clone()
    cu = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    k_new = synth.randn_bf16((int(cu[-1]), Hkv, 128), gen, device)
    v_new = synth.randn_bf16((int(cu[-1]), Hkv, 128), gen, device)
    max_pos = int((start + np.asarray(n)).max())
    table = rope_table(1e6, max_pos)
    cs = torch.from_numpy(table).to(device) if rope else None
    k0, v0 = bits(k), bits(v)
    scales = (KS, VS) if fp8 else (None, None)
    args = (i32(cu, device), i32(start, device))
    ra.kv_page_write(k_new, v_new, *args, ra.PagedKV(k, v, i32(lay.block_table, device), *scales),
                     max(n), max_pos, cos_sin=cs)
    # the same write inside the append call (one query head per KV head)
    ra.append_write(k_new, k_new, v_new, *args,
                    ra.PagedKV(kf, vf, i32(lay.block_table, device), *scales), max(n), max_pos,
                    cos_sin=cs)
    torch.cuda.synchronize()
    src = bits(k_new)
    if rope:
        pos = np.concatenate([np.arange(s, s + t) for s, t in zip(start, n)]).astype(np.int32)
        src = oracle.rope(src, pos, table)
    if fp8:
        kx, vx = oracle.page_write_fp8(src, bits(v_new), cu, start, lay.block_table, k0, v0, KS, VS)
    else:
        kx, vx = oracle.page_write(src, bits(v_new), cu, start, lay.block_table, k0, v0)
    assert np.array_equal(bits(k), kx) and np.array_equal(bits(v), vx), "page write"
    assert np.array_equal(bits(kf), kx) and np.array_equal(bits(vf), vx), "fused write"


@pytest.mark.parametrize("first", [5, 40, 300])
def test_slice_of_a_longer_cu(device, first):
    """Rows `first`.. of a longer call: cu_new starts past 0, so the first page items lie
    before its first row. Both writes leave the pools of the same rows written alone."""
    print(f"[gpu-test] slice of cu from row {first}", flush=True)
    n = ([1, 17, 0, 33] * 100)[:first] + [1] * 40 + [500, 0, 16]
    rng = np.random.default_rng(43)
    start = rng.integers(0, 40, len(n)).astype(np.int32)
    lay = synth.make_layout(rng, start + np.asarray(n))
    gen = synth.value_generator(43, device)
    k, v = synth.randn_bf16((lay.num_pages, 2, 16, 128), gen, device), \
        synth.randn_bf16((lay.num_pages, 2, 128, 16), gen, device)
    kf, vf = k.clone(), v.clone()
    cu = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    k_new = synth.randn_bf16((int(cu[-1]), 2, 128), gen, device)
    v_new = synth.randn_bf16((int(cu[-1]), 2, 128), gen, device)
    k0, v0 = bits(k), bits(v)
    bt, max_pos = lay.block_table[first:], int((start + np.asarray(n))[first:].max())
    args = (i32(cu[first:], device), i32(start[first:], device))
    ra.kv_page_write(k_new, v_new, *args, ra.PagedKV(k, v, i32(bt, device)), 500, max_pos)
    ra.append_write(k_new, k_new, v_new, *args, ra.PagedKV(kf, vf, i32(bt, device)), 500, max_pos)
    torch.cuda.synchronize()
    own = slice(int(cu[first]), int(cu[-1]))
    kx, vx = oracle.page_write(bits(k_new)[own], bits(v_new)[own], cu[first:] - cu[first],
                               start[first:], bt, k0, v0)
    assert np.array_equal(bits(k), kx) and np.array_equal(bits(v), vx), "page write"
    assert np.array_equal(bits(kf), kx) and np.array_equal(bits(vf), vx), "fused write"
