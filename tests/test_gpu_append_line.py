"""GPU parity of the append when few tiles are cut into equal shares of key blocks.

With fewer, longer tiles than fill the GPU, the append cuts the key blocks of all
(KV head, query block) tiles into equal shares and merges the pieces of a tile
(any call here whose longest tile is over 16 blocks of 64 keys longer than a
share). The cases put share ends inside tiles, at their ends and across KV heads,
leave waves and whole query blocks without queries, and cover group sizes from 1
to 32; each is compared with the fp64 oracle, and the mixed call's append part
must be bitwise the same. Pieces are merged in fp32, so the attention tolerance
of tests.gpu_util holds unchanged.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2603_18815_amd as ra
import synth
from tests.gpu_util import APPEND_LSE_ATOL, assert_attn_close, bits
from tests.test_gpu_rope import rope_table

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)


def i32(x, dev):
    return torch.as_tensor(np.ascontiguousarray(np.asarray(x, np.int32)), device=dev)


# (Hq, Hkv, ctx, T): 17 blocks in one tile up to many tiles per row
CASES = [
    (8, 2, [1088], [1]),                       # two tiles of 18 blocks, one query each
    (32, 8, [4000], [65]),                     # a second query block with one query
    (32, 8, [4096 - 64], [64]),                # whole blocks: shares end at tile ends
    (8, 8, [5000], [257]),                     # groups of one: 256 queries per tile
    (32, 1, [3000], [20]),                     # groups of 32: 8 queries per tile
    (15, 3, [2500, 1800], [52, 7]),            # groups of 5 (51 per tile), 3 KV heads
    (32, 8, [6000, 0, 40, 3000], [3, 70, 0, 1]),   # short, context-free and empty rows among them
    (4, 1, [20000], [16]),                     # one tile of 313 blocks over all shares
]


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("Hq,Hkv,ctx,T", CASES)
def test_cut_tiles_vs_oracle(device, Hq, Hkv, ctx, T, fp8):
    print(f"[gpu-test] append line Hq={Hq} Hkv={Hkv} ctx={ctx} T={T} fp8={fp8}", flush=True)
    w = synth.append_workload(17, len(T), Hq, Hkv, lambda r, n: np.asarray(ctx),
                              lambda r, n: np.asarray(T), "append line")
    t = synth.make_tensors(w, device)
    k, v, scales = t.k_pool, t.v_pool, ()
    if fp8:
        gen = synth.value_generator(18, device)
        scales = (0.02, 0.015)
        k = synth.randn_fp8_codes(t.k_pool.shape, gen, device, scales[0])
        v = synth.randn_fp8_codes(t.v_pool.shape, gen, device, scales[1])
    kv = ra.PagedKV(k, v, i32(w.append_table(), device), *scales)
    synth.poison_unowned(k, v, w.layout, rows=w.append_rows, lens=w.ctx_lens + w.q_lens)
    args = (t.q_append, i32(w.cu_q(), device), i32(w.ctx_lens, device))
    mq, mk = max(T), int(max(c + n for c, n in zip(ctx, T)))
    out, lse = ra.append(*args, kv, mq, mk, SCALE, want_lse=True)
    again, _ = ra.append(*args, kv, mq, mk, SCALE)
    # one decode row over the first row's cache, beside the same append rows
    od, oa, _, la = ra.mixed(t.q_append[:1], kv, i32([ctx[0]], device), *args, kv, ctx[0], mq, mk,
                             SCALE, want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(out, again), "not deterministic"
    assert torch.equal(oa, out) and torch.equal(la, lse), "append part of mixed() differs"
    if fp8:
        ref, ref_lse = oracle.append_fp8(bits(t.q_append), w.cu_q(), w.ctx_lens, bits(k), bits(v),
                                         *scales, w.append_table(), SCALE)
    else:
        ref, ref_lse = oracle.append(bits(t.q_append), w.cu_q(), w.ctx_lens, bits(k), bits(v),
                                     w.append_table(), SCALE)
    assert_attn_close(out.cpu().numpy(), ref, "append line")
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, atol=APPEND_LSE_ATOL, rtol=0)


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("Hq,Hkv,ctx,T", [(32, 8, 6000, 70), (8, 1, 3001, 33), (6, 6, 2100, 257)])
def test_cut_tile_is_the_uncut_tile(device, Hq, Hkv, ctx, T, fp8, rope):
    """A row alone (its tiles cut) and among so many copies of itself that none is.

    Both round the same weights to bf16 against the same reference, so they differ by
    the order of fp32 sums over the n <= 6,070 keys: each output and each weight sum is a
    sum of n terms, off by at most about n 2^-24 of the sum of their magnitudes, in practice
    sqrt(n) 2^-24 = 5e-6. Weights rounded against another reference differ by 2e-3.
    """
    tiles = -(-T // (256 // (Hq // Hkv)))
    longest, least = -(-(ctx + T) // 64), -(-ctx // 64)
    copies = 256 * longest // (least * tiles * Hkv) + 1       # a line longer than any cut
    print(f"[gpu-test] cut tile Hq={Hq} Hkv={Hkv} ctx={ctx} T={T} fp8={fp8} rope={rope}", flush=True)
    gen = synth.value_generator(19, device)
    lay = synth.make_layout(np.random.default_rng(19), np.asarray([ctx + T]))
    scales = (0.02, 0.015) if fp8 else ()
    make = (lambda s: synth.randn_fp8_codes(s, gen, device, 0.02)) if fp8 else \
        (lambda s: synth.randn_bf16(s, gen, device))
    k, v = make((lay.num_pages, Hkv, 16, 128)), make((lay.num_pages, Hkv, 128, 16))
    q = synth.randn_bf16((T, Hq, 128), gen, device)
    new = synth.randn_bf16((T, Hkv, 128), gen, device)
    cs = torch.from_numpy(rope_table(1e6, ctx + T)).to(device) if rope else None

    def call(n):
        kv = ra.PagedKV(k, v, i32(np.repeat(lay.block_table, n, 0), device), *scales)
        # every copy writes the same tokens to the same pages
        return ra.append_write(q.repeat(n, 1, 1), new.repeat(n, 1, 1), new.repeat(n, 1, 1),
                               i32(np.arange(n + 1) * T, device), i32([ctx] * n, device), kv, T,
                               ctx + T, SCALE, want_lse=True, cos_sin=cs)
    one, lse = call(1)
    many, lse_many = call(copies)
    torch.cuda.synchronize()
    whole = many[:T].double()
    assert torch.equal(many[-T:], many[:T])
    rel = ((one.double() - whole).norm() / whole.norm()).item()
    print(f"[parity] cut against uncut: rel_l2={rel:.2e}", flush=True)
    assert rel <= 2e-5
    assert (lse - lse_many[:T]).abs().max().item() <= 2e-5


@pytest.mark.parametrize("B,Hq,Hkv,ctx,T", [(100, 8, 1, 8000, 32), (70, 16, 2, 12800, 20),
                                            (1100, 4, 1, 1200, 1)])
def test_many_equal_rows_repeat(device, B, Hq, Hkv, ctx, T):
    """More equal rows than a wave has lanes, cut: every row keeps its place from call to call.

    Rows of one length share a bucket of the plan's sort; a row's place among them decides
    where it is cut, so its bits. The last row is long (its tiles make the call one that is
    cut), the others share its pages and have queries of their own.
    """
    print(f"[gpu-test] many equal rows B={B} Hkv={Hkv} ctx={ctx} T={T}", flush=True)
    gen = synth.value_generator(20, device)
    long = 64 * (16 + -(-B * Hkv * (ctx // 64 + 1) // 256) + 2) + ctx    # a line shorter than 256 x it
    lay = synth.make_layout(np.random.default_rng(20), np.asarray([long + T]))
    k = synth.randn_bf16((lay.num_pages, Hkv, 16, 128), gen, device)
    v = synth.randn_bf16((lay.num_pages, Hkv, 128, 16), gen, device)
    kv = ra.PagedKV(k, v, i32(np.repeat(lay.block_table, B, 0), device))
    q = synth.randn_bf16((B * T, Hq, 128), gen, device)
    lens = [ctx] * (B - 1) + [long]
    args = (q, i32(np.arange(B + 1) * T, device), i32(lens, device), kv)
    out, lse = ra.append(*args, T, long + T, SCALE, want_lse=True)
    one = ra.PagedKV(k, v, i32(lay.block_table, device))
    for _ in range(8):
        again, lse2 = ra.append(*args, T, long + T, SCALE, want_lse=True)
        _, mixed, _, _ = ra.mixed(q[:1], one, i32([ctx], device), *args, ctx, T, long + T, SCALE)
        torch.cuda.synchronize()
        assert torch.equal(out, again) and torch.equal(lse, lse2), "not deterministic"
        assert torch.equal(out, mixed), "append part of mixed() differs"
    rows = [0, 1, B // 2, B - 2, B - 1]
    pick = np.concatenate([np.arange(b * T, (b + 1) * T) for b in rows])
    sel = bits(q)[pick]
    ref, _ = oracle.append(sel, np.arange(len(rows) + 1) * T, np.asarray(lens)[rows], bits(k), bits(v),
                           np.repeat(lay.block_table, len(rows), 0), SCALE)
    assert_attn_close(out.cpu().numpy()[pick], ref, "many equal rows")


@pytest.mark.parametrize("Hq,Hkv,T", [(32, 8, 1), (32, 8, 63), (32, 8, 65), (5, 1, 1), (15, 3, 52), (32, 1, 9)])
def test_cut_tiles_stay_in_the_workspace(device, Hq, Hkv, T):
    """A workspace of exactly the asked size: the pieces, as large as the call's fullest tile,
    overlap nothing and reach no further."""
    print(f"[gpu-test] append line workspace Hq={Hq} Hkv={Hkv} T={T}", flush=True)
    w = synth.append_workload(27, 2, Hq, Hkv, lambda r, n: np.asarray([5000, 3000]),
                              lambda r, n: np.asarray([T, T]), "append line workspace")
    t = synth.make_tensors(w, device)
    kv = ra.PagedKV(t.k_pool, t.v_pool, i32(w.append_table(), device))
    size = ra.append_workspace_size(2, Hq, Hkv, T)
    ws = torch.full((size + 4096,), 255, dtype=torch.uint8, device=device)
    out, lse = ra.append(t.q_append, i32(w.cu_q(), device), i32(w.ctx_lens, device), kv, T, 5000 + T,
                         SCALE, want_lse=True, workspace=ws[:size])
    torch.cuda.synchronize()
    assert torch.all(ws[size:] == 255), "written past the workspace"
    ref, ref_lse = oracle.append(bits(t.q_append), w.cu_q(), w.ctx_lens, bits(t.k_pool),
                                 bits(t.v_pool), w.append_table(), SCALE)
    assert_attn_close(out.cpu().numpy(), ref, "append line workspace")
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, atol=APPEND_LSE_ATOL, rtol=0)
