"""GPU parity of decode at the sizes where its split and its merge change.

Rows of up to 512 keys are one split whose result is final; longer ones are split
into at least 128 keys, more finely the fewer rows and KV heads there are, and
merged a thread per dim (up to 8 slots a row, and with many rows and heads) or one
slot per lane in rounds of 64. Each case states the slots that its call plans.
Each call mixes lengths (empty rows and single keys among them) and is compared
with the fp64 oracle at the decode tolerance; the same rows as one-row groups
without a shared prefix must give the same bits.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2603_18815_amd as ra
import synth
from tests.gpu_util import DECODE_LSE_ATOL, assert_attn_close, bits

pytestmark = pytest.mark.gpu
SCALE = 1.0 / math.sqrt(128)

# (Hq, Hkv, lengths, slots of the longest row: splits of 128, 256 or 512 keys)
CASES = [
    (8, 2, [256, 0, 1, 511, 512, 33], 1),    # final splits, an empty row
    (17, 1, [512, 0, 100], 1),               # the same in two 16-column tiles
    (4, 4, [513, 0, 128, 129, 512], 5),
    (8, 1, [1024, 1000, 31], 8),             # the last small merge
    (8, 1, [1152, 1025, 1024], 9),           # the first larger one, and a small one beside it
    (8, 1, [4096, 4000, 1], 32),
    (8, 1, [1025, 4000, 4097], 17),          # 256-key splits
    (4, 1, [16896, 16385, 512], 33),         # 512-key splits
    (32, 1, [8192, 8193, 0, 5], 17),         # two tiles
    (32, 1, [4000] * 15 + [3999], 16),       # two tiles, more rows: 256 keys where 128 would do
    (1, 1, [20000, 17], 40),
    (1, 1, [32769, 32768, 32256], 65),       # a round of 64 slots in the merge, one less, one more
    (2, 1, [65600, 40], 129),                # a third round
    (32, 8, [16000, 16001], 32),             # more heads: longer splits
    # over 1,024 (row, head) pairs: a thread per dim, eight slots at a time
    (64, 4, [4700, 4097, 4096, 513, 0, 1] * 2 + [1000, 2, 3, 4, 5], 10),
]


def i32(x, dev):
    return torch.as_tensor(np.ascontiguousarray(np.asarray(x, np.int32)), device=dev)


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("Hq,Hkv,lens,slots", CASES)
def test_decode_splits_vs_oracle(device, Hq, Hkv, lens, slots, fp8):
    print(f"[gpu-test] decode splits Hq={Hq} Hkv={Hkv} lens={lens} fp8={fp8}", flush=True)
    w = synth.decode_workload(23, len(lens), Hq, Hkv, lambda r, n: np.asarray(lens), "splits")
    t = synth.make_tensors(w, device)
    k, v, scales = t.k_pool, t.v_pool, ()
    if fp8:
        gen = synth.value_generator(24, device)
        scales = (0.02, 0.015)
        k = synth.randn_fp8_codes(k.shape, gen, device, scales[0])
        v = synth.randn_fp8_codes(v.shape, gen, device, scales[1])
    synth.poison_unowned(k, v, w.layout)
    kv = ra.PagedKV(k, v, i32(w.decode_table(), device), *scales)
    kl, mk, B = i32(lens, device), max(lens), len(lens)
    assert ra.decode_workspace_size(B, Hq, Hkv, mk) == B * Hq * slots * 130 * 4
    out, lse = ra.decode(t.q_decode, kv, kl, mk, SCALE, want_lse=True)
    out2 = torch.empty_like(out)
    ra.decode_noalloc(t.q_decode, kv, kl, mk, out2, SCALE)
    groups = i32(np.arange(B + 1), device)
    out3, lse3 = ra.decode_shared_prefix(t.q_decode, kv, kl, groups, i32([0] * B, device), 1, 0, mk,
                                         SCALE, want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(out, out2), "no-allocation decode differs"
    assert torch.equal(out, out3) and torch.equal(lse, lse3), "one-row groups differ"
    if fp8:
        ref, ref_lse = oracle.decode_fp8(bits(t.q_decode), bits(k), bits(v), *scales,
                                         w.decode_table(), np.asarray(lens), SCALE)
    else:
        ref, ref_lse = oracle.decode(bits(t.q_decode), bits(k), bits(v), w.decode_table(),
                                     np.asarray(lens), SCALE)
    rows = np.asarray(lens) > 0
    assert torch.all(out[~rows] == 0) and torch.all(torch.isneginf(lse[~rows]))
    assert_attn_close(out.cpu().numpy()[rows], ref[rows], "decode splits")
    np.testing.assert_allclose(lse.cpu().numpy()[rows], ref_lse[rows], atol=DECODE_LSE_ATOL, rtol=0)


@pytest.mark.parametrize("B,Hkv,mk,rows", [(9, 1, 4096, 16), (3, 8, 4096, 4), (5, 8, 1000, 9), (1, 2, 4096, 1)])
def test_workspace_of_other_shapes(device, B, Hkv, mk, rows):
    """A workspace that holds splits of 512 keys for the call's rows, such as one sized for
    more rows, is enough: the shorter splits are taken only as far as it holds them."""
    print(f"[gpu-test] workspace of other shapes B={B} Hkv={Hkv} mk={mk}", flush=True)
    Hq = 4 * Hkv
    lens = np.linspace(mk, 1, B).astype(np.int64)
    w = synth.decode_workload(25, B, Hq, Hkv, lambda r, n: lens, "ws")
    t = synth.make_tensors(w, device)
    kv = ra.PagedKV(t.k_pool, t.v_pool, i32(w.decode_table(), device))
    kl = i32(lens, device)
    slots = (mk + 511) // 512
    least = B * Hq * slots * 130 * 4
    full = ra.decode_workspace_size(B, Hq, Hkv, mk)
    assert full > least
    ref, ref_lse = oracle.decode(bits(t.q_decode), bits(t.k_pool), bits(t.v_pool),
                                 w.decode_table(), lens, SCALE)
    for size in {least, min(full, max(least, ra.decode_workspace_size(rows, Hq, Hkv, mk)))}:
        ws = torch.full((size + 4096,), 255, dtype=torch.uint8, device=device)
        out, lse = ra.decode(t.q_decode, kv, kl, mk, SCALE, want_lse=True, workspace=ws[:size])
        torch.cuda.synchronize()
        assert torch.all(ws[size:] == 255), "written past the workspace"
        assert_attn_close(out.cpu().numpy(), ref, "smaller workspace")
        np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, atol=DECODE_LSE_ATOL, rtol=0)
        two = i32([0, (B + 1) // 2, B] if B > 1 else [0, 1], device)
        ng = two.numel() - 1
        same = ra.decode_shared_prefix(t.q_decode, kv, kl, two, i32([0] * ng, device),
                                       (B + 1) // 2, 0, mk, SCALE, workspace=ws[:size])[0]
        assert torch.equal(same, out), "groups without a prefix differ"
    ws = torch.empty(least - 1, dtype=torch.uint8, device=device)
    with pytest.raises(ra.RolloutAttnError, match="RA_ERR_WORKSPACE"):
        ra.decode(t.q_decode, kv, kl, mk, SCALE, workspace=ws)
