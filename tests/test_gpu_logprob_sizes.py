"""Token log-probabilities at the sizes where the kernel or the cut of the vocabulary changes.

Up to 128 tokens a row-major head goes through LDS (4 or 8 waves, 64 or 128
tokens), and so do more tokens over few rows; from 129 to 511 tokens tiles of 384 vocabulary rows fill the 256 compute
units and lower ones (128, 256 or 384 rows) take the rest, in one or two blocks of
up to 192 or 256 tokens; from 512 tokens the last round's tiles may be cut along
the tokens. Every case is compared with the fp64 oracle (tolerance as
in tests.test_gpu_logprob) and, bit for bit, with the packed head.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_18815_amd as ra
from tests.gpu_util import bits
from tests.test_gpu_logprob import check, inputs

pytestmark = pytest.mark.gpu

SIZES = [
    # N <= 128: fewer steps than the LDS ring's stages, ragged chunks, tokens at a tile's edges
    (1, 130, 64), (64, 257, 128), (65, 500, 192), (128, 1025, 320), (33, 127, 448),
    # the same over 256 chunks of 128 rows, the last of 4-wave workgroups, and the next
    (70, 32768, 64), (128, 32769, 128),
    # 129 <= N < 512, few rows: 128 x 128 tiles in two, three and four blocks of tokens
    (141, 1000, 192), (256, 16384, 64), (301, 700, 128), (384, 10880, 64), (500, 8192, 448),
    (256, 16385, 64),                       # and tiles of 192 or 256 tokens from there on
    # 129 <= N < 512 with fewer rows than one round of tiles: one height only
    (129, 1000, 192), (192, 70000, 64), (193, 98304, 64),
    # one full round of 384-row chunks, then chunks of 128, 256 and 384 rows
    (256, 98304 + 200, 64), (200, 98304 + 128 * 300, 64), (130, 98304 + 128 * 700 + 5, 64),
    # two token blocks (128 chunks a round)
    (257, 49152 + 1, 128), (384, 49152 + 128 * 200, 64), (385, 49152 + 128 * 300 + 77, 64),
    (511, 3000, 320),
    # N >= 512: the last round of tiles in 64- or 128-token parts, alone and after a full one
    (512, 1000, 64), (520, 11000, 64), (1000, 384 * 70, 64), (1000, 384 * 86 - 50, 64),
    (700, 384 * 50, 64),                    # over half a round: whole tiles
]


@pytest.mark.parametrize("N,V,D", SIZES)
def test_logprob_sizes_vs_oracle(device, N, V, D):
    print(f"[gpu-test] logprob N={N} V={V} D={D}", flush=True)
    h, W = inputs(N + V + D, N, V, D, device)
    t = np.random.default_rng(N + V).integers(0, V, size=N).astype(np.int32)
    t[-1] = V - 1
    if N > 2:
        t[:2] = [0, V]                      # the first row, and one out of range
    targets = torch.as_tensor(t, device=device)
    lp, ls = ra.token_logprob(h, W, targets, 0.9, want_lse=True)
    lq, lt = ra.token_logprob_packed(h, ra.token_logprob_pack_weight(W), V, targets, 0.9,
                                     want_lse=True)
    torch.cuda.synchronize()
    ref_lp, ref_ls = oracle.token_logprob(bits(h), bits(W), t, 0.9)
    check(lp, ls, ref_lp, ref_ls, f"N={N} V={V} D={D}")
    assert torch.equal(torch.nan_to_num(lp), torch.nan_to_num(lq)) and torch.equal(ls, lt)
