"""GPU parity of the fp32 kernel at the edges of its blocks (16 keys), key
slices (4 wavefronts paged, 8 packed) and column groups (16 columns)."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2608_06146_amd as pa
from _cases import TOL, decode_case, forward_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 129, 300])
@pytest.mark.parametrize("heads,d", [((1, 1), 64), ((17, 1), 128), ((28, 4), 64)])
def test_block_and_slice_edges(n, heads, d):
    """A root of n keys below a 3-token child: every remainder of blocks over
    slices, column groups with 1, 17 and 7 heads per KV head."""
    nodes = [(-1, 0, n, min(n, 5)), (0, n - n // 3, 3, 3), (0, n, 1, 1)]
    forward_case(nodes, heads[0], heads[1], d, "f32", n)
    decode_case(nodes, heads[0], heads[1], d, "f32", n)
    decode_case(nodes, heads[0], heads[1], d, "f32", n, max_chunk_keys=64)


@pytest.mark.parametrize("bad", [math.inf, math.nan])
def test_values_of_unseen_keys_stay_unseen(bad):
    """A key that one stream sees and its siblings do not, in a block they
    share: a non-finite V there reaches that stream's output alone."""
    nodes = [(-1, 0, 40, 0), (0, 40, 21, 1), (1, 20, 9, 1), (1, 3, 30, 1)]  # the stream's newest token is at 20
    Hq, Hkv, d = 8, 2, 128
    o, lse, plan, (q, kc, vc, bt, ids) = decode_case(nodes, Hq, Hkv, d, "f32", 3, check=False)
    O, L = oracle.tree_attention_paged(nodes, q, kc, vc, ids, 1 / math.sqrt(d), Hq, Hkv, 16)
    blk = int(ids[3 + 20 // 16])
    vc[blk, :, 5, 20 % 16] = bad
    o, lse = pa.branch_decode(q, kc, vc, bt, plan)
    torch.cuda.synchronize()
    e = np.abs(o.double().cpu().numpy() - O)
    assert e[1:].max() <= TOL["f32"][0]
    assert not torch.isfinite(o[0, :, 5]).any()
    assert np.delete(e[0], 5, axis=1).max() <= TOL["f32"][0]
    assert np.abs(lse.double().cpu().numpy() - L).max() <= TOL["f32"][1]
