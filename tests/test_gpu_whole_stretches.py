"""Short lines: stretches end with their request where whole requests take no more stretches than there are workgroups, and the
outputs are the same attention.  Both planners, on both sides of 64 and of 256 requests."""
import numpy as np
import pytest
import torch

from gpu_util import assert_attention_close
from test_gpu_speed_history import Batch, stretches, workspace

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,B,tokens", [
    ((8, 1, 256, 5), 40, (64, 1500)), ((8, 1, 256, 5), 75, (64, 1400)), ((16, 4, 64, 9), 48, (9, 1600)), ((16, 2, 128, 16), 65, (100, 700)),
    ((8, 1, 128, 9), 64, (64, 2000)), ((8, 1, 128, 1), 1, (5000, 5001)), ((2, 1, 64, 2), 256, (2, 600)), ((2, 1, 64, 2), 257, (2, 600)),
    ((4, 4, 128, 3), 30, (3, 900))])
def test_no_stretch_goes_on_into_the_next_request(shape, B, tokens):
    from paper_2511_14617_amd import binding
    Hq, Hkv, D, T = shape
    batch = Batch(B, Hq, Hkv, D, T, tokens)
    if B > 2:
        batch.lengths[B // 2] = T                                  # one tile
    batch.ctx.copy_(torch.from_numpy(batch.lengths.astype(np.int32)))
    # (a wide table: not a call that takes whole requests in one workgroup)
    batch.table = torch.cat([batch.table] * (1 + 40000 // (batch.table.shape[1] * 32)), dim=1).contiguous()
    p = batch.params(B)
    ws = workspace(p)
    out = batch.call(B, ws)
    # D = 128 rounds the probabilities to bf16, each by up to half a step of its 8 significant bits: beside the plain bound, 2^-9 of
    # the sum of p |v| (a row of some hundred tokens has some that carry much of the weight; one element in two million needed it)
    ref, v = batch.reference(), batch.v
    batch.v = v.abs()
    ref_abs, batch.v = batch.reference(), v
    assert_attention_close(out, ref, "whole stretches", ref_abs=ref_abs)
    other = workspace(p)
    batch.call(B, other, flags=binding.SEER_ATTN_GENERAL_KERNEL)
    cut, tiles = stretches(ws, p), -(-batch.lengths // 32)
    assert np.array_equal(cut, stretches(other, p))
    W, total, ends = len(cut), int(tiles.sum()), np.cumsum(tiles)
    assert cut[0, 0] == 0 and cut[-1, 1] == total and (cut[1:, 0] == cut[:-1, 1]).all() and (cut[:, 0] <= cut[:, 1]).all()
    if total >= 8 * W or B > 256:
        return
    longest = int((cut[:, 1] - cut[:, 0]).max())
    if sum(-(-tiles // longest)) <= W:
        used = cut[cut[:, 0] < cut[:, 1]]
        request = np.searchsorted(ends, used[:, 0], side="right")
        assert (used[:, 1] <= ends[request]).all()
