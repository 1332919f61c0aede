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
    assert_attention_close(out, ref, "whole stretches", ref_abs=ref_abs if D == 128 else None)
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


def documented_cut(tiles, W, D, rows_bytes):
    """(kind, first tile and the tile behind it of every stretch), from the rules alone: stretches of c tiles, at least one tile (four, where D = 128 has
    two or three tiles a stretch anyway and the pieces would leave more than 24 MB) and so many that a request fits 256 pieces; whole requests with c tiles a
    stretch, or from c = 3 on with one more, if that takes no more than W stretches and there are no more than 256 requests."""
    total, B = int(tiles.sum()), len(tiles)
    per = -(-total // W)
    fine = per < 2 or per >= 4 or D != 128 or total <= ((24 << 20) // rows_bytes - B) * per
    least = max(1 if fine else 4, -(-int(tiles.max()) // 255))
    c = max(least, per)
    assert total < max(2 * least, 8) * W, "a line that follows the measured speeds"
    off = np.cumsum(tiles) - tiles
    for e in (c, c + 1)[: 2 if c >= 3 else 1] if c > 1 and B <= 256 else ():
        begins = np.concatenate([o + np.arange(0, t, e) for o, t in zip(off, tiles)])
        if len(begins) <= W:
            begins = np.concatenate([begins, np.full(W + 1 - len(begins), total)])
            return "whole" if e == c else "one more", np.stack([begins[:-1], begins[1:]], axis=1)
    begins = np.minimum(np.arange(W + 1) * c, total)
    return "across", np.stack([begins[:-1], begins[1:]], axis=1)


# (both planners: up to 64 requests, and more)
@pytest.mark.parametrize("kind,shape,B,tokens", [
    ("whole", (8, 1, 256, 5), 40, (64, 1500)), ("whole", (8, 1, 256, 5), 75, (64, 1400)), ("whole", (16, 2, 128, 16), 65, (100, 700)),
    ("whole", (2, 1, 64, 2), 256, (300, 700)), ("one more", (8, 8, 128, 9), 40, (100, 700)), ("one more", (16, 1, 256, 8), 20, (500, 2500)),
    ("one more", (8, 8, 64, 4), 66, (200, 500)), ("across", (8, 8, 128, 9), 64, (100, 700)), ("across", (2, 1, 64, 2), 257, (300, 700)),
    ("across", (8, 1, 128, 1), 1, (5000, 5001)), ("across", (2, 1, 256, 2), 256, (20, 60))])
@pytest.mark.parametrize("empty", [False, True])
def test_the_cut_is_the_documented_one(kind, shape, B, tokens, empty):
    """Exactly, whichever kernel plans; with requests without tiles in front, inside and at the end of the line, too."""
    from paper_2511_14617_amd import binding
    Hq, Hkv, D, T = shape
    batch = Batch(B, Hq, Hkv, D, T, tokens)
    if B > 2:
        batch.lengths[B // 2] = T                                  # one tile
    if empty and B > 8:
        batch.lengths[[0, 3, 4, B - 1]] = T - 1
    batch.ctx.copy_(torch.from_numpy(batch.lengths.astype(np.int32)))
    batch.table = torch.cat([batch.table] * (1 + 40000 // (batch.table.shape[1] * 32)), dim=1).contiguous()
    p = batch.params(B)
    assert "attn_short_kernel" not in binding.seer_verify_attention_kernel(p)
    tiles = np.where(batch.lengths < T, 0, -(-batch.lengths // 32))
    for flags in (0, binding.SEER_ATTN_GENERAL_KERNEL):
        ws = workspace(p)
        batch.call(B, ws, flags=flags)
        cut = stretches(ws, p)
        want_kind, want = documented_cut(tiles, len(cut), D, 4 * T * Hq * D)
        assert empty or want_kind == kind
        assert np.array_equal(cut, want)
