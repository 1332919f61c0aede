"""GPU parity of the matrix-core kernel for head sizes (64, 64), (256, 256) and (192, 128): edges of tiles, pages and row
blocks against the oracle, and infinities or NaN in V against the general kernel.  Probabilities keep fp32's precision there
(three bf16 terms), so what is left is the rounding of the bf16 output: at most 2^-9 of each value, hence of the signal's rms."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_14617_amd import workloads as W
from gpu_util import assert_attention_close, attention_device_inputs, attention_margin

pytestmark = pytest.mark.gpu

SIZES = [(64, 64), (256, 256), (192, 128)]


def _call(inp, **kw):
    from paper_2511_14617_amd import binding
    d = attention_device_inputs(inp)
    out = binding.seer_verify_attention(d["q"], d["k_pages"], d["v_pages"], d["block_table"], d["ctx_len"], d["tree_mask"],
                                        inp.scale, Dv=inp.cfg.Dv, **kw)
    torch.cuda.synchronize()
    return out


def _cfg(dims, **kw):
    return W.CONFIGS[1].scaled(Dqk=dims[0], Dv=dims[1], **kw)


# pages of one token, odd sizes, larger than a tile; one row, a full wave, one row more, the most rows of one workgroup and
# two row blocks; contexts shorter than a tile, at its edges, of several window loads of the block table
SHAPES = {
    "page1": dict(B=3, Hq=4, Hkv=2, T=3, page_size=1, ctx=("uniform", 3, 300)),
    "page7_tree": dict(B=4, Hq=4, Hkv=1, T=9, tree=(2, 4), page_size=7, ctx=("uniform", 9, 700)),
    "page48": dict(B=3, Hq=6, Hkv=3, T=5, page_size=48, ctx=("uniform", 5, 400)),
    "page2048": dict(B=2, Hq=4, Hkv=2, T=5, page_size=2048, ctx=("uniform", 900, 2500)),
    "decode_T1_G1": dict(B=6, Hq=2, Hkv=2, T=1, page_size=16, ctx=("uniform", 1, 70)),
    "tile_edges": dict(B=5, Hq=8, Hkv=2, T=8, page_size=16, ctx=("fixed", (8, 31, 32, 33, 64))),
    "rows33": dict(B=2, Hq=3, Hkv=1, T=11, page_size=16, ctx=("uniform", 11, 500)),
    "rows128_129": dict(B=2, Hq=3, Hkv=1, T=43, page_size=16, ctx=("uniform", 43, 300)),
    "rows256_T64": dict(B=2, Hq=4, Hkv=1, T=64, page_size=32, ctx=("uniform", 64, 300)),
    "rows520_row_blocks": dict(B=2, Hq=16, Hkv=2, T=64, tree=(7, 9), page_size=16, ctx=("uniform", 64, 300)),
    "many_short": dict(B=200, group_size=4, Hq=4, Hkv=2, T=2, page_size=16, ctx=("uniform", 2, 90)),
    "long": dict(B=2, Hq=4, Hkv=1, T=4, page_size=8, ctx=("uniform", 6000, 9000)),
}


@pytest.mark.parametrize("dims", SIZES, ids=lambda d: "%dx%d" % d)
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_parity(name, dims):
    from paper_2511_14617_amd import binding
    fixed = SHAPES[name]["ctx"][0] == "fixed"
    inp = W.make_attention_inputs(_cfg(dims, **SHAPES[name]), values="peaked", max_pages_per_seq=4 if fixed else None)
    ref = oracle.verify_attention(inp.q, inp.k_pages, inp.v_pages, inp.block_table, inp.ctx_len, inp.tree_mask, inp.scale, Dv=dims[1])
    for flags, splits in ((0, 0), (binding.SEER_ATTN_FIXED_SPLIT, 2), (0, 1)):
        out = _call(inp, flags=flags, max_splits=splits)
        assert_attention_close(out, ref, "%s %s splits %d" % (name, dims, splits), hardened=True)
        assert attention_margin(out.float().cpu().numpy().astype(np.float64), ref)["nrms"] < 2.0 ** -9


@pytest.mark.parametrize("dims", SIZES, ids=lambda d: "%dx%d" % d)
@pytest.mark.parametrize("max_splits", [0, 1])
def test_a_plan_serves_calls_whose_flags_differ(dims, max_splits):
    """The matrix-core and the general kernel share the workspace's layout, so either runs on the other's plan."""
    from paper_2511_14617_amd import binding
    # three row blocks at least: where a layout that followed the flag would differ most
    inp = W.make_attention_inputs(_cfg(dims, B=5, Hq=32, Hkv=2, T=33, tree=(4, 8), ctx=("uniform", 33, 900)), values="peaked")
    d = attention_device_inputs(inp)
    kinds = (0, binding.SEER_ATTN_GENERAL_KERNEL)
    args = (d["q"], d["k_pages"], d["v_pages"], d["block_table"], d["ctx_len"], d["tree_mask"], inp.scale)
    sizes = [binding.seer_verify_attention_workspace(binding.attn_params(d["q"], d["k_pages"], d["v_pages"], d["block_table"], inp.scale,
                                                                         dims[1], max_splits, f)) for f in kinds]
    assert sizes[0] == sizes[1]
    ws = torch.empty(sizes[0], dtype=torch.uint8, device="cuda")
    want = binding.seer_verify_attention(*args, Dv=dims[1], max_splits=max_splits).float()
    for plan in kinds:
        for use in kinds:
            binding.seer_verify_attention(*args, Dv=dims[1], max_splits=max_splits, workspace=ws, flags=plan)
            got = binding.seer_verify_attention(*args, Dv=dims[1], max_splits=max_splits, workspace=ws,
                                                flags=use | binding.SEER_ATTN_REUSE_PLAN).float()
            assert float((got - want).abs().max() / want.abs().max()) < 2.0 ** -8   # a bf16 rounding of either


@pytest.mark.parametrize("dims", SIZES, ids=lambda d: "%dx%d" % d)
def test_infinities_and_nan_in_values_reach_only_the_rows_that_see_them(dims):
    """As the general kernel has it: a draft slot that a query does not see must not touch it whatever its V row holds, and
    an infinite V at a visible position gives that infinity."""
    from paper_2511_14617_amd import binding
    inp = W.make_attention_inputs(_cfg(dims, B=4, Hq=4, Hkv=2, T=9, tree=(2, 4), ctx=("uniform", 150, 400)), values="peaked")
    P, T = inp.cfg.page_size, inp.cfg.T

    def put(b, pos, d, bits):
        inp.v_pages[inp.block_table[b, pos // P], 0, pos % P, d] = bits

    put(0, int(inp.ctx_len[0]) - T + 3, slice(None), 0x7FC0)      # a draft slot of one path: NaN
    put(1, int(inp.ctx_len[1]) - 1, slice(0, 5), 0x7F80)          # the last slot: +inf in a few columns
    put(2, 40, 7, 0xFF80)                                         # far back in the prefix: -inf
    inp.k_pages[inp.block_table[3, 20 // P], 1, 20 % P, :] = 0x7FC0   # a NaN key: every row of that head
    want = _call(inp, flags=binding.SEER_ATTN_GENERAL_KERNEL).float()
    got = _call(inp).float()
    assert torch.isnan(want).any() and torch.isinf(want).any()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)])
    ok = torch.isfinite(want)
    assert torch.isfinite(got[ok]).all()
    assert float((got[ok] - want[ok]).abs().max() / want[ok].abs().max()) < 2.0 ** -8   # a bf16 rounding of either


@pytest.mark.parametrize("dims", SIZES, ids=lambda d: "%dx%d" % d)
def test_probabilities_reach_the_product_with_all_their_bits(dims):
    """Three tokens: two of weight 1 whose values are the first and the second bf16 term of the third one's weight p = exp(-j / 64),
    and the third with value -1.  What is left is the part of p behind 16 bits, over 2 + p.  In fp32, p is off by its exponent's
    rounding (below 2^-23 here) and the exponential's (2^-23), together less than 2^-22; the output is rounded to bf16."""
    from paper_2511_14617_amd import binding
    Dqk, Dv = dims
    B, P = 64, 16
    p = np.exp(-np.arange(1, B + 1) / 64.0)
    first = torch.from_numpy(p).bfloat16().double()
    second = (torch.from_numpy(p) - first).bfloat16().double()
    want = (first + second - torch.from_numpy(p)) / (2.0 + torch.from_numpy(p))
    q = torch.zeros((B, 1, 1, Dqk))
    k, v = torch.zeros((B, 1, P, Dqk)), torch.zeros((B, 1, P, Dv))
    q[..., 5] = 1.0
    k[:, 0, 1, 5] = -torch.arange(1, B + 1) / 64.0                 # exact in bf16
    v[:, 0, 0, :], v[:, 0, 1, :], v[:, 0, 2, :] = first.float()[:, None], -1.0, second.float()[:, None]
    dev = lambda x: x.bfloat16().cuda()  # noqa: E731
    table = torch.arange(B, dtype=torch.int32, device="cuda").view(B, 1)
    n = torch.full((B,), 3, dtype=torch.int32, device="cuda")
    out = binding.seer_verify_attention(dev(q), dev(k), dev(v), table, n, None, 1.0, Dv=Dv).cpu().double()
    assert float(want.abs().max()) > 2.0 ** -20                   # so that two terms alone, which leave zero, are far outside
    assert bool(((out[:, 0, 0, :] - want[:, None]).abs() <= 2.0 ** -22 + 2.0 ** -8 * want.abs()[:, None]).all())
