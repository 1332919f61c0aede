"""What a call promises whichever kernel the width of its block table selects: the same requests over a table of short contexts (taken
whole) and over one too wide for that (stretches and a combine kernel).  Each test asserts which kernel it runs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_14617_amd import workloads as W
from gpu_util import assert_attention_close, attention_device_inputs

pytestmark = pytest.mark.gpu

SIZES = [(128, 128), (64, 64), (256, 256), (192, 128)]
WIDE = 40000                                                   # tokens of a table that no size takes whole
# per head size: dimensions of a batch that is taken whole with more than one tile per wave where there are such batches (64, 128: 8 waves,
# 192/128: 7), the lengths and a token of the prefix that is not in its wave's first tile
WHOLE = {(128, 128): (dict(B=4, Hq=4, Hkv=2), (330, 500), 300), (64, 64): (dict(B=4, Hq=4, Hkv=2), (700, 900), 600),
         (192, 128): (dict(B=16, Hq=16, Hkv=8), (226, 250), 40), (256, 256): (dict(B=4, Hq=4, Hkv=2), (40, 64), 20)}


def _inputs(dims, tokens, whole, **kw):
    P = kw.get("page_size", 16)
    return W.make_attention_inputs(W.CONFIGS[1].scaled(Dqk=dims[0], Dv=dims[1], ctx=("uniform",) + tokens, **kw), values="peaked",
                                   max_pages_per_seq=-(-tokens[1] // P) if whole else -(-WIDE // P))


class Call:
    def __init__(self, inp, whole):
        from paper_2511_14617_amd import binding
        self.inp, self.d, self.binding = inp, attention_device_inputs(inp), binding
        d = self.d
        self.p = binding.attn_params(d["q"], d["k_pages"], d["v_pages"], d["block_table"], inp.scale, Dv=inp.cfg.Dv)
        assert ("attn_short_kernel" in binding.seer_verify_attention_kernel(self.p)) == whole
        self.ws = torch.zeros(binding.seer_verify_attention_workspace(self.p), dtype=torch.uint8, device="cuda")

    def __call__(self, flags=0, table=None, ctx=None):
        d = self.d
        return self.binding.seer_verify_attention(d["q"], d["k_pages"], d["v_pages"], d["block_table"] if table is None else table,
                                                  d["ctx_len"] if ctx is None else ctx, d["tree_mask"], self.inp.scale, Dv=self.inp.cfg.Dv,
                                                  workspace=self.ws, flags=flags).clone()

    def status(self):
        torch.cuda.synchronize()
        return self.binding.seer_verify_attention_status(self.ws)


@pytest.mark.parametrize("whole", [True, False], ids=["whole", "stretches"])
@pytest.mark.parametrize("dims", SIZES[1:], ids=lambda d: "%dx%d" % d)
def test_infinities_and_nan_in_values_reach_only_the_rows_that_see_them(dims, whole):
    """The three-term sizes, as the general kernel has them: NaN in a draft slot that most queries do not see, +inf in the last slot, -inf in a
    tile of the prefix that has no masked slots (it is found when the sums are not finite, and the tiles are taken again), a NaN key."""
    from paper_2511_14617_amd import binding
    shape, tokens, back = WHOLE[dims]
    inp = _inputs(dims, tokens, whole, T=9, tree=(2, 4), **shape)
    P, T = inp.cfg.page_size, inp.cfg.T

    def put(b, pos, d, bits):
        inp.v_pages[inp.block_table[b, pos // P], 0, pos % P, d] = bits
    put(0, int(inp.ctx_len[0]) - T + 3, slice(None), 0x7FC0)
    put(1, int(inp.ctx_len[1]) - 1, slice(0, 5), 0x7F80)
    put(2, back, 7, 0xFF80)
    put(2, 3, 9, 0x7F80)
    inp.k_pages[inp.block_table[3, 20 // P], 1, 20 % P, :] = 0x7FC0
    call = Call(inp, whole)
    got, want = call().float(), call(binding.SEER_ATTN_GENERAL_KERNEL).float()
    assert torch.isnan(want).any() and torch.isinf(want).any()
    assert torch.equal(torch.isnan(got), torch.isnan(want))
    assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)])
    ok = torch.isfinite(want)
    assert float((got[ok] - want[ok]).abs().max() / want[ok].abs().max()) < 2.0 ** -8   # a bf16 rounding of either


@pytest.mark.parametrize("whole", [True, False], ids=["whole", "stretches"])
@pytest.mark.parametrize("dims", SIZES, ids=lambda d: "%dx%d" % d)
def test_slots_past_the_end_and_unusable_lengths(dims, whole):
    """NaN in the rest of a request's last page is never read into its result; a request with an unusable length gets zeros and sets bit
    0, beside others that are not touched by it."""
    shape, tokens, _ = WHOLE[dims]
    inp = _inputs(dims, tokens, whole, T=5, **shape)
    P, B, T = inp.cfg.page_size, inp.cfg.B, inp.cfg.T
    ref = oracle.verify_attention(inp.q, inp.k_pages, inp.v_pages, inp.block_table, inp.ctx_len, None, inp.scale)
    bound = {}
    if dims == (128, 128):
        bound = dict(ref_abs=oracle.verify_attention(inp.q, inp.k_pages, inp.v_pages & np.uint16(0x7FFF), inp.block_table, inp.ctx_len, None, inp.scale))
    for b in range(B):
        n = int(inp.ctx_len[b])
        if n % P:
            pg = inp.block_table[b, (n - 1) // P]
            inp.k_pages[pg, :, n % P:, :] = inp.v_pages[pg, :, n % P:, :] = np.uint16(0x7FC0)
    call = Call(inp, whole)
    assert_attention_close(call(), ref, "past the end %s" % (dims,), hardened=True, **bound)
    assert call.status() == 0
    ctx = call.d["ctx_len"].clone()
    ctx[1], ctx[2] = T - 1, inp.block_table.shape[1] * P + 1
    out = call(ctx=ctx)
    assert call.status() == 1
    assert bool((out[1:3] == 0).all())
    rest = [b for b in range(B) if b not in (1, 2)]
    if bound:
        bound = dict(ref_abs=bound["ref_abs"][rest])
    assert_attention_close(out[rest], ref[rest], "beside unusable lengths %s" % (dims,), hardened=True, **bound)


# sizes whose table has more entries than one round of the look at them (8 per thread): four waves 2048, eight 4096
TABLES = {(128, 128): dict(B=128, Hkv=1, page_size=16, tokens=(600, 640)), (64, 64): dict(B=20, Hkv=2, page_size=1, tokens=(400, 512)),
          (256, 256): dict(B=48, Hkv=2, page_size=1, tokens=(60, 128)), (192, 128): dict(B=40, Hkv=2, page_size=1, tokens=(60, 128))}


@pytest.mark.parametrize("dims", SIZES, ids=lambda d: "%dx%d" % d)
@pytest.mark.parametrize("kind", ["whole", "whole, a small table", "stretches, planned by themselves", "stretches, plan kernel"])
def test_a_page_id_outside_the_pool_is_reported_wherever_it_is(dims, kind):
    """Bit 1 of the status word; cleared by the next good call.  Ids behind a request's end do not count."""
    whole = kind.startswith("whole")
    t = dict(TABLES[dims])
    tokens, B = t.pop("tokens"), t.pop("B")
    if kind != "whole":
        B, tokens, t["page_size"] = (70 if kind.endswith("kernel") else 3), (40, 64), 16
    inp = _inputs(dims, tokens, whole, B=B, group_size=B, Hq=4 * t["Hkv"], T=3, **t)
    call = Call(inp, whole)
    P, pool, n = inp.cfg.page_size, int(call.d["k_pages"].shape[0]), inp.ctx_len
    assert kind != "whole" or call.d["block_table"].numel() > (4096 if dims[0] <= 128 else 2048)
    used = lambda b: -(-int(n[b]) // P)  # noqa: E731
    for b, page, value, want in ((B - 2, used(B - 2) - 1, pool, 2), (0, 0, None, 0), (B - 1, used(B - 1) - 1, -1, 2), (B // 2, 1, None, 0),
                                 (0, 0, pool + 5, 2), (int(np.argmin(n)), used(int(np.argmin(n))), -7, 0)):
        table = call.d["block_table"].clone()
        if value is not None and page < table.shape[1]:
            table[b, page] = value
        call(table=table)
        assert call.status() == want, (b, page, value)


@pytest.mark.parametrize("dims", SIZES[1:], ids=lambda d: "%dx%d" % d)
def test_probabilities_reach_the_product_with_all_their_bits_in_stretches(dims):
    """The three tokens of test_gpu_attention_head_sizes.py, whose table is taken whole, over a wide one."""
    from paper_2511_14617_amd import binding
    Dqk, Dv = dims
    B, P = 64, 16
    p = np.exp(-np.arange(1, B + 1) / 64.0)
    first = torch.from_numpy(p).bfloat16().double()
    second = (torch.from_numpy(p) - first).bfloat16().double()
    want = (first + second - torch.from_numpy(p)) / (2.0 + torch.from_numpy(p))
    q, k, v = torch.zeros((B, 1, 1, Dqk)), torch.zeros((B, 1, P, Dqk)), torch.zeros((B, 1, P, Dv))
    q[..., 5] = 1.0
    k[:, 0, 1, 5] = -torch.arange(1, B + 1) / 64.0                 # exact in bf16
    v[:, 0, 0, :], v[:, 0, 1, :], v[:, 0, 2, :] = first.float()[:, None], -1.0, second.float()[:, None]
    dev = lambda x: x.bfloat16().cuda()  # noqa: E731
    n = torch.full((B,), 3, dtype=torch.int32, device="cuda")
    for columns, whole in ((1, True), (WIDE // P, False)):
        table = torch.zeros((B, columns), dtype=torch.int32, device="cuda")
        table[:, 0] = torch.arange(B, dtype=torch.int32, device="cuda")
        params = binding.attn_params(dev(q), dev(k), dev(v), table, 1.0, Dv=Dv)
        assert ("attn_short_kernel" in binding.seer_verify_attention_kernel(params)) == whole
        out = binding.seer_verify_attention(dev(q), dev(k), dev(v), table, n, None, 1.0, Dv=Dv).cpu().double()
        assert bool(((out[:, 0, 0, :] - want[:, None]).abs() <= 2.0 ** -22 + 2.0 ** -8 * want.abs()[:, None]).all())


@pytest.mark.parametrize("heads", [(8, 2, 128, 16), (36, 2, 128, 32), (4, 2, 64, 20), (4, 1, 256, 16), (8, 2, 192, 16)])
@pytest.mark.parametrize("B,hi", [(1, 9), (3, 300), (63, 40), (64, 700), (9, 1400)])
def test_partition_kernels_plan_as_the_plan_kernel_does(heads, B, hi):
    """Slots, offsets, stretches and shared tiles of short lines with unusable lengths, by a partition kernel that plans for itself and by
    the plan kernel (a call that forces the general kernel); and calls that reuse either plan give the same bits."""
    from paper_2511_14617_amd import binding
    Hq, Hkv, D, P = heads
    inp = _inputs((D, 128 if D == 192 else D), (4, hi), False, B=B, group_size=3, Hq=Hq, Hkv=Hkv, T=4, page_size=P, shared_prefix=2 * P if hi > 3 * P else 0)
    if B > 2:
        inp.ctx_len[B // 2], inp.ctx_len[B - 1] = 3, inp.block_table.shape[1] * P + 1
    one, other = Call(inp, False), Call(inp, False)
    fixed = binding.SEER_ATTN_FIXED_SPLIT
    own = one(fixed)
    other(fixed | binding.SEER_ATTN_GENERAL_KERNEL)
    end = binding.load_library().seer_verify_attention_shared_tiles_offset(one.p) + 4 * B
    assert torch.equal(one.ws[256:end], other.ws[256:end])
    assert one.status() == other.status() == (1 if B > 2 else 0)
    for call in (one, other):
        assert torch.equal(call(fixed | binding.SEER_ATTN_REUSE_PLAN).view(torch.int16), own.view(torch.int16))
