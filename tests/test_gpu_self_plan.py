"""Batches of up to 64 requests, whose partition kernel plans for itself: its tables against the plan kernel's."""
import numpy as np
import pytest
import torch

from gpu_util import ATOL, RTOL
from paper_2511_14617_amd import workloads as W
from paper_2511_14617_amd.device_inputs import attention_device_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads", [(8, 2, 128, 16), (36, 2, 128, 32), (40, 1, 128, 64), (4, 2, 64, 20), (4, 1, 256, 16), (16, 1, 576, 32),
                                   (64, 1, 576, 64)])
@pytest.mark.parametrize("B,hi", [(1, 9), (3, 300), (63, 40), (64, 700), (65, 700), (9, 9000)])
@pytest.mark.parametrize("max_splits", [0, 2])
def test_tables_equal_the_plan_kernels(heads, B, hi, max_splits):
    """A call that forces the general kernel plans with the plan kernel, whatever its batch: after one of either kind the
    workspace holds the same slots, offsets, stretches and shared tiles, for batches on both sides of the limit, lines shorter
    and longer than the stretches, and requests with unusable lengths; and a call reuses them with equal results."""
    from paper_2511_14617_amd import binding
    Hq, Hkv, D, P = heads
    cfg = W.CONFIGS[2].scaled(B=B, group_size=3, Hq=Hq, Hkv=Hkv, T=4, Dqk=D, Dv=512 if D == 576 else D, page_size=P, ctx=("uniform", 4, hi), shared_latent=D == 576,
                              shared_prefix=2 * P if hi > 3 * P else 0)
    inp = W.make_attention_inputs(cfg)
    if B > 2:
        inp.ctx_len[B // 2] = 3                                   # fewer tokens than slots
        inp.ctx_len[B - 1] = inp.block_table.shape[1] * P + 1     # more than the table holds
    d = attention_device_inputs(inp)
    p = binding.attn_params(d["q"], d["k_pages"], d["v_pages"], d["block_table"], inp.scale, Dv=cfg.Dv, max_splits=max_splits)
    n = binding.seer_verify_attention_workspace(p)
    end = binding.load_library().seer_verify_attention_shared_tiles_offset(p) + 4 * B

    def call(ws, flags):
        return binding.seer_verify_attention(d["q"], d["k_pages"], d["v_pages"], d["block_table"], d["ctx_len"], None, inp.scale,
                                             Dv=cfg.Dv, max_splits=max_splits, workspace=ws, flags=flags).clone()
    fixed = binding.SEER_ATTN_FIXED_SPLIT
    one, other = (torch.zeros(n, dtype=torch.uint8, device="cuda") for _ in range(2))
    own = call(one, fixed)
    call(other, fixed | binding.SEER_ATTN_GENERAL_KERNEL)
    assert torch.equal(one[256:end], other[256:end])
    status = 1 if B > 2 else 0
    assert binding.seer_verify_attention_status(one) == binding.seer_verify_attention_status(other) == status
    # the same cut, planned by either kernel: the same sums in the same order
    for ws in (one, other):
        assert torch.equal(call(ws, fixed | binding.SEER_ATTN_REUSE_PLAN).view(torch.int16), own.view(torch.int16))
    # lengths that change from call to call on one workspace (lines too short to follow the speeds: test_gpu_speed_history.py has others);
    # either call is within the bar of the oracle, so they are within twice the bar of one another
    for k in range(3):
        d["ctx_len"].copy_(torch.from_numpy(np.roll(inp.ctx_len, k)).cuda().clamp_(max=int(inp.ctx_len.min()) if k == 2 else 1 << 30))
        out, want = call(one, 0).double(), call(torch.zeros_like(one), fixed | binding.SEER_ATTN_GENERAL_KERNEL).double()
        assert bool(((out - want).abs() <= 2 * (ATOL + RTOL * want.abs())).all())
        assert binding.seer_verify_attention_status(one) == (1 if B > 2 else 0)


@pytest.mark.parametrize("B", [3, 70])
@pytest.mark.parametrize("shape", [(128, 128, 2, 16), (64, 64, 2, 16), (576, 512, 1, 32)])
def test_a_page_id_outside_the_pool_is_reported_wherever_it_is(B, shape):
    """Bit 1 of the status word, by batches that plan for themselves and by others; cleared by the next good call.  The
    kernels clamp such an id to the pool."""
    from paper_2511_14617_amd import binding
    Dqk, Dv, Hkv, P = shape
    cfg = W.CONFIGS[2].scaled(B=B, group_size=B, Hq=4 * Hkv, Hkv=Hkv, T=3, Dqk=Dqk, Dv=Dv, page_size=P, ctx=("uniform", 7 * P, 9 * P),
                              shared_prefix=0, shared_latent=Dqk == 576)
    inp = W.make_attention_inputs(cfg)
    d = attention_device_inputs(inp)
    p = binding.attn_params(d["q"], d["k_pages"], d["v_pages"], d["block_table"], inp.scale, Dv=Dv)
    ws = torch.zeros(binding.seer_verify_attention_workspace(p), dtype=torch.uint8, device="cuda")
    for page, value, want in ((5, cfg_pages(d), 2), (0, None, 0), (6, -1, 2), (1, None, 0)):
        table = d["block_table"].clone()
        if value is not None:
            table[B - 2, page] = value
        binding.seer_verify_attention(d["q"], d["k_pages"], d["v_pages"], table, d["ctx_len"], None, inp.scale, Dv=Dv, workspace=ws)
        torch.cuda.synchronize()
        assert binding.seer_verify_attention_status(ws) == want, (page, value)


def cfg_pages(d):
    return int(d["k_pages"].shape[0])


@pytest.mark.parametrize("heads", [(4, 2, 4), (32, 8, 33), (8, 1, 2)])
@pytest.mark.parametrize("common", [63, 64, 65, 130, 700])
def test_long_common_prompts_only_change_how_pages_are_read(heads, common):
    """Prompts of more pages than a wave looks at in one window, beginnings and ends of pieces inside them, rows that stay equal
    behind a request's end: the same bits as from copies of the pages that no request shares."""
    from paper_2511_14617_amd import binding
    (Hq, Hkv, T), D, P, B = heads, 128, 16, 5
    gen = torch.Generator(device="cuda").manual_seed(common)
    lengths = [common * P + 3, common * P + 200, common * P // 2 + T, common * P + 1000, common * P + 40]
    pages = max(-(-n // P) for n in lengths) + 70
    table = torch.zeros((B, pages), dtype=torch.int32)
    table[:] = torch.randperm(pages, generator=torch.Generator().manual_seed(1)).int()
    for b in range(B):
        if b != 2:                                       # (request 2 ends inside the prompt)
            table[b, common:] = torch.arange(pages - common) + pages * (1 + b)
    pool = pages * (B + 1)
    k, v = (torch.randn((pool, Hkv, P, D), dtype=torch.bfloat16, device="cuda", generator=gen) for _ in range(2))
    own = torch.arange(B * pages, dtype=torch.int32).view(B, pages).cuda()
    src = table.cuda().view(-1).long()
    q = torch.randn((B, T, Hq, D), dtype=torch.bfloat16, device="cuda", generator=gen)
    ctx = torch.tensor(lengths, dtype=torch.int32, device="cuda")
    outs = [binding.seer_verify_attention(q, kk, vv, t, ctx, None, D ** -0.5, flags=binding.SEER_ATTN_FIXED_SPLIT).view(torch.int16)
            for kk, vv, t in ((k, v, table.cuda()), (k[src].contiguous(), v[src].contiguous(), own))]
    assert torch.equal(*outs)


@pytest.mark.parametrize("tiles", [(630, 0, 1290), (630, 0, 1290, 0, 0), (600, 0, 0, 1320), (0, 0, 1920), (0, 540, 0, 2, 0, 1378)])
def test_reused_plans_with_unusable_lengths_give_the_same_bits(tiles):
    """129 .. 144 rows of a KV head, where a stretch takes pairs of tiles or five waves by the number of its pieces: both kinds of
    call count requests without tiles alike (60 tiles a stretch, between twice and three times the least for pairs)."""
    from paper_2511_14617_amd import binding
    B, T, Hq, Hkv, D, P, pool = len(tiles), 33, 32, 8, 128, 32, 64
    gen = torch.Generator(device="cuda").manual_seed(B)
    q = torch.randn((B, T, Hq, D), dtype=torch.bfloat16, device="cuda", generator=gen)
    k, v = (torch.randn((pool, Hkv, P, D), dtype=torch.bfloat16, device="cuda", generator=gen) for _ in range(2))
    table = torch.randint(0, pool, (B, max(tiles)), dtype=torch.int32, device="cuda", generator=gen)
    ctx = torch.tensor([32 * t for t in tiles], dtype=torch.int32, device="cuda")
    p = binding.attn_params(q, k, v, table, D ** -0.5)
    ws = torch.zeros(binding.seer_verify_attention_workspace(p), dtype=torch.uint8, device="cuda")
    own, reused = (binding.seer_verify_attention(q, k, v, table, ctx, None, D ** -0.5, workspace=ws, flags=flags).view(torch.int16).clone()
                   for flags in (binding.SEER_ATTN_FIXED_SPLIT, binding.SEER_ATTN_FIXED_SPLIT | binding.SEER_ATTN_REUSE_PLAN))
    assert torch.equal(own, reused)
