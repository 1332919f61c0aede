"""Calls that take whole requests (block tables of short contexts): edges of tiles, waves and row blocks against the oracle, and the
same requests with a table too wide for that, so that the partition kernels take them."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_14617_amd import workloads as W
from gpu_util import assert_attention_close, attention_device_inputs

pytestmark = pytest.mark.gpu

SIZES = [(128, 128), (64, 64), (256, 256), (192, 128)]
# one and two tiles per wave (four waves up to 128 tokens, else eight), row blocks of 1, 32, 33 and 64 rows, lengths at the
# edges of tiles, of a wave's tiles and of the table, lengths that cannot be used; wide heads are taken whole up to 128 tokens
SHAPES = {
    "one_tile_rows1": dict(B=3, Hq=2, Hkv=2, T=1, ctx=("fixed", (1, 31, 32))),
    "four_waves": dict(B=6, Hq=8, Hkv=2, T=8, ctx=("fixed", (8, 33, 64, 97, 127, 128))),
    "rows33": dict(B=5, Hq=3, Hkv=1, T=11, ctx=("fixed", (11, 225, 256, 257, 290))),
    "rows64_tree": dict(B=9, Hq=16, Hkv=2, T=8, tree=(1, 7), ctx=("uniform", 8, 500)),
    "several_tiles": dict(B=16, Hq=16, Hkv=8, T=5, ctx=("uniform", 300, 512)),
    "batch_70": dict(B=70, Hq=4, Hkv=1, T=9, tree=(2, 4), ctx=("uniform", 9, 450)),
    "common_prompt": dict(B=12, group_size=6, Hq=8, Hkv=2, T=3, ctx=("uniform", 140, 400), shared_prefix=128),
}


@pytest.mark.parametrize("dims", SIZES, ids=lambda d: "%dx%d" % d)
@pytest.mark.parametrize("page", [16, 64, 7])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_whole_requests_against_the_oracle_and_the_partition_kernels(name, page, dims):
    from paper_2511_14617_amd import binding
    if dims == (128, 128) and page == 7:
        page = 32                                              # (heads of 128: powers of two from 16 on)
    kw = SHAPES[name]
    if page > 16 and "shared_prefix" in kw:
        kw = dict(kw, shared_prefix=2 * page)
    most = (512 if dims[0] <= 128 else 128) // page * page
    kw = dict(kw, ctx=("fixed", tuple(min(n, most) for n in kw["ctx"][1])) if kw["ctx"][0] == "fixed" else ("uniform", min(kw["ctx"][1], most // 2), min(kw["ctx"][2], most)))
    if "shared_prefix" in kw and dims[0] > 128:
        kw["shared_prefix"] = page
    cfg = W.CONFIGS[1].scaled(Dqk=dims[0], Dv=dims[1], page_size=page, **kw)
    pages = -(-(max(cfg.ctx[1]) if cfg.ctx[0] == "fixed" else cfg.ctx[2]) // page)

    def whole(cfg, pages):
        return "attn_short_kernel" in binding.seer_verify_attention_kernel(binding.SeerAttnParams(
            B=cfg.B, T=cfg.T, Hq=cfg.Hq, Hkv=cfg.Hkv, Dqk=cfg.Dqk, Dv=cfg.Dv, page_size=page, num_pages=1, max_pages_per_seq=pages, scale=1.0))
    for _ in range(4):                                         # (wide heads are taken whole where there are many of them)
        if not whole(cfg, pages):
            cfg = cfg.scaled(Hq=2 * cfg.Hq, Hkv=2 * cfg.Hkv)
    inp = W.make_attention_inputs(cfg, values="peaked", max_pages_per_seq=pages)
    B, T = inp.cfg.B, inp.cfg.T
    bad = [1, B - 1] if name == "batch_70" else []
    if bad:
        inp.ctx_len[1], inp.ctx_len[B - 1] = T - 1, inp.block_table.shape[1] * page + 1
    ok = [b for b in range(B) if b not in bad]

    def reference(v):
        ref = np.zeros((B, T, inp.cfg.Hq, dims[1]))
        ref[ok] = oracle.verify_attention(inp.q[ok], inp.k_pages, v, inp.block_table[ok], inp.ctx_len[ok],
                                          None if inp.tree_mask is None else inp.tree_mask[ok], inp.scale)
        return ref
    ref = reference(inp.v_pages)
    bound = dict(hardened=True, ref_abs=reference(inp.v_pages & np.uint16(0x7FFF))) if dims == (128, 128) else {}
    d = attention_device_inputs(inp)
    wide = torch.zeros((B, -(-40000 // page)), dtype=torch.int32, device="cuda")
    wide[:, : d["block_table"].shape[1]] = d["block_table"]
    for table, short in ((d["block_table"], True), (wide, False)):
        assert whole(cfg, table.shape[1]) == short
        p = binding.attn_params(d["q"], d["k_pages"], d["v_pages"], table, inp.scale, Dv=dims[1])
        ws = torch.randint(0, 256, (binding.seer_verify_attention_workspace(p),), dtype=torch.uint8, device="cuda")
        ctx = d["ctx_len"].clone()
        if bad and not short:
            ctx[B - 1] = wide.shape[1] * page + 1
        outs = [binding.seer_verify_attention(d["q"], d["k_pages"], d["v_pages"], table, ctx, d["tree_mask"], inp.scale, Dv=dims[1],
                                              workspace=ws, flags=flags).clone() for flags in (binding.SEER_ATTN_FIXED_SPLIT, binding.SEER_ATTN_REUSE_PLAN)]
        torch.cuda.synchronize()
        assert binding.seer_verify_attention_status(ws) == (1 if bad else 0)
        assert_attention_close(outs[0], ref, "%s %s short=%s" % (name, dims, short), **bound)
        assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
