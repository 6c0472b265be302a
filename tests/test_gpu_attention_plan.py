"""The plan that the attention's own waves make for packs of at most 64 tiles
against the plan kernel: the one-call attention equals fb_attention_plan and
the planned call bit for bit (the same pieces are merged in the same order),
and leaves a workspace that the planned call accepts.  Tile capacities at the
edge of the in-wave form (64, 65) and well past it (256, 257: the plan
kernel either way), requested split sizes, several row groups, windows of
uneven length and prefixes from one block to many chunks."""
import numpy as np
import pytest
import torch

from harness import log
from paper_2607_17652_amd import binding as fb
from paper_2607_17652_amd import synth
from paper_2607_17652_amd.runner import WavefrontStep

pytestmark = pytest.mark.gpu


def _both(dtype, B, W, split, Hq=8, Hkv=4, d=64, bl=8, page=32, lo=8, hi=2048, layout="ragged",
          seed=3):
    wl = synth.workload("single", dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, d=d, bl=bl, page_size=page,
                        W_max=W, window=("uniform", 1, W), prefix=("loguniform", lo, hi),
                        layout=layout, n_blocks=max(8, W), prefix_jitter=5)
    host = synth.make_host_state(wl, seed=seed)
    t = synth.make_device_tensors(wl, host, seed, device="cuda", with_logits=False)
    step = WavefrontStep(wl, host, dict(t, logits=None))
    step.shape = fb.make_shape(Hq, Hkv, d, dtype, page, host["max_pages"], host["num_pages"],
                               kv_split=split)
    ws = fb.fb_attention_workspace_bytes(step.pack, step.shape)
    step.attn_ws = torch.full((max(ws, 16),), 0x7F, dtype=torch.uint8, device="cuda")
    step.pack_step()
    step.kv_step()
    step.out.fill_(7.0)
    step.attention_step()
    args = (t["q"], t["k_cache"], t["v_cache"], step.page_table, step.pack, step.shape)
    again = torch.full_like(step.out, 7.0)
    if dtype == "bf16":
        fb.fb_wavefront_attention_planned(*args, again, step.attn_ws)   # the one call's plan
    fresh = torch.full_like(step.attn_ws, 0x7F)
    planned = torch.full_like(step.out, 7.0)
    fb.fb_attention_plan(step.pack, step.shape, fresh)
    fb.fb_wavefront_attention_planned(*args, planned, fresh)
    torch.cuda.synchronize()
    assert fb.fb_pack_read_status(step.pack)["code"] == 0
    live = torch.from_numpy(synth_live(step)).cuda()
    assert torch.equal(step.out[live], planned[live])
    assert torch.isfinite(step.out[live].float()).all()
    if dtype == "bf16":
        assert torch.equal(again, step.out)


def synth_live(step):
    return np.flatnonzero(step.pack.view()["row_req"].cpu().numpy() >= 0)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,W", [(1, 1), (16, 4), (13, 5), (64, 4), (257, 1), (32, 8)])
def test_inline_plan_equals_the_plan_kernel(dtype, B, W):
    log(f"[plan] {dtype} B={B} W={W}")
    _both(dtype, B, W, split=0)


@pytest.mark.parametrize("split", [32, 64, 1024])
@pytest.mark.parametrize("B,W", [(3, 4), (16, 4), (40, 4)])
def test_inline_plan_requested_split(B, W, split):
    log(f"[plan] split {split} B={B} W={W}")
    _both("bf16", B, W, split=split, lo=64, hi=4096, seed=5)


@pytest.mark.parametrize("form", [
    dict(bl=96, Hq=16, Hkv=2, d=128, page=16, hi=1024),      # 6 row groups, small pages
    dict(bl=128, Hq=8, Hkv=8, d=32, page=64, hi=6000),       # one row group per head
    dict(bl=32, Hq=16, Hkv=4, d=128, page=8, layout="padded"),
])
def test_inline_plan_forms(form):
    log(f"[plan] {form}")
    _both("bf16", 16, 4, split=0, **form)


def test_inline_plan_reports_blocks_past_the_page_table():
    """A page table too short for some blocks: those are reported and left out,
    the others attended to, as by the plan kernel."""
    wl = synth.workload("single", dtype="bf16", B=6, Hq=8, Hkv=4, d=64, bl=8, page_size=32,
                        W_max=4, window=("fixed", 4), prefix=("uniform", 64, 512), n_blocks=8)
    host = synth.make_host_state(wl, seed=9)
    t = synth.make_device_tensors(wl, host, 9, device="cuda", with_logits=False)
    step = WavefrontStep(wl, host, dict(t, logits=None))
    step.pack_step()
    step.kv_step()
    log("[plan] short page table")
    short = int(np.median(host["o"])) // 32 + 1
    step.shape = fb.make_shape(8, 4, 64, "bf16", 32, short, host["num_pages"])
    step.page_table = step.page_table[:, :short].contiguous()
    out = []
    for planned in (False, True):
        step.pack_step()
        step.out.fill_(7.0)
        ws = torch.full((fb.fb_attention_workspace_bytes(step.pack, step.shape),), 0x7F,
                        dtype=torch.uint8, device="cuda")
        args = (t["q"], t["k_cache"], t["v_cache"], step.page_table, step.pack, step.shape,
                step.out, ws)
        if planned:
            fb.fb_attention_plan(step.pack, step.shape, ws)
            fb.fb_wavefront_attention_planned(*args)
        else:
            fb.fb_wavefront_attention(*args)
        torch.cuda.synchronize()
        s = fb.fb_pack_read_status(step.pack)
        out.append((step.out.clone(), s["code"], s["request"]))
    assert out[0][1] == out[1][1] == fb.FB_DERR_PAGE and out[0][2] == out[1][2]
    assert torch.equal(out[0][0], out[1][0])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,W,Hkv", [(4, 2, 8), (13, 5, 1), (16, 4, 4), (13, 5, 4)])
def test_merge_of_every_row_split(dtype, B, W, Hkv):
    """64, 65, 256 and 260 units (the edges of the merge's row counts), each in
    many pieces, against the same units in one piece: float32 sums in another
    order, and bf16 outputs rounded once (a weight's rounding to bf16 differs
    with the running maximum)."""
    wl = synth.workload("single", dtype=dtype, B=B, Hq=8, Hkv=Hkv, d=64, bl=16, page_size=32,
                        W_max=W, window=("fixed", W), prefix=("uniform", 600, 1500), n_blocks=8)
    host = synth.make_host_state(wl, seed=2)
    t = synth.make_device_tensors(wl, host, 2, device="cuda", with_logits=False)
    log(f"[plan] merge {dtype} B={B} W={W} Hkv={Hkv}")
    outs = []
    for split in (64, 1 << 14):
        step = WavefrontStep(wl, host, dict(t, logits=None), kv_split=split)
        step.pack_step()
        step.kv_step()
        step.attention_step()
        torch.cuda.synchronize()
        assert fb.fb_pack_read_status(step.pack)["code"] == 0
        outs.append(step.out.double())
    err = (outs[0] - outs[1]).norm() / outs[1].norm()
    # bf16: each of about 1000 weights is rounded by at most 2^-9, independently,
    # and the output by 2^-9; float32: a few 2^-24
    assert float(err) < (2 ** -8 if dtype == "bf16" else 1e-6)
