"""The attention over pages smaller than a key tile (8 and 16 keys, several
per tile) against pages that hold whole tiles: the same keys in the same order,
so outputs are equal bit for bit.  Prefixes end at every place of a page, the
last page of a block is partly filled (with NaN past the block's keys), and a
page id outside the cache is reported."""
import numpy as np
import pytest
import torch

from harness import log
from paper_2607_17652_amd import binding as fb
from paper_2607_17652_amd import synth
from paper_2607_17652_amd.runner import WavefrontStep

pytestmark = pytest.mark.gpu


def _attend(step, q, K, V, ps, seed, bad=None):
    """Attention over K, V [B, T, Hkv, d] in pages of ps keys, shuffled."""
    B, T, Hkv, d = K.shape
    n = -(-T // ps)
    table = torch.randperm(B * n, generator=torch.Generator().manual_seed(seed)).view(B, n)
    pad = torch.full((B, n * ps - T, Hkv, d), float("nan"), dtype=K.dtype, device="cuda")
    kc = torch.zeros((B * n, Hkv, ps, d), dtype=K.dtype, device="cuda")
    vc = torch.zeros((B * n, Hkv, d, ps), dtype=K.dtype, device="cuda")
    at = table.view(-1).cuda()
    kc[at] = torch.cat([K, pad], 1).view(B * n, ps, Hkv, d).transpose(1, 2)
    vc[at] = torch.cat([V, pad], 1).view(B * n, ps, Hkv, d).permute(0, 2, 3, 1)
    table = table.to(torch.int32).cuda()
    if bad is not None:
        table[bad] = -1
    shape = fb.make_shape(q.shape[1], Hkv, d, "bf16", ps, n, B * n)
    ws = torch.full((fb.fb_attention_workspace_bytes(step.pack, shape),), 0x7F,
                    dtype=torch.uint8, device="cuda")
    out = torch.full_like(q, 7.0)
    step.pack_step()
    fb.fb_wavefront_attention(q, kc, vc, table, step.pack, shape, out, ws)
    torch.cuda.synchronize()
    return out, fb.fb_pack_read_status(step.pack)


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("B,bl,Hq,Hkv", [(5, 8, 8, 2), (3, 96, 4, 4), (20, 16, 8, 1)])
def test_small_pages_equal_whole_tiles(d, B, bl, Hq, Hkv):
    log(f"[pages] d={d} B={B} bl={bl}")
    wl = synth.workload("single", dtype="bf16", B=B, Hq=Hq, Hkv=Hkv, d=d, bl=bl, page_size=32,
                        W_max=4, window=("uniform", 1, 4), prefix=("uniform", 1, 700),
                        n_blocks=8, prefix_jitter=31)
    host = synth.make_host_state(wl, seed=d)
    t = synth.make_device_tensors(wl, host, d, device="cuda", with_logits=False)
    step = WavefrontStep(wl, host, dict(t, logits=None))
    T = int((host["o"] + host["w"] * bl).max())
    gen = torch.Generator(device="cuda").manual_seed(d)
    K, V = (torch.randn((B, T, Hkv, d), generator=gen, device="cuda").bfloat16()
            for _ in range(2))
    for b in range(B):      # past a request's own keys anything may stand
        K[b, int(host["o"][b] + host["w"][b] * bl):] = float("nan")
        V[b, int(host["o"][b] + host["w"][b] * bl):] = float("nan")
    ref, s = _attend(step, t["q"], K, V, 64, seed=1)
    assert s["code"] == 0
    for ps in (8, 16, 32):
        out, s = _attend(step, t["q"], K, V, ps, seed=ps)
        assert s["code"] == 0 and torch.equal(out, ref), ps
    assert torch.isfinite(ref.float()).all()
    last = int(np.argmax(host["o"] + host["w"] * bl))
    for ps in (8, 16):      # a key of request `last`'s own last block has no page
        _, s = _attend(step, t["q"], K, V, ps, seed=ps, bad=(last, (T - 1) // ps))
        assert s["code"] == fb.FB_DERR_PAGE and s["request"] == last
