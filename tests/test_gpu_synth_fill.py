"""The synthetic logits' stores at every row alignment: whole 16-byte runs in a
row's aligned body, single elements around it, nothing outside live rows."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from oracle import pack as opack  # noqa: E402
from paper_2607_17652_amd import binding as fb  # noqa: E402
from paper_2607_17652_amd import synth  # noqa: E402
from paper_2607_17652_amd.runner import WavefrontStep  # noqa: E402


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
# rows shorter than a 16-byte run, one run and two, whole in fp32 alone, a
# remainder at both ends of one split and of the first and last of several,
# whole rows of one split and of several
@pytest.mark.parametrize("V", [5, 9, 16, 1003, 1004, 32768, 32769, 65543, 65600])
def test_fill_rows(dtype, V):
    wl = synth.workload("single", V=V, B=3, Hq=2, Hkv=1, d=32, bl=8,
                        window=("uniform", 1, 3), W_max=3, layout="padded")
    host = synth.make_host_state(wl, seed=6)
    t = synth.make_device_tensors(wl, host, 6, device="cuda", with_logits=False)
    step = WavefrontStep(wl, host, dict(t, logits=None))
    step.pack_step()
    levels = synth.loop_levels(V)
    cap = wl.row_cap
    ldt = torch.bfloat16 if dtype == "bf16" else torch.float32
    flat = torch.full((cap * V + 1,), -7.0, dtype=ldt, device="cuda")
    logits = flat[:cap * V].view(cap, V)
    pred = torch.full((cap, 2), -1, dtype=torch.int32, device="cuda")
    print(f"[fill] {dtype} V={V}", flush=True)
    fb.fb_synth_logits(step.st, step.tokens, step.pack, fb.make_model(77, levels), pred, logits)
    torch.cuda.synchronize()
    live = opack.pack_wavefronts(host["state"], wl.W_max, wl.bl, wl.layout)["row_req"] >= 0
    p = pred.cpu().numpy()
    exp = np.full((cap, V), -7.0, dtype=np.float32)
    for r in np.flatnonzero(live):
        exp[r] = 0.0
        exp[r, p[r, 0]] = levels[p[r, 1]]
    assert 0 < live.sum()
    assert np.array_equal(logits.float().cpu().numpy(), exp)
    assert flat[-1] == -7.0
