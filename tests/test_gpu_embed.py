"""The synthetic embeddings' vector and single-element stores, bit for bit
against the oracle: whole 16-byte runs per thread where every buffer is
16-byte aligned and the row long enough (bf16: from 256 elements on), one
element per store otherwise."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from oracle import pack as opack  # noqa: E402
from oracle import synth_model as osm  # noqa: E402
from paper_2607_17652_amd import binding as fb  # noqa: E402
from paper_2607_17652_amd import synth  # noqa: E402
from paper_2607_17652_amd.runner import WavefrontStep  # noqa: E402


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Hq,Hkv,d", [(2, 1, 32), (5, 1, 32), (4, 2, 32), (8, 8, 64), (32, 8, 128)])
@pytest.mark.parametrize("shifted", [None, "q", "v"])
def test_embed_rows(dtype, Hq, Hkv, d, shifted):
    wl = synth.workload("single", dtype=dtype, B=3, Hq=Hq, Hkv=Hkv, d=d, bl=8,
                        window=("uniform", 1, 3))
    host = synth.make_host_state(wl, seed=4)
    t = synth.make_device_tensors(wl, host, 4, device="cuda", with_logits=False)
    step = WavefrontStep(wl, host, dict(t, logits=None))
    step.pack_step()

    def buffer(x, name):
        off = 1 if name == shifted else 0      # one element: not 16-byte aligned
        flat = torch.full((x.numel() + off,), 7.0, dtype=x.dtype, device="cuda")
        return flat[off:].view(x.shape)
    q, kn, vn = buffer(t["q"], "q"), buffer(t["k_new"], "k"), buffer(t["v_new"], "v")
    seed = 0x9E3779B97F4A7C15
    fb.fb_synth_embed(step.pack, step.shape, seed, q, kn, vn)
    torch.cuda.synchronize()
    packed = opack.pack_wavefronts(host["state"], wl.W_max, wl.bl, wl.layout)
    live = packed["row_req"] >= 0
    pos = packed["row_pos"][live]
    tok = [int(host["tokens"][packed["row_req"][r], packed["row_pos"][r]])
           for r in np.flatnonzero(live)]
    for kind, (T, H) in enumerate([(q, Hq), (kn, Hkv), (vn, Hkv)]):
        got = T.double().cpu().numpy()
        assert np.array_equal(got[:len(live)][live], osm.embed_rows(seed, kind, pos, tok, H, d))
        dead = np.ones(len(got), dtype=bool)
        dead[:len(live)] = ~live
        assert np.all(got[dead] == 7.0), kind      # rows that are not live stay unwritten
