"""The LM head's weight-streaming form (at most 128 rows): both token widths
and the first row count past it, vocabularies with a partial last 32-id group,
fewer groups than CUs and ranges of one group up, one and several K stages,
against the oracle as the general form's tests are."""
import numpy as np
import pytest
import torch

from harness import log
from paper_2607_17652_amd import binding as fb
from paper_2607_17652_amd import synth
from paper_2607_17652_amd.runner import WavefrontStep
from test_gpu_lmhead import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,D,kw", [
    (33, 64, dict(bl=1, page_size=8, W_max=1, window=("fixed", 1))),    # 1 row, 2 groups, 1 stage
    (5003, 128, dict(bl=32, W_max=1, window=("fixed", 1))),             # 32 rows
    (8193, 192, dict(bl=32, W_max=2, window=("fixed", 2))),             # 64: the narrow form's last
    (70001, 192, dict(bl=13, W_max=5, window=("fixed", 5))),            # 65: the wide form's first
    (157184, 1024, dict(bl=32, W_max=4, window=("fixed", 4))),          # 128: the form's last
    (40000, 256, dict(bl=43, W_max=3, window=("fixed", 3))),            # 129: past it
    (65537, 2048, dict(B=4, bl=32, W_max=4, window=("fixed", 1))),      # 128 live of 512
    (65537, 2048, dict(B=4, bl=16, W_max=4, window=("fixed", 1))),      # 64 live of 256
    (65537, 2048, dict(B=5, bl=32, W_max=4, window=("fixed", 1))),      # 160: past the form
    # 64 live of 256 padded rows: past the form
    (65537, 2048, dict(B=2, bl=32, W_max=4, window=("fixed", 1), layout="padded")),
    (9001, 256, dict(B=4, bl=8, W_max=4, window=("uniform", 1, 4), layout="padded")),
])
def test_lmhead_few_rows(V, D, kw):
    run_case("single", V, D, seed=7, prefix=("fixed", 64), **kw)


@pytest.mark.parametrize("tied", [[5, 9, 37, 300, 5000], [4999, 5000, 157000]])
def test_lmhead_few_rows_ties_take_the_lowest_id(tied):
    """Exact ties across lane halves, groups, waves and ranges."""
    def edit(hid, weight):
        hid[:, 0] = 1.0
        weight[tied] = 0
        weight[tied, 0] = 256.0
    wl, host, packed, g, rows, o, tie, tok0 = run_case("single", 157184, 256, seed=6, edit=edit)
    assert (g["argmax"][rows] == min(tied)).all()


def test_lmhead_few_rows_of_no_live_request():
    """A pack that may take the form and holds no live row: nothing is written."""
    wl = synth.workload("single", V=65537, B=4, W_max=4, bl=32, prefix=("fixed", 64))
    host = synth.make_host_state(wl, seed=7)
    host["state"]["active"][:] = 0
    log("[lmhead] no live request")
    t = synth.make_device_tensors(wl, host, 7, device="cuda", with_logits=False)
    step = WavefrontStep(wl, host, dict(t, logits=None))
    hid, weight = synth.make_lmhead_tensors(wl, 2048, 7)
    lm_ws = torch.empty(fb.fb_lmhead_workspace_bytes(step.pack, wl.V, 2048), dtype=torch.uint8,
                        device="cuda")
    before = [x.clone() for x in (step.conf, step.argmax, step.tokens, step.st)]
    step.pack_step()
    fb.fb_lmhead_reduce(hid, weight, step.pack, lm_ws, step.upd_ws)
    fb.fb_denoise_apply(wl.V, step.tokens, step.conf, step.argmax, step.st, step.pe, step.fin,
                        step.pack, step.params, step.stats, step.upd_ws)
    torch.cuda.synchronize()
    assert fb.fb_pack_read_status(step.pack)["n_rows"] == 0
    for x, b in zip((step.conf, step.argmax, step.tokens, step.st), before):
        assert torch.equal(x, b)


def test_lmhead_forms_agree_on_the_same_rows():
    """One request's 96 rows alone (the few-rows form) and among seven others
    (the tile form): the logits' float32 sums differ in their order, so argmax
    is the same wherever the top two are further apart than both forms' bounds,
    and conf within them."""
    V, D, kept = 65537, 2048, []

    def keep(hid, weight):
        kept.extend([hid.clone(), weight.clone()])

    def same(hid, weight):
        hid[:96] = kept[0][:96]
        weight.copy_(kept[1])
    kw = dict(W_max=3, bl=32, window=("fixed", 3), prefix=("fixed", 64))
    _, _, _, few, rows, o, tie, _ = run_case("single", V, D, seed=7, edit=keep, **kw)
    _, _, _, tiles, _, _, _, _ = run_case("single", V, D, seed=8, sample=32, edit=same, B=8, **kw)
    assert np.array_equal(rows, np.arange(96))
    assert np.array_equal(few["argmax"][rows][~tie], tiles["argmax"][rows][~tie])
    tol = 2 * o["p"] * (np.expm1(2 * o["bound"]) + 2e-5)
    assert np.all(np.abs(few["conf"][rows].astype(np.float64) - tiles["conf"][rows]) <= tol)
