"""The fp32 attention's MFMA kernel at the sizes where it can go wrong: every
head size, pages of one key (V key by key) to whole tiles and more, partial
key and row tiles, whole and split units, and a block with a bad page."""
import numpy as np
import pytest
import torch

from harness import ATTN_TOL, OracleCase, compare_case, gather_kv, gpu_results, log, setup
from paper_2607_17652_amd import binding as fb

pytestmark = pytest.mark.gpu


def f32(seed=0, **kw):
    base = dict(dtype="f32", V=256, B=3, n_blocks=8, prefix=("uniform", 20, 400),
                window=("uniform", 1, 3), prefix_jitter=13)
    base.update(kw)
    return setup("single", seed, **base)


def past_windows(host, wl, page_table, value, *caches):
    """Every cache slot past a request's window (keys no query sees) := value."""
    for b in range(wl.B):
        end = int(host["o"][b] + host["w"][b] * wl.bl)
        top = int(host["state"]["gen_start"][b]) + wl.n_blocks * wl.bl
        pos = torch.arange(end, top, device="cuda")
        page, slot = page_table[b][pos // wl.page_size].long(), pos % wl.page_size
        caches[0][page, :, slot, :] = value
        caches[1][page, :, :, slot] = value


@pytest.mark.parametrize("kw", [
    dict(d=32, Hq=3, Hkv=3, bl=5, page_size=1),            # pages of one key, 5 rows of 32
    dict(d=64, Hq=4, Hkv=2, bl=8, page_size=2),            # pages of two keys
    dict(d=128, page_size=4),                              # one V chunk per page
    dict(d=32, Hq=4, Hkv=2, bl=4, page_size=32, prefix=("fixed", 8), n_blocks=4),  # no split
    dict(d=64, Hq=8, Hkv=8, bl=33, page_size=64),          # 33 rows: a second wave with one
    dict(d=128, Hq=8, Hkv=1, bl=17, page_size=16, W_max=4, window=("fixed", 4)),   # 136 rows
    dict(d=128, prefix=("uniform", 1500, 1600), kv_split=32, B=1),   # one key tile per piece
    dict(d=32, Hq=4, Hkv=4, prefix=("uniform", 3000, 4000), B=2),
    dict(d=64, Hq=4, Hkv=2, bl=8, page_size=2, prefix=("uniform", 900, 1000)),   # split, V by key
])
def test_f32_attention(kw):
    kw = dict(kw)
    split = kw.pop("kv_split", 0)
    wl, host, t, step = f32(kv_split=split, **kw)
    log(f"[f32 attention] {kw} kv_split={split}")
    case = OracleCase(wl, host, t, list(range(wl.B)), step.page_table)
    step.run()
    torch.cuda.synchronize()
    first = step.out.clone()
    case.run(wl.params())
    compare_case(wl, case, gpu_results(step), step)
    # keys past the windows are never used, whatever they hold (the update
    # moved the windows on, but the pack still describes this step)
    past_windows(host, wl, step.page_table, float("nan"), t["k_cache"], t["v_cache"])
    step.out.zero_()
    step.attention_step()
    torch.cuda.synchronize()
    assert torch.equal(step.out, first)


@pytest.mark.parametrize("prefix", [("fixed", 32), ("uniform", 1500, 2000)])
def test_f32_bad_page_skips_the_blocks_that_read_it(prefix):
    """A block with an invalid page leaves its rows as they were and is
    reported, split or not; the others are computed."""
    def edit(wl, host):
        host["page_table"][1, 0] = host["num_pages"] + 7
    wl, host, t, step = f32(prefix=prefix, prefix_jitter=0, page_size=32, n_blocks=4,
                            host_edit=edit)
    log(f"[f32 attention] bad page in request 1, prefix={prefix}")
    step.pack_step()
    step.kv_step()
    step.out.fill_(7.0)
    step.attention_step()
    torch.cuda.synchronize()
    s = fb.fb_pack_read_status(step.pack)
    assert s["code"] == fb.FB_DERR_PAGE and s["request"] == 1
    req = step.pack.view()["row_req"]
    assert bool((step.out[req == 1] == 7.0).all())
    assert bool((step.out[(req == 0) | (req == 2)] != 7.0).any(dim=-1).all())


def attend(step):
    step.pack_step()
    step.kv_step()
    step.out.fill_(7.0)
    step.attention_step()
    torch.cuda.synchronize()
    assert fb.fb_pack_read_status(step.pack)["code"] == 0
    return step.out.clone()


# one workgroup per unit without a plan, planned whole units, units in pieces
FORMS = [dict(d=32, prefix=("uniform", 20, 100)), dict(prefix=("uniform", 600, 900), kv_split=2048),
         dict(prefix=("uniform", 600, 900), kv_split=64)]


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("kw", FORMS)
def test_f32_nan_query_rows_come_out_as_nan(kw, value):
    """A live row whose scores are all NaN is written as NaN, in whichever
    form; the others are as without it (up to the moment at which a wave
    rescales its rows: a few 2^-24)."""
    wl, host, t, step = f32(n_blocks=4, page_size=32, **kw)
    log(f"[f32 attention] {value} in a query, {kw}")
    ref = attend(step)
    row = int(torch.nonzero(step.pack.view()["row_req"] == 1).flatten()[2])
    t["q"][row, 1, 5] = value
    out = attend(step)
    assert bool(torch.isnan(out[row, 1]).all())
    out[row, 1] = ref[row, 1]
    assert torch.allclose(out, ref, rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("value", [float("-inf"), float(np.finfo(np.float32).min)])
@pytest.mark.parametrize("masked", [range(0, 32), range(64, 192), range(0, 160)])
@pytest.mark.parametrize("kw", [dict(d=32, prefix=("fixed", 224)),
                                dict(d=64, prefix=("fixed", 640), kv_split=2048),
                                dict(d=64, prefix=("fixed", 640), kv_split=64)])
def test_f32_masked_keys(kw, masked, value):
    """Keys put out of sight by a score of -inf or of the lowest float (one
    head element is the mask's: 1 in the queries, the value in masked keys),
    at a scale that takes the lowest float past the range: whole key tiles and
    pieces weigh nothing, wherever they lie."""
    wl, host, t, step = f32(B=2, n_blocks=4, page_size=32, prefix_jitter=0, **kw)
    log(f"[f32 attention] keys {masked} at {value}, {kw}")
    step.shape.sm_scale = 1.0
    t["q"][..., 0] = 1.0
    t["k_new"][..., 0] = 0.0
    t["k_cache"][..., 0] = 0.0
    pos = torch.tensor(list(masked), device="cuda")
    for b in range(wl.B):
        page = step.page_table[b][pos // wl.page_size].long()
        t["k_cache"][page, :, pos % wl.page_size, 0] = value
    out = attend(step)
    view = step.pack.view()
    row_req, row_pos = view["row_req"].tolist(), view["row_pos"].tolist()
    got, q = out.double().cpu().numpy(), t["q"].double().cpu().numpy()
    for b in range(wl.B):
        o = int(host["o"][b])
        K, V = gather_kv(t["k_cache"], t["v_cache"], step.page_table[b],
                         o + int(host["w"][b]) * wl.bl, wl.page_size)
        for r in (r for r in range(wl.row_cap) if row_req[r] == b):
            seen = np.setdiff1d(np.arange(o + ((row_pos[r] - o) // wl.bl + 1) * wl.bl), masked)
            for h in range(wl.Hq):
                kh = h // (wl.Hq // wl.Hkv)
                z = K[seen, kh] @ q[r, h]
                p = np.exp(z - z.max())
                ref = (p / p.sum()) @ V[seen, kh]
                err = np.abs(got[r, h] - ref).max()
                assert err <= ATTN_TOL["f32"], (b, r, h, err)
