"""The cases that performance work on this library is measured by: the calls a
user of it makes, through its public entry points, with inputs of the shapes
and distributions of the seeded workloads in ``paper_2607_17652_amd.synth``.

A case is a dict of plain values: ``kind`` names the entry points, the rest the
shapes.  ``prepare`` makes what a program has in hand before the call (device
tensors, packed batch, workspaces), ``run`` is one pass, ``work`` the bytes and
operations it cannot do without, ``tolerance`` what a correct implementation at
the same precision may differ by, and ``exact`` the same outputs in float64 with
plain torch.

Calls that update request state in place begin a pass with one device copy
that puts the state back, so that every pass does the same work.
"""
import math

import numpy as np
import torch

from paper_2607_17652_amd import binding as fb
from paper_2607_17652_amd import synth
from paper_2607_17652_amd.runner import DecodeLoop

_BASE = dict(Hq=32, Hkv=8, d=128, bl=32, page=32, W=4, layout="ragged", dtype="bf16",
             V=157184, n_blocks=64, prefix="uniform", lo=1024, hi=1024, jitter=0,
             w_lo=4, w_hi=4, mask="half")


def _case(kind, B, **kw):
    return dict(_BASE, kind=kind, B=B, **kw)


def listed():
    return [
        # The smallest call of the library: a whole fp32 step of one short
        # request (the correctness workload).  Launches and latency.
        dict(_case("step", 1, Hq=2, Hkv=2, d=32, bl=4, page=4, W=2, dtype="f32", V=1000,
                   n_blocks=4, lo=8, hi=8, w_lo=2, w_hi=2), name="step_tiny"),
        # Interactive decoding: a whole bf16 step of a single request.
        dict(_case("step", 1, Hq=16, Hkv=4, W=3, w_lo=3, w_hi=3), name="step_single"),
        # Serving: a whole step of 256 requests of mixed lengths and windows.
        dict(_case("step", 256, prefix="loguniform", lo=128, hi=8192, w_lo=1, w_hi=4,
                   mask="block_uniform"), name="step_serve256"),
        # Attention of a medium batch in the padded layout (Eq. 4's dense batch).
        dict(_case("attention", 64, Hq=16, Hkv=4, layout="padded", lo=256, hi=4096, w_lo=1,
                   w_hi=4, mask="block_uniform"), name="attn_hetero64"),
        # Attention of a few long-context requests.
        dict(_case("attention", 8, lo=16384, hi=32768), name="attn_long8"),
        # Odd and ragged: blocks of 96, pages of 16 (smaller than a key tile),
        # 64-wide heads without grouping, prefixes that end inside a page.
        dict(_case("attention", 24, Hq=8, Hkv=8, d=64, bl=96, page=16, W=3, n_blocks=21,
                   lo=200, hi=3000, jitter=37, w_lo=1, w_hi=3), name="attn_odd24"),
        # Attention in fp32, as a model run in full precision (or checked
        # against one) calls it.
        dict(_case("attention", 8, Hq=16, Hkv=4, dtype="f32", lo=256, hi=2048, w_lo=1,
                   w_hi=4), name="attn_f32"),
        # The window prologue (RoPE and the KV write) of the serving batch.
        dict(_case("prologue", 256, prefix="loguniform", lo=128, hi=8192, w_lo=1, w_hi=4),
             name="prologue_serve256"),
        # The denoise update of a few requests: full vocabulary, few rows.
        dict(_case("update", 8, lo=16384, hi=32768), name="update_long8"),
        # The LM head with the reduction fused: one request's rows (the weight
        # matrix is read for 96 rows) and the serving batch's.
        dict(_case("lmhead", 1, W=3, w_lo=3, w_hi=3, D=2048), name="lmhead_single"),
        dict(_case("lmhead", 256, prefix="loguniform", lo=128, hi=8192, w_lo=1, w_hi=4,
                   mask="block_uniform", D=2048), name="lmhead_serve256"),
        # A whole decode on the device: 64 requests of 16 blocks, attention leg
        # on, steps replayed from a graph.
        dict(_case("loop", 64, n_blocks=16, lo=256, hi=1024), name="loop64"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges."""
    kind = rng.choice(["attention", "attention", "attention", "attention_f32", "step",
                       "update", "update", "prologue", "lmhead", "lmhead", "loop"])
    heads = rng.choice([(32, 8), (32, 8), (16, 4), (16, 2), (8, 8)])
    d = rng.choice([128, 128, 128, 64, 32])
    bl = rng.choice([32, 32, 32, 8, 16, 64, 96, 128])
    W = rng.choice([1, 2, 3, 4, 4, 5])
    w_lo = rng.randint(1, W)
    page = rng.choice([32, 32, 64, 128, 16, 8])
    layout = rng.choice(["ragged", "ragged", "padded"])
    jitter = rng.choice([0, 0, rng.randint(1, 63)])
    mask = rng.choice(["half", "block_uniform"])
    common = dict(Hq=heads[0], Hkv=heads[1], d=d, bl=bl, page=page, W=W, layout=layout,
                  n_blocks=max(8, 1024 // bl), w_lo=w_lo, w_hi=W, mask=mask, jitter=jitter)
    if kind == "loop":
        return _case("loop", _log_int(rng, 1, 64), bl=rng.choice([8, 16, 32]), W=W, w_lo=1,
                     w_hi=1, n_blocks=rng.randint(2, 12), V=_log_int(rng, 1000, 157184),
                     lo=_log_int(rng, 16, 256), hi=_log_int(rng, 257, 1024),
                     layout=layout, Hq=heads[0], Hkv=heads[1], d=d, page=32)
    B = _log_int(rng, 1, 256)
    if kind == "attention_f32":
        B = _log_int(rng, 1, 12)
        hi = _log_int(rng, 64, 2048)
        return _case("attention", B, **dict(common, dtype="f32", bl=min(bl, 64)),
                     lo=max(1, hi // rng.randint(1, 16)), hi=hi)
    # at most 2^19 prefix positions over the batch, and the serving batch's rows
    hi = _log_int(rng, 64, max(65, min(32768, (1 << 19) // B)))
    lo = max(1, hi // rng.randint(1, 32))
    while B * W * bl > 32768:
        B = max(1, B // 2)
    if kind in ("attention", "prologue"):
        return _case(kind, B, **common, prefix=rng.choice(["uniform", "loguniform"]),
                     lo=lo, hi=hi)
    V = _log_int(rng, 1000, 157184)
    if kind == "lmhead":
        return _case("lmhead", B, **dict(common, n_blocks=8), lo=32, hi=64,
                     V=V, D=64 * rng.randint(4, 32))
    dtype = "f32" if kind == "update" and rng.random() < 0.4 else "bf16"
    while B * W * bl * V * (4 if dtype == "f32" else 2) > 10 << 30:
        B = max(1, B // 2)
    if kind == "update":
        return _case("update", B, **common, dtype=dtype, lo=32, hi=64, V=V)
    return _case("step", B, **common, V=V, lo=lo, hi=hi)


# ----------------------------------------------------------------- inputs ---
def _workload(c):
    return synth.Workload(
        c["kind"], B=c["B"], Hq=c["Hq"], Hkv=c["Hkv"], d=c["d"], bl=c["bl"],
        page_size=c["page"], W_max=c["W"], layout=c["layout"], dtype=c["dtype"], V=c["V"],
        sigma=(1.0, 8.0), planted=0.4, prefix=(c["prefix"], c["lo"], c["hi"]),
        window=("uniform", c["w_lo"], c["w_hi"]), mask=c["mask"], n_blocks=c["n_blocks"],
        prefix_jitter=c["jitter"])


def _capacity(c, host):
    """Token columns and cache pages sized for the longest request the case
    can draw, as a server sizes them (so a case's shapes do not depend on the
    seed); the extra pages belong to no request."""
    longest = max(c["hi"], c["bl"]) + c["jitter"] + c["n_blocks"] * c["bl"]
    pages = -(-longest // c["page"]) + 1
    B, T = host["tokens"].shape
    assert T <= pages * c["page"] and host["max_pages"] <= pages
    tokens = np.full((B, pages * c["page"]), c["V"] - 1, dtype=np.int64)
    tokens[:, :T] = host["tokens"]
    table = np.full((B, pages), -1, dtype=np.int64)
    table[:, :host["max_pages"]] = host["page_table"]
    host.update(tokens=tokens, page_table=table, T_max=pages * c["page"], max_pages=pages)
    return B * pages


def _cache(x, num_pages):
    """The cache x with pages up to num_pages."""
    out = torch.zeros((num_pages,) + x.shape[1:], dtype=x.dtype, device="cuda")
    out[:x.shape[0]] = x
    return out


def _inputs(c, seed):
    """Host state and device tensors (no call of the library)."""
    wl = _workload(c)
    host = synth.make_host_state(wl, seed)
    num_pages = _capacity(c, host)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1_000_003 + 7)
    t = {}
    if c["kind"] in ("step", "attention", "prologue"):
        t = synth.make_device_tensors(wl, host, seed, with_logits=False)
        t["k_cache"] = _cache(t["k_cache"], num_pages)
        t["v_cache"] = _cache(t["v_cache"], num_pages)
        host["num_pages"] = num_pages
    if c["kind"] in ("step", "update"):
        t["logits"] = synth.make_logits(wl, wl.row_cap, gen, "cuda")
    if c["kind"] == "lmhead":
        t["hidden"], t["weight"] = synth.make_lmhead_tensors(wl, c["D"], seed)
    return wl, host, t


class _State:
    """A program's buffers: the request state in one allocation (and a copy of
    it as it was), the packed batch, workspaces and outputs."""

    def __init__(self, c, wl, host, t):
        self.kind, self.wl, self.t = c["kind"], wl, t
        dev = synth.host_to_device_state(host)
        names = ("req_state", "tokens", "pe", "fin")
        at, spans = 0, []
        for n in names:
            nbytes = dev[n].numel() * dev[n].element_size()
            spans.append((n, at, nbytes))
            at += (nbytes + 255) // 256 * 256
        self.flat = torch.zeros(at, dtype=torch.uint8, device="cuda")
        view = {}
        for n, a, nbytes in spans:
            v = self.flat[a:a + nbytes].view(dev[n].dtype).view(dev[n].shape)
            v.copy_(dev[n])
            view[n] = v
        self.st, self.tokens, self.pe, self.fin = (view[n] for n in names)
        self.before = self.flat.clone()
        self.page_table = dev["page_table"]
        self.n_max, self.T_max = host["n_max"], host["T_max"]
        buf = torch.zeros(fb.fb_pack_bytes(wl.B, wl.W_max, wl.bl), dtype=torch.uint8,
                          device="cuda")
        self.pack = fb.fb_pack_init(buf, wl.B, wl.W_max, wl.bl, wl.layout)
        self.params = fb.make_params(wl.tau_mask, wl.tau_edit, wl.theta, wl.mask_id,
                                     wl.eos_id, wl.S_pe, wl.W_max)
        self.pack_batch()
        if "q" in t:
            self.shape = fb.make_shape(wl.Hq, wl.Hkv, wl.d, wl.dtype, wl.page_size,
                                       host["max_pages"], host["num_pages"])
            self.out = torch.zeros_like(t["q"])
        if self.kind in ("step", "attention"):
            nbytes = fb.fb_attention_workspace_bytes(self.pack, self.shape)
            self.attn_ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
            self.write_kv()
        if self.kind in ("step", "update", "lmhead"):
            nbytes = fb.fb_update_workspace_bytes(self.pack, wl.V)
            self.upd_ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
            self.conf = torch.zeros(wl.row_cap, dtype=torch.float32, device="cuda")
            self.argmax = torch.full((wl.row_cap,), -1, dtype=torch.int32, device="cuda")
            self.stats = torch.zeros(wl.B * fb.REQ_STATS_DTYPE.itemsize, dtype=torch.uint8,
                                     device="cuda")
        if self.kind == "lmhead":
            nbytes = fb.fb_lmhead_workspace_bytes(self.pack, wl.V, c["D"])
            self.lm_ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")

    def pack_batch(self):
        fb.fb_pack_wavefronts(self.st, self.tokens, self.n_max, self.T_max, self.pack)

    def write_kv(self):
        t = self.t
        fb.fb_write_window_kv(t["k_new"], t["v_new"], t["k_cache"], t["v_cache"],
                              self.page_table, self.pack, self.shape)

    def attention(self):
        t = self.t
        fb.fb_wavefront_attention(t["q"], t["k_cache"], t["v_cache"], self.page_table,
                                  self.pack, self.shape, self.out, self.attn_ws)

    def updated(self):
        return dict(conf=self.conf, argmax=self.argmax, tokens=self.tokens, st=self.st,
                    pe=self.pe, fin=self.fin, stats=self.stats)


class _LoopState:
    """A decode loop and its request state as it was."""

    def __init__(self, c, seed):
        rng = np.random.default_rng(seed)
        prompts = rng.integers(c["lo"], c["hi"] + 1, size=c["B"])
        host = synth.make_loop_host_state(c["B"], prompts, c["n_blocks"], c["bl"], c["V"],
                                          page_size=c["page"], seed=seed)
        host["num_pages"] = _capacity(c, host)
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed + 17)
        P, dt = host["num_pages"], torch.bfloat16
        kc = (torch.randn((P, c["Hkv"], c["page"], c["d"]), generator=gen, device="cuda")
              * 0.1).to(dt)
        vc = (torch.randn((P, c["Hkv"], c["d"], c["page"]), generator=gen, device="cuda")
              * 0.1).to(dt)
        prm = dict(tau_mask=0.9, tau_edit=0.8, theta=0.5, mask_id=c["V"] - 1, eos_id=-1,
                   S_pe=2, W=c["W"], edit_masked=False, force_progress=False,
                   sync_window=False)
        attn = dict(Hq=c["Hq"], Hkv=c["Hkv"], d=c["d"], dtype="bf16", page_size=c["page"],
                    k_cache=kc, v_cache=vc, embed_seed=seed + 5)
        self.loop = DecodeLoop(host, c["bl"], c["W"], c["V"], prm, seed + 99,
                               synth.loop_levels(c["V"]), layout=c["layout"], attn=attn)
        lp = self.loop
        self.live = (lp.st, lp.tokens, lp.pe, lp.fin, lp.counters, lp.forwards)
        self.before = [x.clone() for x in self.live]
        self.stream = torch.cuda.Stream()


def prepare(case, seed):
    if case["kind"] == "loop":
        return _LoopState(case, seed)
    return _State(case, *_inputs(case, seed))


# ------------------------------------------------------------------- pass ---
def run(s):
    if isinstance(s, _LoopState):
        for x, b in zip(s.live, s.before):
            x.copy_(b)
        lp = s.loop
        lp.run(max_steps=4096, check_every=16, use_graph=True, stream=s.stream)
        return dict(logits=lp.logits, attn=lp.out, k_cache=lp.k_cache, v_cache=lp.v_cache,
                    conf=lp.conf, argmax=lp.argmax, tokens=lp.tokens, st=lp.st, pe=lp.pe,
                    fin=lp.fin, counters=lp.counters, forwards=lp.forwards)
    t = s.t
    if s.kind == "attention":
        s.attention()
        return dict(attn=s.out)
    if s.kind == "prologue":
        fb.fb_window_prologue(t["q"], s.out, t["k_new"], t["v_new"], t["k_cache"],
                              t["v_cache"], s.page_table, s.pack, s.shape)
        return dict(q=s.out, k_cache=t["k_cache"], v_cache=t["v_cache"])
    s.flat.copy_(s.before)
    if s.kind == "lmhead":
        fb.fb_lmhead_reduce(t["hidden"], t["weight"], s.pack, s.lm_ws, s.upd_ws)
        fb.fb_denoise_apply(s.wl.V, s.tokens, s.conf, s.argmax, s.st, s.pe, s.fin, s.pack,
                            s.params, s.stats, s.upd_ws)
        return s.updated()
    if s.kind == "step":
        s.pack_batch()
        s.write_kv()
        s.attention()
    fb.fb_denoise_update(t["logits"], s.tokens, s.conf, s.argmax, s.st, s.pe, s.fin, s.pack,
                         s.params, s.stats, s.upd_ws)
    if s.kind == "step":
        return dict(s.updated(), attn=s.out, k_cache=t["k_cache"], v_cache=t["v_cache"])
    return s.updated()


# ------------------------------------------------------------------- work ---
# Mean forwards a block of the synthetic loop takes part in between admission
# and retirement (counted over decodes of the listed case).
_LOOP_FORWARDS = 6.4


def work(case):
    """Bytes and operations of one pass, expected over the seeded draws."""
    c, elt = case, 2 if case["dtype"] == "bf16" else 4
    w1 = (c["w_lo"] + c["w_hi"]) / 2.0
    w2 = sum(w * (w + 1) / 2.0 for w in range(c["w_lo"], c["w_hi"] + 1)) / \
        (c["w_hi"] - c["w_lo"] + 1)
    o = (c["lo"] + c["hi"]) / 2.0
    if c["prefix"] == "loguniform" and c["hi"] > c["lo"]:
        o = (c["hi"] - c["lo"]) / math.log(c["hi"] / c["lo"])
    o = max(o + c["jitter"] / 2.0, c["bl"])
    rows = c["B"] * w1 * c["bl"]
    kv_row = 2.0 * c["Hkv"] * c["d"] * elt          # K and V of one position
    qo_row = 2.0 * c["Hq"] * c["d"] * elt           # Q in, O out of one row
    attn_flops = 4.0 * c["bl"] * c["Hq"] * c["d"] * c["B"] * (w1 * o + c["bl"] * w2)
    attn_bytes = c["B"] * (o + w1 * c["bl"]) * kv_row + rows * qo_row
    logit_bytes = rows * c["V"] * elt
    # max, exponential and sum of each logit
    upd = dict(bytes=logit_bytes + rows * 16, flops=3.0 * rows * c["V"])
    if c["kind"] == "attention":
        return dict(bytes=attn_bytes, flops=attn_flops)
    if c["kind"] == "prologue":
        return dict(bytes=rows * (qo_row + 2 * kv_row),
                    flops=3.0 * rows * (c["Hq"] + c["Hkv"]) * c["d"])
    if c["kind"] == "update":
        return upd
    if c["kind"] == "lmhead":
        return dict(bytes=2.0 * c["D"] * (c["V"] + rows) + rows * 16,
                    flops=2.0 * rows * c["V"] * c["D"])
    if c["kind"] == "step":
        return dict(bytes=attn_bytes + rows * 2 * kv_row + upd["bytes"],
                    flops=attn_flops + upd["flops"])
    blocks = c["B"] * c["n_blocks"]
    f = _LOOP_FORWARDS * blocks * c["bl"]           # row forwards of the whole decode
    mean_kv = o + c["n_blocks"] * c["bl"] / 2.0
    return dict(bytes=f * (2.0 * c["V"] * elt + 2 * qo_row + 4 * kv_row),
                flops=f * (4.0 * c["Hq"] * c["d"] * mean_kv + 3.0 * c["V"]))


# -------------------------------------------------------------- tolerance ---
# About four times the error measured against float64.
def tolerance(case):
    if case["kind"] in ("step", "attention", "loop") and case["dtype"] == "bf16":
        # outputs and softmax weights rounded to bf16
        return {"rel": 8e-3, "max": 0.05}
    if case["kind"] == "prologue":
        # rotated in float32 and rounded to bf16: one rounding may go the other way
        return {"rel": 1e-3, "max": 1e-2}
    if case["kind"] == "lmhead":
        # float32 sums of D products in another order move a logit by about
        # 1e-5 and so a confidence; a near tie may go the other way
        return {"rel": 1e-5, "max": 1e-4, "differ": 2e-3}
    # float32 sums
    return {"rel": 4e-6, "max": 4e-5}


# ------------------------------------------------------------------ exact ---
def _row0(wl, host):
    if wl.layout == "padded":
        return np.arange(wl.B) * wl.W_max * wl.bl
    n = host["w"] * wl.bl
    return np.cumsum(n) - n


def _live(wl, host):
    r0 = _row0(wl, host)
    rows = [np.arange(r0[b], r0[b] + host["w"][b] * wl.bl) for b in range(wl.B)]
    return torch.from_numpy(np.concatenate(rows)).cuda()


def _exact_attention(wl, host, t):
    out = torch.zeros(t["q"].shape, dtype=torch.float64, device="cuda")
    r0, g = _row0(wl, host), wl.Hq // wl.Hkv
    for b in range(wl.B):
        o, w = int(host["o"][b]), int(host["w"][b])
        T, n = o + w * wl.bl, w * wl.bl
        rows = slice(int(r0[b]), int(r0[b]) + n)
        pos = torch.arange(T, device="cuda")
        page = torch.from_numpy(host["page_table"][b]).cuda()[pos // wl.page_size]
        K = t["k_cache"][page, :, pos % wl.page_size, :].double()     # [T, Hkv, d]
        V = t["v_cache"][page, :, :, pos % wl.page_size].double()
        K[o:] = t["k_new"][rows].double()
        V[o:] = t["v_new"][rows].double()
        q = t["q"][rows].double()                                     # [n, Hq, d]
        row_pos = torch.arange(n, device="cuda") // wl.bl
        seen = pos[None, :] < (o + (row_pos + 1) * wl.bl)[:, None]    # [n, T]
        for h in range(wl.Hkv):
            k, v = K[:, h].contiguous(), V[:, h].contiguous()
            for j in range(h * g, h * g + g):
                s = q[:, j].contiguous() @ k.t().contiguous() / math.sqrt(wl.d)
                s = s.masked_fill(~seen, float("-inf")).softmax(dim=1)
                out[rows, j] = s @ v
    return out


def _conf_of(z):
    m = z.max(dim=1, keepdim=True).values
    return 1.0 / (z - m).exp().sum(dim=1)


def _exact_conf(wl, host, t):
    conf = torch.zeros(wl.row_cap, dtype=torch.float64, device="cuda")
    live = _live(wl, host)
    for i in range(0, len(live), 512):
        r = live[i:i + 512]
        if "logits" in t:
            conf[r] = _conf_of(t["logits"][r].double())
            continue
        z = [t["hidden"][r].double() @ t["weight"][v:v + 32768].double().t()
             for v in range(0, wl.V, 32768)]
        conf[r] = _conf_of(torch.cat(z, dim=1))
    return conf


def _exact_prologue(wl, host, t, base=10000.0):
    half, r0 = wl.d // 2, _row0(wl, host)
    theta = base ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / wl.d)

    def turn(x, pos):
        a = pos.double()[:, None, None] * theta
        lo, hi = x[..., :half].double(), x[..., half:].double()
        return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], dim=-1)

    q = torch.zeros(t["q"].shape, dtype=torch.float64, device="cuda")
    kc = t["k_cache"].double()
    for b in range(wl.B):
        n, o = int(host["w"][b]) * wl.bl, int(host["o"][b])
        rows = slice(int(r0[b]), int(r0[b]) + n)
        pos = torch.arange(o, o + n, device="cuda")
        page = torch.from_numpy(host["page_table"][b]).cuda()[pos // wl.page_size]
        q[rows] = turn(t["q"][rows], pos)
        kc[page, :, pos % wl.page_size, :] = turn(t["k_new"][rows], pos)
    return q, kc


def exact(case, seed):
    if case["kind"] == "loop":
        return None
    wl, host, t = _inputs(case, seed)
    if case["kind"] == "prologue":
        q, kc = _exact_prologue(wl, host, t)
        return dict(q=q, k_cache=kc, v_cache=None)
    if case["kind"] == "attention":
        return dict(attn=_exact_attention(wl, host, t))
    upd = dict(conf=_exact_conf(wl, host, t), argmax=None, tokens=None, st=None, pe=None,
               fin=None, stats=None)
    if case["kind"] == "step":
        return dict(upd, attn=_exact_attention(wl, host, t), k_cache=None, v_cache=None)
    return upd
