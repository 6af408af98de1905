"""The workloads that the performance of this framework is followed on, through its public entry points.

A case is one call, or one denoising step's calls, as a user's program makes them:

  step   d3tom_merge_layer (or the separate importance / selection / merge calls, with the decider update in front) and the
         attention over the shortened sequence: what the merge layer of a model does in one denoising step
  kv     d3tom_merge_kv on a key/value cache
  attend d3tom_attend / d3tom_attend_weighted alone: every layer in front of and behind the merge layer
  stack  d3tom_stack_step_batch: whole blocks (normalisation, projections, attention, feed-forward part), with the merge
         layer inside the first block, or unmerged (the first step of a trajectory, when nothing has been decided yet)

Inputs are drawn on the GPU from the seed.  Visual rows are near-duplicates (cluster centres plus noise), a fraction of
the visual tokens draws the deciders' attention.  Three things are chosen so that the outputs of two correct programs
can be compared: the salient fraction is the kept fraction (which tokens are kept then follows from the data, not from
the rounding of near-equal scores), there are several kept tokens per cluster (a near-tie of two cosines then exchanges two rows that
are alike), and the stack merges in its first block (behind it the rounding of two blocks decides such ties).
"""
import math
import random

import torch

from paper_2511_12280_amd import binding as B


# ---- cases -------------------------------------------------------------------------------------------------------------
def _step(**kw):
    c = dict(kind="step", dtype="bf16", calls="layer", B=1, P=64, O=64, H=32, dh=128, sizes=0)
    c.update(kw)
    return c


def _stack(**kw):
    c = dict(kind="stack", dtype="bf16", B=1, P=64, O=64, H=32, dh=128, F=11008, L=4, sizes=0)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest single layer, float32: 32 prompt + 144 visual + 32 response tokens, hidden 256 (launch latency and host work)
        _step(name="tiny_f32", dtype="f32", P=32, V_lo=144, V_hi=144, O=32, D_lo=16, D_hi=16, keep_lo=0.25, keep_hi=0.25, H=4, dh=64),
        # one image crop through the separate entry points (a caller with a host decision between the stages), a narrow model
        # with heads of 64, odd sizes, the decider set built on the device first
        _step(name="one_crop_729_calls", calls="separate", P=37, V_lo=729, V_hi=729, O=51, D_lo=13, D_hi=13, keep_lo=1 / 3, keep_hi=1 / 3,
              H=16, dh=64),
        # the single-image step: 1024 visual tokens, 103 kept
        _step(name="image_1024", V_lo=1024, V_hi=1024, D_lo=32, D_hi=32, keep_lo=0.10, keep_hi=0.10),
        # the multi-crop sweep's two ends: few deciders and few kept tokens, many deciders and half of the tokens kept
        _step(name="crops_3645_first", V_lo=3645, V_hi=3645, D_lo=2, D_hi=2, keep_lo=0.10, keep_hi=0.10),
        _step(name="crops_3645_last", V_lo=3645, V_hi=3645, D_lo=64, D_hi=64, keep_lo=0.50, keep_hi=0.50),
        # batched serving: 16 samples of 2304 visual tokens, decider counts and keep ratios of their own
        _step(name="serving_b16", B=16, P=128, V_lo=2304, V_hi=2304, O=256, D_lo=8, D_hi=256, keep_lo=0.1, keep_hi=0.5),
        # key/value cache of prompt and visual rows shortened to a quarter of the visual ones
        dict(name="kv_cache_3709", kind="kv", dtype="bf16", B=1, P=64, V_lo=3645, V_hi=3645, keep_lo=0.25, keep_hi=0.25, d=4096, sizes=0),
        # attention of a layer in front of the merge (full length), and a ragged batch of merged samples with member counts as weights
        dict(name="attend_3773", kind="attend", dtype="bf16", B=1, n_lo=3773, n_hi=3773, H=32, dh=128, weighted=False, sizes=0),
        dict(name="attend_weighted_b4", kind="attend", dtype="bf16", B=4, n_lo=493, n_hi=1951, H=32, dh=128, weighted=True, sizes=0),
        # blocks of the full-width stack: a trajectory's first step (unmerged), a merged step, a ragged batch of merged samples.
        # All blocks are the same work: four of them (1.6 GB of weights, far above every cache) stand for a model's 32.
        _stack(name="stack_first_step", V_lo=3645, V_hi=3645, D_lo=0, D_hi=0, keep_lo=0.10, keep_hi=0.10),
        _stack(name="stack_merged_step", V_lo=3645, V_hi=3645, D_lo=1, D_hi=1, keep_lo=0.10, keep_hi=0.10),
        _stack(name="stack_merged_b6", B=6, V_lo=700, V_hi=1300, D_lo=1, D_hi=4, keep_lo=0.10, keep_hi=0.40),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step_f32", "kv", "attend", "attend", "stack"])
    sizes = rng.randrange(1, 1 << 20)
    batch = rng.choice([1, 1, 1, _log_int(rng, 2, 16)])
    if kind == "step":
        hi = _log_int(rng, 96, 3645 if batch == 1 else 2304)
        H, dh = rng.choice([(32, 128), (32, 128), (16, 64), (8, 128)])
        O = _log_int(rng, 16, 256)
        D = rng.randint(1, O)
        r = rng.uniform(0.1, 0.5)
        return _step(calls=rng.choice(["layer", "layer", "separate"]), B=batch, P=_log_int(rng, 8, 128), V_lo=hi if batch == 1 else (hi + 1) // 2,
                     V_hi=hi, O=O, D_lo=D if batch == 1 else max(1, D // 4), D_hi=D, keep_lo=r if batch == 1 else 0.1, keep_hi=r, H=H, dh=dh,
                     sizes=sizes)
    if kind == "step_f32":
        V = _log_int(rng, 48, 576)
        r = rng.uniform(0.1, 0.5)
        D = rng.randint(1, 32)
        return _step(dtype="f32", P=_log_int(rng, 8, 64), V_lo=V, V_hi=V, O=32, D_lo=D, D_hi=D, keep_lo=r, keep_hi=r, H=4, dh=64, sizes=sizes)
    if kind == "kv":
        batch = min(batch, 8)
        V = _log_int(rng, 256, 3645)
        r = rng.uniform(0.1, 0.5)
        return dict(kind="kv", dtype="bf16", B=batch, P=_log_int(rng, 8, 128), V_lo=V if batch == 1 else (V + 1) // 2, V_hi=V, keep_lo=r,
                    keep_hi=r, d=rng.choice([4096, 4096, 1024]), sizes=sizes)
    if kind == "attend":
        weighted = rng.random() < 0.3
        n = _log_int(rng, 128, 3584 if weighted else 3773)
        H, dh = rng.choice([(32, 128), (32, 128), (16, 64), (8, 128)])
        return dict(kind="attend", dtype="bf16", B=batch, n_lo=n if batch == 1 else (n + 2) // 3, n_hi=n, H=H, dh=dh, weighted=weighted, sizes=sizes)
    batch = min(batch, 4)
    V = _log_int(rng, 200, 3645 if batch == 1 else 900)
    r = rng.uniform(0.1, 0.5)
    D = rng.choice([0, 1, rng.randint(1, 8)])
    H, F = rng.choice([(32, 11008), (16, 5632)])
    return _stack(B=batch, P=_log_int(rng, 8, 128), V_lo=V if batch == 1 else (V + 1) // 2, V_hi=V, O=rng.randint(16, 96), D_lo=D, D_hi=D,
                  keep_lo=r, keep_hi=r, H=H, F=F, L=rng.randint(2, 4), sizes=sizes)


# ---- sizes of a case's samples (part of the case, not of the seed) -------------------------------------------------------
def _samples(c):
    rng = random.Random(c["sizes"])
    out = []
    for _ in range(c["B"]):
        V = rng.randint(c["V_lo"], c["V_hi"])
        D = rng.randint(c.get("D_lo", 0), c.get("D_hi", 0))
        r = rng.uniform(c["keep_lo"], c["keep_hi"])
        k = max(1, min(V, math.ceil(r * V - 1e-9)))
        N = c["P"] + V + c.get("O", 0)
        out.append(dict(V=V, D=D, ratio=r, k=k, N=N, Nm=N - (V - k)))
    return out


def _lengths(c):
    rng = random.Random(c["sizes"])
    n = [rng.randint(c["n_lo"], c["n_hi"]) for _ in range(c["B"])]
    n[0] = c["n_hi"]
    return n


# ---- inputs ----------------------------------------------------------------------------------------------------------------
class _Draw:
    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)
        self.dt = torch.float32 if dtype == "f32" else torch.bfloat16

    def normal(self, *shape, std=1.0):
        t = torch.empty(shape, dtype=self.dt, device="cuda").normal_(generator=self.g)
        return t if std == 1.0 else t.mul_(std)

    def ints(self, hi, n):
        return torch.randint(0, hi, (n,), generator=self.g, device="cuda")

    def subset(self, V, k):
        """k of V positions, ascending"""
        return torch.sort(torch.randperm(V, generator=self.g, device="cuda")[:k])[0]

    def visual(self, V, d, kept):
        """V rows around fewer centres than tokens are kept, noise 0.3"""
        n = max(2, kept // 3)
        return self.normal(n, d)[self.ints(n, V)] + self.normal(V, d, std=0.3)


def _i32(a):
    return torch.tensor(a, dtype=torch.int32, device="cuda")


def _offsets(a):
    out = [0]
    for v in a:
        out.append(out[-1] + v)
    return _i32(out)


def _zeros(n, dtype=torch.int32):
    return torch.zeros(n, dtype=dtype, device="cuda")


def _prepare_step(c, seed):
    dr, sm = _Draw(seed, c["dtype"]), _samples(c)
    H, dh, P, O = c["H"], c["dh"], c["P"], c["O"]
    d, scale = H * dh, 1.0 / math.sqrt(dh)
    lift = math.sqrt(2.5 / scale)               # a salient key's logit is 2.5 above the others' on average
    xs, qs, ks, qa, ka, va, decs = [], [], [], [], [], [], []
    for s in sm:
        x, q, k = dr.normal(s["N"], d), dr.normal(s["N"], H, dh), dr.normal(s["N"], H, dh)
        x[P:P + s["V"]] = dr.visual(s["V"], d, s["k"])
        dec = P + s["V"] + dr.subset(O, s["D"])
        u = torch.nn.functional.normalize(dr.normal(H, dh).float(), dim=1).mul_(lift).to(dr.dt)
        q[dec] += u
        k[P + dr.subset(s["V"], s["k"])] += u
        xs.append(x); qs.append(q); ks.append(k); decs.append(dec)
        qa.append(dr.normal(s["Nm"], H, dh))
        for t in (ka, va):
            r = dr.normal(s["Nm"], H, dh)
            r[P:P + s["k"]] = dr.visual(s["k"], d, s["k"]).view(-1, H, dh)
            t.append(r)
    lay = B.Layout([s["N"] for s in sm], [P] * c["B"], [s["V"] for s in sm], [t.cpu().numpy() for t in decs], [s["k"] for s in sm])
    st = dict(kind="step", separate=c["calls"] == "separate", lay=lay, scale=scale, q=torch.cat(qs), k=torch.cat(ks), x=torch.cat(xs),
              qa=torch.cat(qa), ka=torch.cat(ka), va=torch.cat(va), cu=_offsets(lay.Nm), min_keep=min(lay.keep), max_keep=max(lay.keep))
    out = dict(scores=_zeros(lay.sum_V, torch.float32), kept_idx=_zeros(lay.sum_keep), y=_zeros((lay.sum_Nm, d), dr.dt), assign=_zeros(lay.sum_V),
               counts=_zeros(lay.sum_keep), src_pos=_zeros(lay.sum_Nm), o=_zeros((lay.sum_Nm, H, dh), dr.dt))
    if st["separate"]:
        mask_id, max_D = 126336, lay.max_D
        cur = dr.ints(32000, lay.sum_N).to(torch.int32)
        prev = cur.clone()
        for b, dec in enumerate(decs):
            prev[sum(lay.N[:b]) + dec] = mask_id
        out.update(slot_of=_zeros(lay.sum_V), dec_idx=_zeros(c["B"] * max_D), dec_off=_zeros(c["B"] + 1), dec_count=_zeros(c["B"]))
        lay.dec_idx, lay.dec_off = out["dec_idx"], out["dec_off"]
        st.update(prev=prev, cur=cur, mask_id=mask_id, max_D=max_D)
        sizes = (c["B"], lay.max_N, lay.max_V, H, dh, lay.max_D)
        st["ws"] = B.workspace(max(B.d3tom_workspace_bytes(op, *sizes) for op in (B.D3TOM_OP_IMPORTANCE, B.D3TOM_OP_SELECT_TOPK, B.D3TOM_OP_MERGE)))
    else:
        out.update(keep_k=_zeros(c["B"]), kept_off=_zeros(c["B"] + 1), out_off=_zeros(c["B"] + 1))
        out["kept_idx"] = _zeros(c["B"] * st["max_keep"])
        st["ratio"] = torch.tensor([s["ratio"] for s in sm], dtype=torch.float64, device="cuda")
        st["ws"] = B.workspace(B.d3tom_merge_layer_workspace_bytes(c["B"], lay.max_N, lay.max_V, H, dh, lay.max_D))
    st["out"] = out
    return st


def _prepare_kv(c, seed):
    dr, sm = _Draw(seed, c["dtype"]), _samples(c)
    d, P = c["d"], c["P"]
    kc, vc, kept = [], [], []
    for s in sm:
        k = dr.normal(s["N"], d)
        k[P:] = dr.visual(s["V"], d, s["k"])
        kc.append(k); vc.append(dr.normal(s["N"], d)); kept.append(dr.subset(s["V"], s["k"]).to(torch.int32))
    lay = B.Layout([s["N"] for s in sm], [P] * c["B"], [s["V"] for s in sm], [[0]] * c["B"], [s["k"] for s in sm])
    out = dict(k_out=_zeros((lay.sum_Nm, d), dr.dt), v_out=_zeros((lay.sum_Nm, d), dr.dt), assign=_zeros(lay.sum_V), counts=_zeros(lay.sum_keep),
               src_pos=_zeros(lay.sum_Nm))
    ws = B.workspace(B.d3tom_workspace_bytes(B.D3TOM_OP_MERGE, c["B"], lay.max_N, lay.max_V, 1, d, 1))
    return dict(kind="kv", lay=lay, k_cache=torch.cat(kc), v_cache=torch.cat(vc), kept=torch.cat(kept), ws=ws, out=out)


def _prepare_attend(c, seed):
    dr, n = _Draw(seed, c["dtype"]), _lengths(c)
    H, dh, tot = c["H"], c["dh"], sum(n)
    st = dict(kind="attend", weighted=c["weighted"], q=dr.normal(tot, H, dh), k=dr.normal(tot, H, dh), v=dr.normal(tot, H, dh), cu=_offsets(n),
              longest=max(n), scale=1.0 / math.sqrt(dh), out=dict(o=_zeros((tot, H, dh), dr.dt)))
    if c["weighted"]:
        # all but 64 rows in front of the merged ones and 64 behind them (or a quarter of a short sample) stand for several tokens
        pad = [min(64, v // 4) for v in n]
        kept = [v - 2 * p for v, p in zip(n, pad)]
        st.update(counts=(1 + dr.ints(6, sum(kept))).to(torch.int32), kept_off=_offsets(kept), vis_start=_i32(pad))
    return st


def _prepare_stack(c, seed):
    dr, sm = _Draw(seed, c["dtype"]), _samples(c)
    H, dh, F, P, O, L = c["H"], c["dh"], c["F"], c["P"], c["O"], c["L"]
    d = H * dh
    gain = lambda: dr.normal(d, std=0.1) + 1
    blocks = [dict(attn_norm=gain(), w_qkv=dr.normal(3 * d, d, std=0.02), w_o=dr.normal(d, d, std=0.02), ffn_norm=gain(),
                   w_gate_up=dr.normal(2 * F, d, std=0.02), w_down=dr.normal(d, F, std=0.02)) for _ in range(L)]
    mask_row, xs, decs = dr.normal(d), [], []
    for s in sm:
        x = dr.normal(s["N"], d)
        x[P:P + s["V"]] = dr.visual(s["V"], d, s["k"])
        dec = P + s["V"] + dr.subset(O, s["D"])
        resp = x[dec].clone()
        x[P + s["V"]:] = mask_row                # response positions hold the mask row, except the decided ones
        x[dec] = resp
        xs.append(x); decs.append(dec.to(torch.int32))
    N, V, D, k = ([s[f] for s in sm] for f in ("N", "V", "D", "k"))
    merged = min(D) > 0
    rows = sum(s["Nm"] if merged else s["N"] for s in sm)
    y, src = _zeros((sum(N), d), dr.dt), _zeros(sum(N))
    ws = B.workspace(B.d3tom_stack_batch_workspace_bytes(c["B"], sum(N), max(N), d, H, F, sum(V), max(V), max(max(D), 1)))
    return dict(kind="stack", x=torch.cat(xs), N=N, V=V, D=D, k=k, vis=[P] * c["B"], H=H, F=F, L=L, keep=blocks, blocks=B.block_weights(blocks),
                dec=torch.cat(decs) if merged else None, y=y, src=src, ws=ws, out=dict(y=y[:rows], src_pos=src[:rows]))


def prepare(case, seed):
    return {"step": _prepare_step, "kv": _prepare_kv, "attend": _prepare_attend, "stack": _prepare_stack}[case["kind"]](case, seed)


# ---- one pass --------------------------------------------------------------------------------------------------------------
def _run_step(s):
    lay, out = s["lay"], s["out"]
    if s["separate"]:
        B.d3tom_update_deciders(s["prev"], s["cur"], s["mask_id"], lay.seq_off, s["max_D"], out["dec_idx"], out["dec_off"], out["dec_count"])
        B.d3tom_importance(s["q"], s["k"], lay, s["scale"], out["scores"], s["ws"])
        B.d3tom_select_topk(out["scores"], lay, out["kept_idx"], out["slot_of"])
        B.d3tom_merge(s["x"], None, lay, out["kept_idx"], B.D3TOM_MERGE_MEAN, out["y"], out["assign"], out["counts"], out["src_pos"], s["ws"])
    else:
        B.d3tom_merge_layer(s["q"], s["k"], s["x"], None, lay, s["scale"], s["ratio"], s["min_keep"], s["max_keep"], B.D3TOM_MERGE_MEAN,
                            out["scores"], out["keep_k"], out["kept_off"], out["kept_idx"], out["out_off"], out["y"], out["assign"],
                            out["counts"], out["src_pos"], s["ws"])
    B.d3tom_attend(s["qa"], s["ka"], s["va"], s["cu"], lay.max_Nm, s["scale"], out["o"])
    return out


def run(state):
    s, out = state, state["out"]
    if s["kind"] == "step":
        return _run_step(s)
    if s["kind"] == "kv":
        B.d3tom_merge_kv(s["k_cache"], s["v_cache"], s["lay"], s["kept"], B.D3TOM_MERGE_MEAN, out["k_out"], out["v_out"], out["assign"],
                         out["counts"], out["src_pos"], s["ws"])
    elif s["kind"] == "attend":
        if s["weighted"]:
            B.d3tom_attend_weighted(s["q"], s["k"], s["v"], s["cu"], s["longest"], s["scale"], s["counts"], s["kept_off"], s["vis_start"], out["o"])
        else:
            B.d3tom_attend(s["q"], s["k"], s["v"], s["cu"], s["longest"], s["scale"], out["o"])
    else:
        B.d3tom_stack_step_batch(s["x"], s["N"], s["H"], s["F"], s["blocks"], s["L"], 1, s["dec"], s["D"], s["vis"], s["V"], s["k"],
                                 B.D3TOM_MERGE_MEAN, 1e-5, 10000.0, s["y"], s["ws"], src_pos=s["src"])
    return out


# ---- what a pass cannot do without -------------------------------------------------------------------------------------------
def work(case):
    eb = 4 if case["dtype"] == "f32" else 2
    by = fl = 0.0
    if case["kind"] == "attend":
        d = case["H"] * case["dh"]
        n = _lengths(case)
        return {"bytes": 4.0 * sum(n) * d * eb, "flops": 4.0 * d * sum(v * v for v in n)}
    sm = _samples(case)
    if case["kind"] == "kv":
        d = case["d"]
        for s in sm:
            by += 2.0 * (s["N"] + s["Nm"]) * d * eb + 4 * (2 * s["V"] + s["k"] + s["Nm"])
            fl += 2.0 * (s["V"] - s["k"]) * s["k"] * d
        return {"bytes": by, "flops": fl}
    d = case["H"] * case["dh"]
    if case["kind"] == "step":
        for s in sm:
            by += (s["N"] + s["D"]) * d * eb                                       # keys, decider queries
            by += (s["N"] + s["Nm"]) * d * eb + 4 * (2 * s["V"] + 2 * s["k"] + s["Nm"])   # rows in, rows out, scores and indices
            by += 4 * s["Nm"] * d * eb                                             # attention
            fl += 2.0 * s["D"] * s["N"] * d + 2.0 * (s["V"] - s["k"]) * s["k"] * d + 4.0 * s["Nm"] ** 2 * d
        return {"bytes": by, "flops": fl}
    F, L = case["F"], case["L"]
    merged = min(s["D"] for s in sm) > 0
    by += 2.0 * L * (4 * d * d + 3 * d * F)                                        # weights
    for s in sm:
        Nm = s["Nm"] if merged else s["N"]
        by += (s["N"] + Nm) * d * eb
        att = lambda n: 8.0 * n * d * d + 4.0 * n * n * d
        fl += att(s["N"]) + (L - 1) * att(Nm) + L * 6.0 * Nm * d * F
        if merged:
            fl += 2.0 * s["D"] * s["N"] * d + 2.0 * (s["V"] - s["k"]) * s["k"] * d
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    if case["kind"] == "stack":
        # every stored tensor between two stages is rounded to bf16; four blocks cross some forty of them
        return {"rel": 2e-2, "max": 0.8}
    if case["kind"] == "attend":
        return {"rel": 1e-2}
    # a near-tie of two cosines may send a token to another row of its cluster
    return {"rel": 1e-2, "max": 0.8, "differ": 5e-3}
