"""What a user of the refresh step has it do, as cases that can be timed and checked.

A case is a dict of plain values; ``prepare`` makes its inputs on the GPU from a
seed, ``run`` takes them once through the package's public calls, and ``exact``
gives the same outputs from plain torch in 64 bits.  The kinds of case:

  step      one request: every layer scored, one selection, merge and refresh
            of the selected rows in every layer (RefreshStep);
  score     the scoring pass over one or several layers;
  select    image reweighting and the global top-k;
  refresh   merge and refresh attention of a given set of rows;
  residual  the residual-error diagnostic of a refresh set.

Inputs follow the synthetic workloads of the package: keys and queries ~ N(0, 1)
elementwise, values of log-normal norm, a few attention sinks (keys along one
direction that every span query leans toward, small values), and a quarter of
the images aligned with the span queries.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_05821_amd import api

DEV = "cuda"


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------

def _case(kind, **kw):
    c = dict(kind=kind, dtype="bf16", layers=1, hq=28, hkv=4, d=128, n_q=128, prefix=512, sep=0, images=16,
             tokens=16384, ragged=False, k=0, page=0, text=False, tabled=False, norm="causal", agg="mean",
             rule="composite", lam=1.0, samples=0)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest request: one small image, fp32 cache, 8 heads of 64 (launch latency).
        _case("step", name="step_image_f32", dtype="f32", hq=8, hkv=8, d=64, n_q=32, prefix=64, images=1,
              tokens=576, k=57),
        # One ordinary image through a grouped-head bf16 model, one layer.
        _case("step", name="step_image_gqa", n_q=64, prefix=256, images=1, tokens=1024, k=102),
        # A few images through every layer of a 28-layer model at a 10% budget.
        _case("step", name="step_images_28_layers", layers=28, n_q=96, prefix=128, images=4, tokens=5184, k=518),
        # The scoring pass of a 16k-token multi-image context.
        _case("score", name="score_16k", sep=16),
        # The same span where the model's own attention left the row log-sum-exps and the cache its value norms.
        _case("score", name="score_16k_tabled", sep=16, tabled=True),
        # The selection over that context.
        _case("select", name="select_16k", sep=16, k=1638),
        # Its merge and recompute at a 10% budget: the headline step's largest part.
        _case("refresh", name="refresh_16k", sep=16, k=1638),
        # A served request: paged cache, images of odd sizes, heads of 64, and the text rows recomputed beside the
        # selected ones.
        _case("refresh", name="refresh_slides_paged", hq=16, hkv=4, d=64, n_q=77, prefix=201, sep=5, images=13,
              tokens=9001, ragged=True, k=911, page=256, text=True),
        # A 64-page document: scoring of a span over four scored layers.
        _case("score", name="score_document", layers=4, n_q=256, prefix=1024, images=64, tokens=65536),
        # The selection over the document.
        _case("select", name="select_document", n_q=256, prefix=1024, images=64, tokens=65536, k=6553),
        # The document's recompute in those four layers: the largest call.
        _case("refresh", name="refresh_document", layers=4, n_q=256, prefix=1024, images=64, tokens=65536, k=6553),
        # The diagnostic of a 10% refresh set at 16k with five displacement samples.
        _case("residual", name="residual_16k", sep=16, k=1638, samples=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "score", "score", "select", "refresh", "refresh", "residual"])
    hq, hkv, d = rng.choice([(28, 4, 128), (28, 4, 128), (32, 8, 128), (16, 4, 64), (8, 8, 64), (14, 2, 64)])
    images = _log_int(rng, 1, 64)
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    # The span, the context and the budget; each kind within the work of the largest listed case.
    top = {"step": 12000, "score": 60000, "select": 120000, "refresh": 40000, "residual": 16000}[kind]
    if dtype == "f32" and kind != "select":
        top = 4000
    tokens = max(images, _log_int(rng, 300, top))
    layers = 1
    if kind == "step":
        layers = rng.choice([1, 1, 4, 9, 28]) if dtype == "bf16" else rng.choice([1, 3])
    elif kind == "score" and dtype == "bf16":
        layers = rng.choice([1, 1, 2, 5])
    elif kind == "refresh" and dtype == "bf16":
        layers = rng.choice([1, 1, 3])
    c = _case(kind, dtype=dtype, layers=layers, hq=hq, hkv=hkv, d=d, n_q=_log_int(rng, 5, 256),
              prefix=_log_int(rng, 8, 1024), sep=rng.choice([0, 3, 16]), images=images, tokens=tokens,
              ragged=rng.random() < 0.5, lam=rng.choice([1.0, 1.0, 0.5]))
    c["k"] = max(1, min(tokens, int(tokens * rng.choice([0.05, 0.1, 0.1, 0.2]))))
    if kind == "score":
        c["k"] = 0
        if layers == 1:
            c["tabled"] = rng.random() < 0.3
        if not c["tabled"]:
            c["norm"] = rng.choice(["causal", "causal", "visual"])
        c["agg"] = rng.choice(["mean", "mean", "rms"])
    elif kind == "select":
        c["rule"] = rng.choice(["composite", "composite", "attention"])
    elif kind == "refresh":
        c["text"] = rng.random() < 0.5
    elif kind == "residual":
        c["samples"] = rng.choice([0, 3, 5])
    if kind in ("score", "refresh", "residual") and rng.random() < 0.4:
        c["page"] = rng.choice([64, 256])
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _layout(c):
    """(img_pos, img_off, q_pos0, n_ctx): [prefix][separator, image]...[span]."""
    n = c["images"]
    if c["ragged"]:  # sizes between about 1/2 and 3/2 of the mean
        w = np.array([0.5 + ((7 * j + 3) % 11) / 10.0 for j in range(n)])
        off = np.floor(np.concatenate([[0.0], np.cumsum(w)]) / w.sum() * (c["tokens"] - n)).astype(np.int64)
        off = off + np.arange(n + 1)
    else:
        off = (np.arange(n + 1, dtype=np.int64) * c["tokens"]) // n
    off[-1] = c["tokens"]
    pos = c["prefix"] + c["sep"] * np.arange(1, n + 1) + off[:-1]
    q0 = int(c["prefix"] + c["sep"] * n + c["tokens"])
    return pos.astype(np.int32), off.astype(np.int32), q0, q0 + c["n_q"]


def _vis_positions(pos, off):
    return np.concatenate([np.arange(p, p + off[j + 1] - off[j]) for j, p in enumerate(pos)])


class _Gen:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device=DEV, dtype=torch.float32)

    def uniform(self, *shape):
        return torch.rand(*shape, generator=self.g, device=DEV, dtype=torch.float32)


def _dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _relevant(c, gen):
    """A quarter of the images, one at least unless there is only one image."""
    rel = torch.zeros(c["images"], dtype=torch.bool, device=DEV)
    if c["images"] > 1:
        rel[torch.argsort(gen.uniform(c["images"]))[: max(1, c["images"] // 4)]] = True
    return rel


def _caches(c, gen, lay, rel):
    """k, v [layers, n_ctx, hkv, d] and q [layers, n_q, hq, d]."""
    pos, off, q0, n_ctx = lay
    dt, hkv, hq, d = _dtype(c), c["hkv"], c["hq"], c["d"]
    vis = torch.from_numpy(_vis_positions(pos, off)).to(DEV)
    img = torch.from_numpy(np.repeat(np.arange(c["images"]), np.diff(off))).to(DEV)
    b = torch.nn.functional.normalize(gen.normal(hkv, d), dim=1)
    w = gen.normal(hkv, d)
    w = torch.nn.functional.normalize(w - (w * b).sum(1, keepdim=True) * b, dim=1)
    sinks = vis[torch.argsort(gen.uniform(c["tokens"]))[: max(1, c["tokens"] // 100)]]
    rel_pos = vis[rel[img]]
    head = torch.arange(hq, device=DEV) // (hq // hkv)
    k = torch.empty(c["layers"], n_ctx, hkv, d, dtype=dt, device=DEV)
    v = torch.empty_like(k)
    q = torch.empty(c["layers"], c["n_q"], hq, d, dtype=dt, device=DEV)
    for li in range(c["layers"]):
        x = gen.normal(n_ctx, hkv, d)
        x[rel_pos] = math.sqrt(0.7) * x[rel_pos] + math.sqrt(0.3 * d) * w
        x[sinks] = 3.0 * math.sqrt(d) * b
        k[li] = x
        y = torch.nn.functional.normalize(gen.normal(n_ctx, hkv * d), dim=1)
        rho = torch.exp(0.5 * gen.normal(n_ctx, 1))
        rho[sinks] *= 0.05
        v[li] = (y * rho).view(n_ctx, hkv, d)
        z = gen.normal(c["n_q"], hq, d)
        if bool(rel.any()):
            z = math.sqrt(0.7) * z + math.sqrt(0.3 * d) * w[head]
        q[li] = z + 2.0 * b[head]
    return k, v, q


def _rows(c, gen, lay, rel):
    """Sequence positions of a refresh set of k visual tokens, mostly in the relevant images, ascending."""
    pos, off, _, _ = lay
    vis = torch.from_numpy(_vis_positions(pos, off)).to(DEV)
    img = torch.from_numpy(np.repeat(np.arange(c["images"]), np.diff(off))).to(DEV)
    score = torch.log(gen.uniform(c["tokens"]).clamp_min(1e-9)) / (1.0 + 2.0 * rel[img].float())
    sel = torch.sort(torch.topk(score, c["k"]).indices).values
    return sel, vis[sel]


def _paged(c, gen, k, v, n_ctx):
    """The caches as pools of pages in a shuffled order, with spare pages."""
    page = c["page"]
    n = -(-n_ctx // page)
    pool = n + n // 8 + 1
    table = torch.argsort(gen.uniform(pool))[:n]
    row = (table[:, None] * page + torch.arange(page, device=DEV)[None, :]).reshape(-1)[:n_ctx]
    out = []
    for x in (k, v):
        p = torch.zeros(c["layers"], pool * page, c["hkv"], c["d"], dtype=x.dtype, device=DEV)
        p[:, row] = x
        out.append(p.view(c["layers"], pool, page, c["hkv"], c["d"]))
    return out[0], out[1], table.to(torch.int32), row


def _lse64(c, q, k, q0):
    """Row log-sum-exps [n_q, hq] of the span over its causal rows, in 64 bits."""
    hkv, g, d = c["hkv"], c["hq"] // c["hkv"], c["d"]
    out = torch.empty(c["n_q"], c["hq"], dtype=torch.float64, device=DEV)
    key = torch.arange(k.shape[0], device=DEV)
    for h in range(hkv):
        kh = k[:, h].double()
        for r0 in range(0, c["n_q"], 64):
            r1 = min(c["n_q"], r0 + 64)
            z = q[r0:r1, h * g:(h + 1) * g].double().reshape(-1, d) @ kh.t() / math.sqrt(d)
            z = z.view(r1 - r0, g, -1)
            z.masked_fill_((key[None, :] > q0 + torch.arange(r0, r1, device=DEV)[:, None])[:, None, :], -math.inf)
            out[r0:r1, h * g:(h + 1) * g] = torch.logsumexp(z, dim=2)
    return out


def prepare(case, seed):
    c, gen, lay = case, _Gen(seed), _layout(case)
    pos, off, q0, n_ctx = lay
    img = api.ImageTable(pos, off)
    st = {"c": c, "img": img, "q0": q0}
    rel = _relevant(c, gen)
    f32 = dict(dtype=torch.float32, device=DEV)
    if c["kind"] == "select":
        # layer sums as a scoring pass leaves them: log-normal attention, more of it in the relevant images
        of = torch.from_numpy(np.repeat(np.arange(c["images"]), np.diff(off))).to(DEV)
        a = torch.exp(gen.normal(c["tokens"])) * (1.0 + 3.0 * rel[of].float()) / n_ctx
        s = a * torch.exp(0.5 * gen.normal(c["tokens"]))
        nbytes = int(api.lib().conduit_select_workspace_bytes(c["tokens"], c["images"]))
        st.update(a=a, s=s, ws=torch.empty(max(nbytes, 1), dtype=torch.uint8, device=DEV),
                  idx=torch.zeros(c["k"], dtype=torch.int32, device=DEV),
                  pos=torch.zeros(c["k"], dtype=torch.int32, device=DEV),
                  mask=torch.zeros(c["tokens"], dtype=torch.uint8, device=DEV),
                  shat=torch.zeros(c["tokens"], **f32), coef=torch.zeros(c["images"], **f32))
        return st
    k, v, q = _caches(c, gen, lay, rel)
    if c["kind"] == "step":
        st.update(k=k, v=v, q=q)
        layers = [{"k": k[i], "v": v[i], "q": q[i]} for i in range(c["layers"])]
        st["step"] = api.RefreshStep(layers, c["hq"], q0, img, c["k"], lam=c["lam"], device=DEV)
        shape = (c["layers"], c["k"], c["hkv"], c["d"])
        kn, vn = gen.normal(*shape).to(k.dtype), (gen.normal(*shape) / math.sqrt(c["hkv"] * c["d"])).to(k.dtype)
        qs = gen.normal(c["layers"], c["k"], c["hq"], c["d"]).to(k.dtype)
        st["fresh"] = [{"k_new": kn[i], "v_new": vn[i], "q_sel": qs[i]} for i in range(c["layers"])]
        return st
    if c["page"]:
        kp, vp, table, row = _paged(c, gen, k, v, n_ctx)
        st.update(k=kp, v=vp, table=table, row=row)
        kvs = [api.kv_desc_paged(kp[i], vp[i], table, n_ctx, c["hq"]) for i in range(c["layers"])]
    else:
        st.update(k=k, v=v)
        kvs = [api.kv_desc(k[i], v[i], c["hq"]) for i in range(c["layers"])]
    st.update(kvs=kvs, q=[q[i] for i in range(c["layers"])])
    if c["kind"] == "score":
        st.update(s=torch.zeros(c["tokens"], **f32), a=torch.zeros(c["tokens"], **f32),
                  norm=api.NORM_VISUAL_ONLY if c["norm"] == "visual" else api.NORM_CAUSAL_ROW,
                  agg=api.AGG_RMS if c["agg"] == "rms" else api.AGG_MEAN)
        nbytes = api.score_layers_workspace_bytes(kvs[0], c["n_q"], img, c["layers"])
        st["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        st["lse"] = torch.zeros(c["n_q"], c["hq"], **f32)
        if c["tabled"]:
            vis = torch.from_numpy(_vis_positions(pos, off)).to(DEV)
            st["lse_in"] = _lse64(c, q[0], k[0], q0).float()
            st["vnorm"] = v[0][vis].double().reshape(c["tokens"], -1).norm(dim=1).float()
        return st
    sel, rows = _rows(c, gen, lay, rel)
    if c["kind"] == "residual":
        st["lse"] = _lse64(c, q[0], k[0], q0).float()
        st["refreshed"] = torch.zeros(c["tokens"], dtype=torch.uint8, device=DEV)
        st["refreshed"][sel] = 1
        m = c["samples"]
        st["z"] = gen.normal(m, c["tokens"], c["hkv"], c["d"]).to(k.dtype) if m else None
        st["err"] = torch.zeros(max(m, 1), c["n_q"], c["hq"], **f32)
        nbytes = api.residual_workspace_bytes(kvs[0], c["n_q"], img, max(m, 1), m > 0)
        st["ws"] = torch.empty(max(nbytes, 1), dtype=torch.uint8, device=DEV)
        return st
    # refresh
    if c["text"]:
        keep = torch.ones(n_ctx, dtype=torch.bool, device=DEV)
        keep[torch.from_numpy(_vis_positions(pos, off)).to(DEV)] = False
        rows = torch.cat([rows, keep.nonzero()[:, 0]])
    n = rows.numel()
    st["rows"] = rows.to(torch.int32)
    st["k_new"] = [gen.normal(n, c["hkv"], c["d"]).to(k.dtype) for _ in kvs]
    st["v_new"] = [(gen.normal(n, c["hkv"], c["d"]) / math.sqrt(c["hkv"] * c["d"])).to(k.dtype) for _ in kvs]
    st["q_sel"] = [gen.normal(n, c["hq"], c["d"]).to(k.dtype) for _ in kvs]
    st["out"] = [torch.zeros(n, c["hq"], c["d"], dtype=k.dtype, device=DEV) for _ in kvs]
    st["lse"] = [torch.zeros(n, c["hq"], **f32) for _ in kvs]
    nbytes = api.refresh_layers_workspace_bytes(kvs[0], n, len(kvs))
    st["ws"] = torch.empty(max(nbytes, 1), dtype=torch.uint8, device=DEV)
    return st


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    c, st = state["c"], state
    if c["kind"] == "step":
        step = st["step"]
        step.score_and_select()
        step.refresh(st["fresh"])
        return {"idx": step.idx, "pos": step.pos, "mask": step.mask, "shat": step.shat, "c": step.c,
                "out": step.out, "lse": step.lse, "k": st["k"], "v": st["v"]}
    if c["kind"] == "score":
        if c["layers"] > 1:
            api.conduit_score_layers(st["kvs"], st["q"], st["q0"], st["img"], st["s"], st["a"], norm=st["norm"],
                                     agg=st["agg"], ws=st["ws"])
            return {"s": st["s"], "a": st["a"]}
        if c["tabled"]:
            api.conduit_score(st["kvs"][0], st["q"][0], st["q0"], st["img"], st["s"], st["a"], agg=st["agg"],
                              row_lse_in=st["lse_in"], vnorm_in=st["vnorm"], ws=st["ws"])
            return {"s": st["s"], "a": st["a"]}
        api.conduit_score(st["kvs"][0], st["q"][0], st["q0"], st["img"], st["s"], st["a"], norm=st["norm"],
                          agg=st["agg"], row_lse_out=st["lse"], ws=st["ws"])
        return {"s": st["s"], "a": st["a"], "lse": st["lse"]}
    if c["kind"] == "select":
        api.conduit_select_topk(st["s"], st["a"], c["layers"], st["img"], c["lam"], c["k"], st["idx"], st["pos"],
                                mask_out=st["mask"], shat_out=st["shat"], c_out=st["coef"], ws=st["ws"],
                                rule=api.RANK_ATTENTION if c["rule"] == "attention" else api.RANK_COMPOSITE)
        return {"idx": st["idx"], "pos": st["pos"], "mask": st["mask"], "shat": st["shat"], "c": st["coef"]}
    if c["kind"] == "residual":
        api.conduit_residual_error(st["kvs"][0], st["q"][0], st["q0"], st["img"], st["lse"], st["refreshed"],
                                   st["err"], z=st["z"], ws=st["ws"])
        return {"err": st["err"]}
    if c["layers"] > 1:
        api.conduit_scatter_kv_layers(st["kvs"], st["rows"], st["k_new"], st["v_new"])
        api.conduit_refresh_attn_layers(st["kvs"], st["q_sel"], st["rows"], st["out"], lse_out=st["lse"],
                                        ws=st["ws"])
    else:
        api.conduit_merge_refresh_attn(st["kvs"][0], st["rows"], st["k_new"][0], st["v_new"][0], st["q_sel"][0],
                                       st["out"][0], lse_out=st["lse"][0], ws=st["ws"])
    return {"out": st["out"], "lse": st["lse"], "k": st["k"], "v": st["v"]}


# ---------------------------------------------------------------------------
# The work of one pass and how far results may be apart
# ---------------------------------------------------------------------------

def _row_keys(c, lay):
    """Keys that the refreshed rows attend to, in all (rows spread over the images), and the rows."""
    pos, off, q0, n_ctx = lay
    mean = float(_vis_positions(pos, off).mean()) + 1.0
    n, keys = c["k"], c["k"] * mean
    if c["text"]:
        vis = np.zeros(n_ctx, dtype=bool)
        vis[_vis_positions(pos, off)] = True
        text = np.flatnonzero(~vis)
        n, keys = n + len(text), keys + float((text + 1).sum())
    return n, keys


def work(case):
    c, lay = case, _layout(case)
    _, _, q0, n_ctx = lay
    e = 4 if c["dtype"] == "f32" else 2
    hq, hkv, d, nq, nv, nl = c["hq"], c["hkv"], c["d"], c["n_q"], c["tokens"], c["layers"]
    row = hkv * d * e
    b = f = 0.0
    if c["kind"] in ("score", "step"):
        # both passes over the logits (row sums, then column sums); the visual rows' V for their norms
        f += nl * 2.0 * nq * hq * d * nv
        if not c["tabled"]:
            dom = nv if c["norm"] == "visual" else q0 + (nq + 1) / 2
            f += nl * 2.0 * nq * hq * d * dom
            keys = nv if c["norm"] == "visual" else n_ctx
            b += nl * (keys * row + nv * row)
        else:
            b += nv * row + nv * 4 + nq * hq * 4
        b += nl * nq * hq * d * e + 8.0 * nv
    if c["kind"] in ("select", "step"):
        b += nv * (8 + 4 + 1) + 8.0 * c["k"]
    if c["kind"] in ("refresh", "step"):
        n, keys = _row_keys(c, lay)
        f += nl * 4.0 * hq * d * keys
        b += nl * (2.0 * n_ctx * row + 4.0 * n * row + 2.0 * n * hq * d * e + 4.0 * n * hq)
    if c["kind"] == "residual":
        m = max(c["samples"], 1)
        f += 2.0 * nq * hq * d * nv * (1 + m)
        # K of the visual keys, V once (its norms, or the displacement itself), the samples
        b += 2.0 * nv * row + nq * hq * (d * e + 4) + c["samples"] * nv * row + 4.0 * m * nq * hq + nv
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times the distance from exact() measured on the card: 5e-8 (select), 3e-7 (score), 3e-7 to 7e-7 (fp32
    attention and residual), 2.8e-3 (bf16 attention: 16-bit probabilities and outputs), 5.4e-4 (bf16 residual)."""
    c = case
    bf16 = c["dtype"] == "bf16"
    if c["kind"] == "select":
        # image means in another order; a swap at the threshold moves the entries between the two
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}
    if c["kind"] == "score":
        # 32-bit sums; the row log-sum-exp enters an exponent, |b| 2^-24 absolute
        return {"rel": 3e-6, "max": 1e-4}
    if c["kind"] == "step":
        return {"rel": 1e-2 if bf16 else 3e-6, "max": 0.2 if bf16 else 2e-4, "differ": 0.01}
    if c["kind"] == "residual":
        return {"rel": 3e-3 if bf16 else 4e-6, "max": 0.1 if bf16 else 2e-4}
    return {"rel": 1e-2, "max": 0.2} if bf16 else {"rel": 3e-6, "max": 2e-4}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits
# ---------------------------------------------------------------------------

_CHUNK = 1 << 27  # logits held at once


def _score64(c, lay, k, v, q, lse_in=None, vnorm=None):
    """a_t, ||V_t|| of one layer and the row log-sum-exps."""
    pos, off, q0, _ = lay
    vis = torch.from_numpy(_vis_positions(pos, off)).to(DEV)
    hkv, g, d = c["hkv"], c["hq"] // c["hkv"], c["d"]
    a = torch.zeros(c["tokens"], dtype=torch.float64, device=DEV)
    lse = torch.empty(c["n_q"], c["hq"], dtype=torch.float64, device=DEV)
    key = torch.arange(k.shape[0], device=DEV)
    rows = max(1, _CHUNK // (g * k.shape[0]))
    for h in range(hkv):
        kh = k[:, h].double()
        for r0 in range(0, c["n_q"], rows):
            r1 = min(c["n_q"], r0 + rows)
            z = (q[r0:r1, h * g:(h + 1) * g].double().reshape(-1, d) @ kh.t() / math.sqrt(d)).view(r1 - r0, g, -1)
            if lse_in is not None:
                b = lse_in[r0:r1, h * g:(h + 1) * g].double()
            else:
                if c["norm"] == "visual":
                    b = torch.logsumexp(z[:, :, vis], dim=2)
                else:
                    z.masked_fill_((key[None, :] > q0 + torch.arange(r0, r1, device=DEV)[:, None])[:, None, :],
                                   -math.inf)
                    b = torch.logsumexp(z, dim=2)
                lse[r0:r1, h * g:(h + 1) * g] = b
            p = torch.exp(z[:, :, vis] - b[:, :, None])
            a += (p * p).sum(dim=(0, 1)) if c["agg"] == "rms" else p.sum(dim=(0, 1))
    a /= c["n_q"] * c["hq"]
    if c["agg"] == "rms":
        a = a.sqrt()
    n = vnorm.double() if vnorm is not None else v[vis].double().reshape(c["tokens"], -1).norm(dim=1)
    return a, n, lse


def _select64(c, lay, s, a):
    pos, off, _, _ = lay
    n = torch.from_numpy(np.diff(off)).to(DEV)
    img = torch.repeat_interleave(torch.arange(c["images"], device=DEV), n)
    g = torch.zeros(c["images"], dtype=torch.float64, device=DEV).index_add_(0, img, a.double())
    g = g / (c["layers"] * n)
    coef = (1.0 - c["lam"]) + c["lam"] * g / g.mean()
    shat = (a if c["rule"] == "attention" else s).double() / c["layers"] * coef[img]
    return coef, shat, torch.sort(torch.topk(shat, c["k"]).indices).values


def _attend64(c, k, v, q, rows):
    """Causal attention of the rows over one layer's merged cache, and their log-sum-exps."""
    hkv, g, d = c["hkv"], c["hq"] // c["hkv"], c["d"]
    n = rows.numel()
    out = torch.empty(n, c["hq"], d, dtype=torch.float64, device=DEV)
    lse = torch.empty(n, c["hq"], dtype=torch.float64, device=DEV)
    key = torch.arange(k.shape[0], device=DEV)
    step = max(1, _CHUNK // (g * k.shape[0]))
    for h in range(hkv):
        kh, vh = k[:, h].double(), v[:, h].double()
        for r0 in range(0, n, step):
            r1 = min(n, r0 + step)
            z = (q[r0:r1, h * g:(h + 1) * g].double().reshape(-1, d) @ kh.t() / math.sqrt(d)).view(r1 - r0, g, -1)
            z.masked_fill_((key[None, :] > rows[r0:r1, None])[:, None, :], -math.inf)
            b = torch.logsumexp(z, dim=2)
            p = z.sub_(b[:, :, None]).exp_()
            out[r0:r1, h * g:(h + 1) * g] = (p.view(-1, p.shape[2]) @ vh).view(r1 - r0, g, d)
            lse[r0:r1, h * g:(h + 1) * g] = b
    return out, lse


def _logical(c, st, x):
    """A layer's cache in token order."""
    return x.reshape(-1, c["hkv"], c["d"])[st["row"]] if c["page"] else x


def exact(case, seed):
    c, lay = case, _layout(case)
    st = prepare(case, seed)
    pos, off, q0, n_ctx = lay
    vis = torch.from_numpy(_vis_positions(pos, off)).to(DEV)
    if c["kind"] == "select":
        coef, shat, _ = _select64(c, lay, st["s"], st["a"])
        return {"idx": None, "pos": None, "mask": None, "shat": shat, "c": coef}
    if c["kind"] == "score":
        s = torch.zeros(c["tokens"], dtype=torch.float64, device=DEV)
        a = torch.zeros_like(s)
        for i in range(c["layers"]):
            ai, ni, lse = _score64(c, lay, _logical(c, st, st["k"][i]), _logical(c, st, st["v"][i]), st["q"][i],
                                   st.get("lse_in"), st.get("vnorm"))
            a += ai
            s += ai * ni
        return {"s": s, "a": a} if c["layers"] > 1 or c["tabled"] else {"s": s, "a": a, "lse": lse}
    if c["kind"] == "residual":
        hkv, g, d, m = c["hkv"], c["hq"] // c["hkv"], c["d"], c["samples"]
        k = _logical(c, st, st["k"][0])[vis].double()
        v = _logical(c, st, st["v"][0])[vis].double()
        left = st["refreshed"] == 0
        sig = 0.5 * v.reshape(c["tokens"], -1).norm(dim=1) / math.sqrt(hkv * d)
        err = torch.empty(max(m, 1), c["n_q"], c["hq"], dtype=torch.float64, device=DEV)
        for h in range(hkv):
            z = st["q"][0][:, h * g:(h + 1) * g].double().reshape(-1, d) @ k[:, h].t() / math.sqrt(d)
            al = torch.exp(z - st["lse"][:, h * g:(h + 1) * g].double().reshape(-1, 1)) * left
            for j in range(max(m, 1)):
                x = st["z"][j, :, h].double() * sig[:, None] if m else v[:, h]
                err[j, :, h * g:(h + 1) * g] = (al @ x).square().sum(dim=1).view(c["n_q"], g)
        return {"err": err}
    if c["kind"] == "step":
        s = torch.zeros(c["tokens"], dtype=torch.float64, device=DEV)
        a = torch.zeros_like(s)
        for i in range(c["layers"]):
            ai, ni, _ = _score64(c, lay, st["k"][i], st["v"][i], st["q"][i])
            a += ai
            s += ai * ni
        coef, shat, sel = _select64(c, lay, s, a)
        rows = vis[sel]
        k, v, out, lse = st["k"].double(), st["v"].double(), [], []
        for i in range(c["layers"]):
            f = st["fresh"][i]
            k[i, rows], v[i, rows] = f["k_new"].double(), f["v_new"].double()
            o, b = _attend64(c, k[i], v[i], f["q_sel"], rows)
            out.append(o)
            lse.append(b)
        return {"idx": None, "pos": None, "mask": None, "shat": shat, "c": coef, "out": out, "lse": lse, "k": k,
                "v": v}
    rows, out, lse = st["rows"].long(), [], []
    k, v = st["k"].double(), st["v"].double()
    for i in range(c["layers"]):
        kf, vf = k[i].view(-1, c["hkv"], c["d"]), v[i].view(-1, c["hkv"], c["d"])
        at = st["row"][rows] if c["page"] else rows
        kf[at], vf[at] = st["k_new"][i].double(), st["v_new"][i].double()
        o, b = _attend64(c, _logical(c, st, k[i]), _logical(c, st, v[i]), st["q_sel"][i], rows)
        out.append(o)
        lse.append(b)
    return {"out": out, "lse": lse, "k": k, "v": v}
