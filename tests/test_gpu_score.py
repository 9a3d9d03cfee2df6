"""Scoring pass on the GPU (conduit_score) against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import conduit_oracle as O
from paper_2609_05821_amd import api, workloads as W
from tests.gpu_helpers import DEV, assert_scores, bits, to_dev, to_f64

pytestmark = pytest.mark.gpu

CASES = {
    "cfg1_fp32_mha": lambda: W.config(1),
    "cfg2_bf16_gqa": lambda: W.config(2),
    "ragged_bf16_gqa7": lambda: W.custom(1, 28, 4, 128, 19, 13, [37, 250, 301], 5, "bf16", n_sinks=6,
                                         n_relevant=1, seed=3),
    "ragged_bf16_d64_gqa4": lambda: W.custom(1, 8, 2, 64, 40, 7, [100, 33], 3, "bf16", n_sinks=2,
                                             seed=4),
    "ragged_bf16_mha": lambda: W.custom(1, 4, 4, 128, 9, 1, [70], 0, "bf16", seed=5),
    "ragged_fp32_d128_gqa2": lambda: W.custom(1, 4, 2, 128, 5, 3, [20, 45, 11], 2, "f32", seed=6),
    "one_visual_token": lambda: W.custom(1, 28, 4, 128, 3, 2, [1], 0, "bf16", seed=8),
    # statistics split into 2 per block, merged inside the column-sum kernel
    "split_span_bf16_gqa7": lambda: W.custom(1, 28, 4, 128, 19, 1100, [300], 4, "bf16", n_sinks=3,
                                             seed=9),
    # 640 x 7 = 4,480 pairs per KV head: statistics split and merged by their own kernel
    "long_span_bf16_gqa7": lambda: W.custom(1, 28, 4, 128, 640, 2000, [600, 600], 16, "bf16",
                                            n_relevant=1, seed=10),
    # 8 span rows over 17k keys: 33 statistics splits per block, more than the
    # column sums rebuild, so the statistics kernel merges them
    "short_span_long_context": lambda: W.custom(1, 28, 4, 128, 8, 512, [1024] * 16, 16, "bf16",
                                                n_relevant=2, seed=12),
}


class Layer:
    def __init__(self, w, li):
        self.np = w.layer(li, fresh=False)
        self.k, self.v, self.q = (to_dev(self.np[x]) for x in ("k", "v", "q"))
        self.kv = api.kv_desc(self.k, self.v, w.n_q_heads)


def score_one(w, L, norm, row_lse_in=None, s_acc=None, a_acc=None, accumulate=False):
    nv = w.n_vis
    f32 = dict(dtype=torch.float32, device=DEV)
    out = {"a": torch.zeros(nv, **f32), "v": torch.zeros(nv, **f32),
           "lse": torch.zeros((w.n_q, w.n_q_heads), **f32),
           "s_acc": s_acc if s_acc is not None else torch.zeros(nv, **f32),
           "a_acc": a_acc if a_acc is not None else torch.zeros(nv, **f32)}
    img = api.ImageTable(w.img_pos, w.img_off)
    api.conduit_score(L.kv, L.q, w.q_pos0, img, out["s_acc"], out["a_acc"], accumulate=accumulate,
                      norm=norm, row_lse_in=row_lse_in, row_lse_out=out["lse"], a_out=out["a"],
                      vnorm_out=out["v"])
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("norm", [O.NORM_CAUSAL_ROW, O.NORM_VISUAL_ONLY], ids=["causal", "visual"])
@pytest.mark.parametrize("case", sorted(CASES))
def test_score_matches_oracle(case, norm):
    w = CASES[case]()
    L = Layer(w, 0)
    got = score_one(w, L, norm)
    a, v, lse = O.score_layer(L.np["q"], L.np["k"], L.np["v"], w.q_pos0, w.img_pos, w.img_off,
                              norm=norm)
    assert_scores(to_f64(got["a"]), a, what="a_t")
    assert_scores(to_f64(got["v"]), v, what="||V_t||")
    assert_scores(to_f64(got["lse"]), lse, what="row lse")
    assert_scores(to_f64(got["s_acc"]), a * v, what="s")
    assert_scores(to_f64(got["a_acc"]), a, what="A")


def test_score_16k_workload_full_size():
    """The 16-image, 16,384-visual-token layer in the benchmark's launch shape."""
    w = W.config(4)
    L = Layer(w, 0)
    got = score_one(w, L, O.NORM_CAUSAL_ROW)
    a, v, lse = O.score_layer(L.np["q"], L.np["k"], L.np["v"], w.q_pos0, w.img_pos, w.img_off)
    assert_scores(to_f64(got["a"]), a, what="a_t")
    assert_scores(to_f64(got["v"]), v, what="||V_t||")
    assert_scores(to_f64(got["lse"]), lse, what="row lse")
    assert_scores(to_f64(got["s_acc"]), a * v, what="s")


@pytest.mark.parametrize("norm", [O.NORM_CAUSAL_ROW, O.NORM_VISUAL_ONLY], ids=["causal", "visual"])
def test_row_lse_in_skips_statistics(norm):
    w = CASES["ragged_bf16_gqa7"]()
    L = Layer(w, 0)
    a, v, lse = O.score_layer(L.np["q"], L.np["k"], L.np["v"], w.q_pos0, w.img_pos, w.img_off,
                              norm=norm)
    lse_in = torch.from_numpy(lse.astype(np.float32)).to(DEV)
    got = score_one(w, L, norm, row_lse_in=lse_in)
    assert_scores(to_f64(got["a"]), a, what="a_t (oracle lse in)")
    np.testing.assert_array_equal(bits(got["lse"]), bits(lse_in))
    own = score_one(w, L, norm)
    again = score_one(w, L, norm, row_lse_in=own["lse"])
    assert_scores(to_f64(again["a"]), a, what="a_t (own lse in)")


def test_layers_accumulate_in_order():
    w = W.custom(3, 28, 4, 128, 12, 9, [64, 130, 77], 4, "bf16", n_relevant=1, seed=11)
    layers = [Layer(w, li) for li in range(3)]
    s_acc = torch.full((w.n_vis,), float("nan"), device=DEV)
    a_acc = torch.full((w.n_vis,), float("nan"), device=DEV)
    a_l, v_l = [], []
    for li, L in enumerate(layers):
        score_one(w, L, O.NORM_CAUSAL_ROW, s_acc=s_acc, a_acc=a_acc, accumulate=li > 0)
        a, v, _ = O.score_layer(L.np["q"], L.np["k"], L.np["v"], w.q_pos0, w.img_pos, w.img_off)
        a_l.append(a)
        v_l.append(v)
    s, A = O.aggregate_layers(a_l, v_l)
    assert_scores(to_f64(s_acc), s * 3, what="sum of a v over layers")
    assert_scores(to_f64(a_acc), A, what="sum of a over layers")


def test_score_is_deterministic():
    w = W.config(2)
    L = Layer(w, 0)
    r1 = score_one(w, L, O.NORM_CAUSAL_ROW)
    r2 = score_one(w, L, O.NORM_CAUSAL_ROW)
    for key in r1:
        np.testing.assert_array_equal(bits(r1[key]), bits(r2[key]))


def test_strided_cache_rows():
    """Cache rows with a token stride wider than one row (e.g. a paged or
    fused K/V buffer) give the same result as dense rows."""
    w = CASES["ragged_bf16_gqa7"]()
    L = Layer(w, 0)
    n_ctx, hkv, d = L.k.shape
    big_k = torch.zeros((n_ctx, hkv + 2, d), dtype=L.k.dtype, device=DEV)
    big_v = torch.zeros_like(big_k)
    big_k[:, :hkv] = L.k
    big_v[:, 1:hkv + 1] = L.v
    L.kv = api.kv_desc(big_k[:, :hkv], big_v[:, 1:hkv + 1], w.n_q_heads)
    got = score_one(w, L, O.NORM_CAUSAL_ROW)
    a, v, _ = O.score_layer(L.np["q"], L.np["k"], L.np["v"], w.q_pos0, w.img_pos, w.img_off)
    assert_scores(to_f64(got["a"]), a, what="a_t")
    assert_scores(to_f64(got["v"]), v, what="||V_t||")


def test_statistics_merge_needs_no_clean_workspace():
    """The statistics kernel's merge marks carry the call's epoch: a
    workspace full of arbitrary bytes, and the same workspace again on the
    next call, give the same bits as a fresh one."""
    w = CASES["short_span_long_context"]()
    L = Layer(w, 0)
    img = api.ImageTable(w.img_pos, w.img_off)
    n = api.score_workspace_bytes(L.kv, w.n_q, img)
    f32 = dict(dtype=torch.float32, device=DEV)
    outs = []
    for fill in ("zeros", "random", "reuse"):
        if fill == "zeros":
            ws = torch.zeros(n, dtype=torch.uint8, device=DEV)
        elif fill == "random":
            ws = torch.randint(0, 256, (n,), dtype=torch.uint8, device=DEV,
                               generator=torch.Generator(device=DEV).manual_seed(5))
        s_acc, a_acc = torch.zeros(w.n_vis, **f32), torch.zeros(w.n_vis, **f32)
        lse = torch.zeros((w.n_q, w.n_q_heads), **f32)
        api.conduit_score(L.kv, L.q, w.q_pos0, img, s_acc, a_acc, row_lse_out=lse, ws=ws)
        torch.cuda.synchronize()
        outs.append((s_acc, a_acc, lse))
    for got in outs[1:]:
        for x, y in zip(got, outs[0]):
            np.testing.assert_array_equal(bits(x), bits(y))
    a, v, lse = O.score_layer(L.np["q"], L.np["k"], L.np["v"], w.q_pos0, w.img_pos, w.img_off)
    assert_scores(to_f64(outs[0][2]), lse, what="row lse")
    assert_scores(to_f64(outs[0][0]), a * v, what="s")


@pytest.mark.parametrize("boost", [400.0, 1200.0], ids=["gap_56_log2", "gap_170_log2"])
def test_visual_only_statistics_far_below_a_text_key(boost):
    """The first token (a text key) out-scores the visual keys by a median
    of 56 or 170 log2 units: with visual-only normalisation its probability
    is left out, and the visual keys' log-sum-exp and column sums must not
    lose precision to it; with causal-row normalisation it dominates.  Some
    rows' visual keys out-score it instead, by up to 54 log2 units.  Checked
    against the oracle for both normalisations."""
    w = W.custom(1, 28, 4, 128, 16, 64, [512, 512, 512], 16, "bf16", seed=14)
    L = Layer(w, 0)
    q = O.to_f64(L.np["q"])  # [n_q, H_q, d]
    G = w.n_q_heads // w.n_kv_heads
    k0 = O.to_f64(L.np["k"]).copy()
    for h in range(w.n_kv_heads):
        u = q[:, h * G:(h + 1) * G].reshape(-1, w.head_dim).mean(axis=0)
        u /= np.linalg.norm(u)
        # logit of the first token ~ boost * |q| * scale above the rest
        k0[0, h] = boost * u
    L.np["k"] = w._cast(k0.astype(np.float32))
    L.k = to_dev(L.np["k"])
    L.kv = api.kv_desc(L.k, L.v, w.n_q_heads)
    for norm in (O.NORM_VISUAL_ONLY, O.NORM_CAUSAL_ROW):
        got = score_one(w, L, norm)
        a, v, lse = O.score_layer(L.np["q"], L.np["k"], L.np["v"], w.q_pos0, w.img_pos, w.img_off, norm=norm)
        assert_scores(to_f64(got["a"]), a, what=f"a_t norm {norm}")
        assert_scores(to_f64(got["lse"]), lse, what=f"row lse norm {norm}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_q,hkv,g,images", [(1, 1, 1, [1]), (9, 2, 7, [255]), (64, 1, 1, [256]), (13, 2, 5, [200, 57]),
                                              (32, 1, 4, [511, 2]), (43, 4, 3, [1000] * 3), (65, 2, 7, [2049]),
                                              (200, 2, 7, [2049]),
                                              (7, 8, 7, [16384]), (43, 8, 3, [9000, 7500]), (90, 8, 7, [20000])])
def test_score_tile_pipeline(d, n_q, hkv, g, images):
    """Row counts around whole 64-row tiles (one tile, odd, even, ragged), key counts around whole 256-key
    workgroups, and launches below and above 512 workgroups (one 8-wave or two 4-wave workgroups per CU): scores of
    both aggregations against float64.  Products of bf16 inputs are exact; the fp32 sums of d of them and the
    exponent's fp32 argument (below 64) leave less than 1e-4 relative."""
    gen = torch.Generator(device=DEV).manual_seed(n_q * 17 + d)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV).to(torch.bfloat16)
    img_pos, img_off, at = [], [0], 5
    for n in images:
        img_pos.append(at)
        img_off.append(img_off[-1] + n)
        at += n + 3
    n_vis, q_pos0, n_ctx = img_off[-1], at, at + n_q
    k, v, q = rnd(n_ctx, hkv, d), rnd(n_ctx, hkv, d), rnd(n_q, hkv * g, d)
    img = api.ImageTable(np.array(img_pos, np.int32), np.array(img_off, np.int32))
    vis = torch.cat([torch.arange(p, p + n, device=DEV) for p, n in zip(img_pos, images)])
    ref = torch.zeros(2, n_vis, dtype=torch.float64, device=DEV)
    hidden = torch.arange(n_ctx, device=DEV)[None] > q_pos0 + torch.arange(n_q, device=DEV)[:, None]
    for h in range(hkv):
        for j in range(g):
            z = q[:, h * g + j].double() @ k[:, h].double().t() / d ** 0.5
            alpha = torch.softmax(z.masked_fill(hidden, -torch.inf), dim=1)[:, vis]
            ref += torch.stack([alpha.sum(0), (alpha ** 2).sum(0)])
    ref /= n_q * hkv * g
    ref[1].sqrt_()
    vnorm = v[vis].double().flatten(1).norm(dim=1)
    for r, agg in enumerate((api.AGG_MEAN, api.AGG_RMS)):
        s, a, a_out = (torch.full((n_vis,), 7.0, device=DEV) for _ in range(3))
        api.conduit_score(api.kv_desc(k, v, hkv * g), q, q_pos0, img, s, a, a_out=a_out, agg=agg)
        assert float((a.double() / ref[r] - 1).abs().max()) < 1e-4
        assert float((s.double() / (ref[r] * vnorm) - 1).abs().max()) < 1e-4
        assert torch.equal(a, a_out)


def _jump_layer(gen, d, n_q, hkv, g, n_ctx):
    """Keys and queries ~ N(0, 1) with every fourth 64-key tile holding one key, in its first or its second half,
    that most rows score 30 to 50 nats above the rest, more from tile to tile."""
    b = torch.nn.functional.normalize(torch.randn(hkv, d, generator=gen, device=DEV), dim=1)
    k = torch.randn(n_ctx, hkv, d, generator=gen, device=DEV)
    jump = torch.arange(3 * 64, n_ctx - n_q, 4 * 64, device=DEV)
    jump += torch.where(torch.arange(len(jump), device=DEV) % 2 == 0, 40, 5)
    amp = torch.linspace(30.0, 50.0, len(jump), device=DEV)
    k[jump] = 0.5 * d ** 0.5 * amp[:, None, None] * b
    q = torch.randn(n_q, hkv * g, d, generator=gen, device=DEV) + 2.0 * b.repeat_interleave(g, 0)
    v = torch.randn(n_ctx, hkv, d, generator=gen, device=DEV)
    return tuple(x.to(torch.bfloat16) for x in (k, v, q))


def _score64(k, v, q, q_pos0, vis):
    """Causal-row a_t, a_t ||V_t|| and the row log-sum-exps of one layer in float64; and the rows' largest logit less
    that of their first 64 keys."""
    (n_q, hq, d), hkv = q.shape, k.shape[1]
    hidden = torch.arange(len(k), device=DEV)[None] > q_pos0 + torch.arange(n_q, device=DEV)[:, None]
    a = torch.zeros(len(vis), dtype=torch.float64, device=DEV)
    lse, gap = (torch.zeros(n_q, hq, dtype=torch.float64, device=DEV) for _ in range(2))
    for h in range(hq):
        z = (q[:, h].double() @ k[:, h // (hq // hkv)].double().t() / d ** 0.5).masked_fill(hidden, -torch.inf)
        lse[:, h] = torch.logsumexp(z, dim=1)
        gap[:, h] = z.amax(1) - z[:, :64].amax(1)
        a += torch.softmax(z, dim=1)[:, vis].sum(0) / (n_q * hq)
    return a, a * v[vis].double().flatten(1).norm(dim=1), lse, gap


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_q,hkv,g,n_vis,layers", [(12, 1, 4, 300, 1), (33, 2, 7, 2500, 1), (20, 8, 2, 16500, 1),
                                                    (33, 2, 7, 2500, 3), (40, 4, 3, 4200, 9)])
def test_score_late_keys_far_above_the_first(d, n_q, hkv, g, n_vis, layers):
    """Keys in later tiles of every split of the statistics out-score the split's first ones by more than the 32 log2
    units that a fixed reference maximum bears: those items are done again with an online maximum, once.  One split,
    several, more than the column sums merge; below and above 512 column-sum workgroups; one layer and several.
    Logits stay below 210 log2 units, so that the fp32 exponent and the fp32 sums of d exact products err by less
    than 5e-5: 1e-4 relative is asked for."""
    gen = torch.Generator(device=DEV).manual_seed(n_vis + d + layers)
    q_pos0, n_ctx = 7 + n_vis, 7 + n_vis + n_q
    L = [_jump_layer(gen, d, n_q, hkv, g, n_ctx) for _ in range(layers)]
    vis = torch.arange(5, 5 + n_vis, device=DEV)
    img = api.ImageTable(np.array([5], np.int32), np.array([0, n_vis], np.int32))
    ref = [_score64(k, v, q, q_pos0, vis) for k, v, q in L]
    assert float((ref[0][3] > 23.0).double().mean()) > 0.25
    kvs, qs = [api.kv_desc(k, v, hkv * g) for k, v, _ in L], [q for _, _, q in L]
    s, a = (torch.full((n_vis,), 7.0, device=DEV) for _ in range(2))
    if layers > 1:
        api.conduit_score_layers(kvs, qs, q_pos0, img, s, a)
    else:
        lse = torch.zeros(n_q, hkv * g, device=DEV)
        api.conduit_score(kvs[0], qs[0], q_pos0, img, s, a, row_lse_out=lse)
        assert float((lse.double() / ref[0][2] - 1).abs().max()) < 1e-4
    assert float((a.double() / sum(r[0] for r in ref) - 1).abs().max()) < 1e-4
    assert float((s.double() / sum(r[1] for r in ref) - 1).abs().max()) < 1e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n_q,hkv,g,n_vis", [(33, 2, 7, 2500), (20, 8, 2, 16500)])
def test_score_with_a_nan_query_row(d, n_q, hkv, g, n_vis):
    """A NaN in one row's query: the call returns, that row's log-sum-exp is NaN and the other rows' are theirs."""
    gen = torch.Generator(device=DEV).manual_seed(n_vis + d)
    q_pos0, n_ctx = 7 + n_vis, 7 + n_vis + n_q
    k, v, q = _jump_layer(gen, d, n_q, hkv, g, n_ctx)
    vis = torch.arange(5, 5 + n_vis, device=DEV)
    ref = _score64(k, v, q, q_pos0, vis)[2]
    q[n_q // 2, 1, 3] = torch.nan
    s, a = (torch.zeros(n_vis, device=DEV) for _ in range(2))
    lse = torch.zeros(n_q, hkv * g, device=DEV)
    api.conduit_score(api.kv_desc(k, v, hkv * g), q, q_pos0,
                      api.ImageTable(np.array([5], np.int32), np.array([0, n_vis], np.int32)), s, a, row_lse_out=lse)
    bad = torch.zeros(n_q, hkv * g, dtype=torch.bool, device=DEV)
    bad[n_q // 2, 1] = True
    assert torch.equal(torch.isnan(lse), bad)
    assert float((lse.double() / ref - 1)[~bad].abs().max()) < 1e-4
