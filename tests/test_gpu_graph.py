"""The refresh step captured in a HIP graph: every replay, with eager steps
run between the replays, reproduces the eager outputs bit for bit (no call on
the path records anything a replay would not repeat)."""
import numpy as np
import pytest
import torch

from paper_2609_05821_amd import api, workloads as W
from tests.gpu_helpers import DEV, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [2, 4])
def test_graph_replays_equal_eager(cfg):
    w = W.config(cfg)
    L = w.layer(0)
    kc, vc, q = to_dev(L["k"]), to_dev(L["v"]), to_dev(L["q"])
    k_pristine, v_pristine = kc.clone(), vc.clone()
    img = api.ImageTable(w.img_pos, w.img_off)
    k = list(w.budgets.values())[0]
    step = api.RefreshStep([{"k": kc, "v": vc, "q": q}], w.n_q_heads, w.q_pos0, img, k, lam=1.0,
                           device=DEV)
    kv = step.kvs[0]
    step.score_and_select()
    torch.cuda.synchronize()
    idx = step.idx[:k].cpu().numpy()
    k_new, v_new = to_dev(np.ascontiguousarray(L["k_star"][idx])), to_dev(np.ascontiguousarray(L["v_star"][idx]))
    q_sel = to_dev(np.ascontiguousarray(L["q_star"][idx]))
    pos, out, lse = step.pos[:k], step.out[0][:k], step.lse[0][:k]

    def one_step():
        api.conduit_score(kv, q, w.q_pos0, img, step.s_acc, step.a_acc, ws=step.ws_score)
        api.conduit_select_topk(step.s_acc, step.a_acc, 1, img, 1.0, k, step.idx, step.pos,
                                mask_out=step.mask, shat_out=step.shat, c_out=step.c)
        api.conduit_scatter_kv(kv, pos, k_new, v_new)
        api.conduit_refresh_attn(kv, q_sel, pos, out, lse_out=lse, ws=step.ws_refresh)

    def restore():
        kc.copy_(k_pristine)
        vc.copy_(v_pristine)

    one_step()
    torch.cuda.synchronize()
    ref = [t.clone() for t in (out, lse, step.idx, step.mask, step.shat, kc, vc)]
    restore()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        one_step()
    torch.cuda.synchronize()
    for _ in range(3):
        restore()
        graph.replay()
        torch.cuda.synchronize()
        got = (out, lse, step.idx, step.mask, step.shat, kc, vc)
        for name, a, b in zip(("out", "lse", "idx", "mask", "shat", "k", "v"), got, ref):
            assert torch.equal(a, b), name
        restore()
        one_step()  # eager work between replays
        torch.cuda.synchronize()


@pytest.mark.parametrize("n_q,hkv,g,d,n_vis,layers", [(20, 8, 2, 64, 16500, 1), (8, 4, 7, 128, 16384, 1),
                                                      (40, 4, 3, 128, 4200, 9), (24, 4, 2, 64, 2000, 18)])
def test_graph_replays_of_merging_statistics(n_q, hkv, g, d, n_vis, layers):
    """Scoring whose statistics kernel merges its own split rows (512 or more column-sum workgroups, more splits than
    the column sums merge, several launches of layers), captured and replayed back to back on new keys and queries
    with nothing else on its workspace: each replay gives the eager call's bits, and the merge marks, the last part
    of the workspace, are unset again after it."""
    gen = torch.Generator(device=DEV).manual_seed(n_vis + layers)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV).to(torch.bfloat16)
    q_pos0, n_ctx = 7 + n_vis, 7 + n_vis + n_q
    L = [(rnd(n_ctx, hkv, d), rnd(n_ctx, hkv, d), rnd(n_q, hkv * g, d)) for _ in range(layers)]
    kvs, qs = [api.kv_desc(k, v, hkv * g) for k, v, _ in L], [q for _, _, q in L]
    img = api.ImageTable(np.array([5], np.int32), np.array([0, n_vis], np.int32))
    lse = torch.zeros(n_q, hkv * g, device=DEV)
    s, a = (torch.zeros(n_vis, device=DEV) for _ in range(2))
    need = (api.score_workspace_bytes(kvs[0], n_q, img) if layers == 1
            else api.score_layers_workspace_bytes(kvs[0], n_q, img, layers))
    ws, ws_eager = (torch.full((need // 4,), 0x5a5a5a5a, dtype=torch.int32, device=DEV) for _ in range(2))

    def score(w):
        if layers == 1:
            api.conduit_score(kvs[0], qs[0], q_pos0, img, s, a, row_lse_out=lse, ws=w)
        else:
            api.conduit_score_layers(kvs, qs, q_pos0, img, s, a, ws=w)

    score(ws_eager)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        score(ws)
    for _ in range(4):
        for k, _, q in L:
            k.copy_(rnd(*k.shape))
            q.copy_(rnd(*q.shape))
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in (lse, s, a)]
        tail = ws.cpu().numpy()
        tail = tail[:np.flatnonzero(tail != 0x5a5a5a5a)[-1] + 1]  # less the alignment of its end
        assert need // 4 - len(tail) < 64
        assert not tail[-512 * min(layers, 16):].any()  # at least 512 slots per layer of a launch
        score(ws_eager)
        torch.cuda.synchronize()
        for x, y in zip(got, (lse, s, a)):
            assert torch.equal(x, y)
