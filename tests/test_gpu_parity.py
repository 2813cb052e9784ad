"""GPU parity: every C-ABI call against the CPU oracle on the same seeded inputs (run with -m gpu)."""
import math

import numpy as np
import pytest
import torch

from oracle import omni_oracle as oc
from paper_2511_12201_amd import binding as ob
from paper_2511_12201_amd import synth
from tests.helpers import (GRAD_RSS, bf16_ulp, check_selection_on_gpu_scores, grad_bar, lists_to_padded, oracle_train, padded_to_lists,
                           to_device, to_host)

pytestmark = pytest.mark.gpu

TOL_OUT = {"f32": 1e-4, "bf16": 2e-2}          # max-abs bar for attention outputs and gradients

# shapes: several 128-row query tiles and 64-key tiles with ragged tails, all dtype / head_dim variants
CFG_BF16 = synth.C2_16K.scaled(name="bf16_d128", frames=7, tok_per_frame=252, n_text=95, n_q_heads=8, n_kv_heads=2)
CFG_BF16_64 = synth.C2_16K.scaled(name="bf16_d64", frames=5, tok_per_frame=100, n_text=37, n_q_heads=4, n_kv_heads=2,
                                  head_dim=64, seed=11)
CFG_F32 = synth.C1_TINY
CFG_F32_128 = synth.C1_TINY.scaled(name="f32_d128", head_dim=128, frames=3, tok_per_frame=150, n_text=29,
                                   n_q_heads=4, n_kv_heads=2, seed=12)
ALL_CFGS = [CFG_BF16, CFG_BF16_64, CFG_F32, CFG_F32_128]


class Case:
    """Inputs on host and device plus the oracle's results for one configuration (cached per test session)."""
    _cache = {}

    def __init__(self, cfg, tau=0.08, recall_p=0.95, probe_block=256, q_mode=0, q_param=0.08):
        self.cfg = cfg
        L = synth.make_layer(cfg)
        self.Q, self.K, self.V = L["Q"], L["K"], L["V"]
        self.side = L["side"]
        self.dQ, self.dK, self.dV = (to_device(x, cfg.dtype) for x in (self.Q, self.K, self.V))
        self.desc = ob.make_layer_desc(self.dQ, self.dK, cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
        self.recall_p, self.probe_block, self.q_mode, self.q_param = recall_p, probe_block, q_mode, q_param
        # oracle pipeline
        self.o_probe = oc.probe_keys(self.K, cfg.vis_begin, cfg.vis_end, cfg.sink_index)
        self.o_scores = oc.score_queries(self.Q, self.o_probe, cfg.scale)
        self.o_scores32 = self.o_scores.astype(np.float32)
        self.o_qidx = oc.select_queries(self.o_scores32, q_mode, q_param, cfg.vis_begin, cfg.vis_end)
        self.o_a = oc.pooled_key_scores(self.Q, self.K, probe_block, cfg.causal, cfg.scale)
        self.o_a32 = self.o_a.astype(np.float32)
        self.o_bud = oc.kv_budget(self.o_a32, recall_p, 0)
        self.o_kvidx = oc.select_kv(self.o_a32, self.o_bud["budget"])

    @classmethod
    def get(cls, cfg, **kw):
        key = (cfg, tuple(sorted(kw.items())))
        if key not in cls._cache:
            cls._cache[key] = cls(cfg, **kw)
        return cls._cache[key]


def case_for(cfg):
    if cfg.structured:
        return Case.get(cfg)
    return Case.get(cfg, q_mode=1, q_param=0.25, probe_block=64)


# ------------------------------------------------------------------ query scoring and selection

@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
def test_score_queries(cfg):
    c = case_for(cfg)
    probe, scores = ob.omni_score_queries(c.desc, c.dQ, c.dK)
    torch.cuda.synchronize()
    np.testing.assert_allclose(to_host(probe), c.o_probe, rtol=2e-5, atol=2e-5)
    np.testing.assert_allclose(to_host(scores), c.o_scores, rtol=0, atol=1e-5)


@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
@pytest.mark.parametrize("mode,param", [(0, 0.08), (0, 0.5), (1, 0.25), (1, 1.0), (0, -1.0), (0, 2.0)])
def test_select_queries_is_bit_exact_on_given_scores(cfg, mode, param):
    c = case_for(cfg)
    scores = torch.from_numpy(c.o_scores32).cuda()
    q_idx, q_cnt = ob.omni_select_queries(c.desc, scores, mode, param)
    torch.cuda.synchronize()
    want = oc.select_queries(c.o_scores32, mode, param, cfg.vis_begin, cfg.vis_end)
    got = padded_to_lists(q_idx, q_cnt)
    for b in range(cfg.batch):
        for h in range(cfg.n_q_heads):
            np.testing.assert_array_equal(got[b][h], want[b][h], err_msg=f"batch {b} head {h}")


def test_select_queries_with_tied_scores():
    cfg = CFG_BF16_64
    c = case_for(cfg)
    rng = np.random.default_rng(5)
    tied = (rng.integers(0, 6, c.o_scores32.shape) / 8.0).astype(np.float32)      # heavy ties, includes 0.0
    scores = torch.from_numpy(tied).cuda()
    for mode, param in [(1, 0.3), (1, 0.01), (0, 0.25)]:
        q_idx, q_cnt = ob.omni_select_queries(c.desc, scores, mode, param)
        torch.cuda.synchronize()
        want = oc.select_queries(tied, mode, param, cfg.vis_begin, cfg.vis_end)
        got = padded_to_lists(q_idx, q_cnt)
        for h in range(cfg.n_q_heads):
            np.testing.assert_array_equal(got[0][h], want[0][h])


# ------------------------------------------------------------------ key scores, budget, KV selection

@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
def test_kv_budget_key_scores_and_statistics(cfg):
    c = case_for(cfg)
    r = ob.omni_kv_budget(c.desc, c.dQ, c.dK, c.recall_p, c.probe_block, 0)
    torch.cuda.synchronize()
    a = to_host(r.key_scores).astype(np.float64)
    amax = c.o_a.max()
    np.testing.assert_allclose(a, c.o_a, rtol=0, atol=1e-4 * amax)
    np.testing.assert_allclose(a.sum(-1), cfg.n_tokens, rtol=1e-5)
    np.testing.assert_allclose(to_host(r.kurtosis), c.o_bud["kurtosis"], rtol=1e-3)
    k_sorted = np.sort(c.o_bud["kurtosis"], axis=-1)
    if np.all((k_sorted[:, 1] - k_sorted[:, 0]) > 1e-3 * np.abs(k_sorted[:, 0])):
        np.testing.assert_array_equal(to_host(r.flattest), c.o_bud["flattest"])
        # budget: minimal under the oracle's own score array up to the probe's numeric error
        for b in range(cfg.batch):
            srt = np.sort(c.o_a32[b, c.o_bud["flattest"][b]].astype(np.float64))[::-1]
            cum = np.cumsum(srt)
            target = float(np.float32(c.recall_p)) * cfg.n_tokens
            bb = int(to_host(r.budget)[b])
            assert cum[bb - 1] >= target * (1 - 1e-4)
            assert bb == 1 or cum[bb - 2] < target * (1 + 1e-4)
    np.testing.assert_allclose(to_host(r.recall), c.o_bud["recall"], atol=2e-4)


@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
@pytest.mark.parametrize("p,mode", [(0.95, 0), (0.5, 0), (0.82, 1), (1.0, 0)])
def test_budget_from_given_scores_is_exact(cfg, p, mode):
    c = case_for(cfg)
    a = torch.from_numpy(c.o_a32).cuda()
    r = ob.omni_budget_from_scores(c.desc, a, p, mode)
    torch.cuda.synchronize()
    want = oc.kv_budget(c.o_a32, p, mode)
    np.testing.assert_allclose(to_host(r.kurtosis), want["kurtosis"], rtol=1e-9)
    np.testing.assert_array_equal(to_host(r.flattest), want["flattest"])
    np.testing.assert_array_equal(to_host(r.budget), want["budget"])
    np.testing.assert_allclose(to_host(r.recall), want["recall"], atol=1e-6)


@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
def test_select_kv_is_bit_exact_on_given_scores(cfg):
    c = case_for(cfg)
    a = torch.from_numpy(c.o_a32).cuda()
    N = cfg.n_tokens
    for budget in (int(c.o_bud["budget"][0]), 1, 63, N - 1, N):
        bud = torch.full((cfg.batch,), budget, dtype=torch.int32, device="cuda")
        kv_idx = ob.omni_select_kv(c.desc, a, bud, N)
        torch.cuda.synchronize()
        want = oc.select_kv(c.o_a32, [budget] * cfg.batch)
        got = to_host(kv_idx)
        for b in range(cfg.batch):
            np.testing.assert_array_equal(got[b, :, :budget], want[b], err_msg=f"budget {budget}")


def test_select_kv_ties_and_capacity_clamp():
    cfg = CFG_BF16_64
    c = case_for(cfg)
    rng = np.random.default_rng(6)
    a_np = (rng.integers(0, 4, c.o_a32.shape) / 4.0).astype(np.float32)
    a = torch.from_numpy(a_np).cuda()
    bud = torch.full((cfg.batch,), 200, dtype=torch.int32, device="cuda")
    got = to_host(ob.omni_select_kv(c.desc, a, bud, 256))
    want = oc.select_kv(a_np, [200])
    np.testing.assert_array_equal(got[0, :, :200], want[0])
    # capacity below the budget: the effective budget is b_cap
    got = to_host(ob.omni_select_kv(c.desc, a, bud, 96))
    want = oc.select_kv(a_np, [96])
    np.testing.assert_array_equal(got[0], want[0])


# ------------------------------------------------------------------ attention forward

def _run_sparse_fwd(c, q_lists, kv_lists):
    cfg = c.cfg
    N = cfg.n_tokens
    q_idx, q_cnt = lists_to_padded(q_lists, cfg.n_q_heads, N)
    b = max(len(x) for x in kv_lists[0])
    kv_idx, _ = lists_to_padded(kv_lists, cfg.n_q_heads, b)
    budget = torch.tensor([len(kv_lists[bb][0]) for bb in range(cfg.batch)], dtype=torch.int32, device="cuda")
    O, lse = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, kv_idx, budget, b)
    torch.cuda.synchronize()
    return to_host(O), to_host(lse)


def _check_fwd(c, O, lse, Oo, Lo):
    tol = TOL_OUT[c.cfg.dtype]
    assert np.max(np.abs(O - Oo)) <= tol
    fin = np.isfinite(Lo)
    np.testing.assert_array_equal(np.isfinite(lse), fin)
    assert np.all(lse[~fin] == -np.inf)
    assert np.max(np.abs(lse[fin] - Lo[fin])) <= (1e-4 if c.cfg.dtype == "f32" else 2e-3)
    assert np.all(O[~fin] == 0)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
def test_sparse_attn_fwd_on_oracle_selection(cfg):
    c = case_for(cfg)
    kv_lists = [list(c.o_kvidx[b]) for b in range(cfg.batch)]
    O, lse = _run_sparse_fwd(c, c.o_qidx, kv_lists)
    Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, c.o_qidx, kv_lists, cfg.causal, cfg.scale)
    _check_fwd(c, O, lse, Oo, Lo)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", [CFG_BF16, CFG_F32], ids=lambda c: c.name)
def test_sparse_attn_fwd_edge_sets(cfg):
    """Tiny budgets, a head with no kept query past the first keys, a head whose queries precede all its keys."""
    c = case_for(cfg)
    N, H = cfg.n_tokens, cfg.n_q_heads
    rng = np.random.default_rng(9)
    q_lists = [[np.arange(N, dtype=np.int32)] + [np.sort(rng.choice(N, int(rng.integers(1, 200)), replace=False)).astype(np.int32)
                                                for _ in range(H - 1)]]
    q_lists[0][1] = np.arange(0, 5, dtype=np.int32)                     # precedes every key of head 1
    for b_sel in (1, 65, 130):
        kv_lists = [[np.sort(rng.choice(np.arange(8, N), b_sel, replace=False)).astype(np.int32) for _ in range(H)]]
        O, lse = _run_sparse_fwd(c, q_lists, kv_lists)
        Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, q_lists, kv_lists, cfg.causal, cfg.scale)
        _check_fwd(c, O, lse, Oo, Lo)
        assert np.all(lse[0, 1] == -np.inf)


def _plain_bf16_layer(seed, N, H, Hkv, d):
    rng = np.random.default_rng(seed)
    mk = lambda *shape: synth.round_to_bf16(rng.standard_normal(shape).astype(np.float32))
    return mk(1, H, N, d), mk(1, Hkv, N, d), mk(1, Hkv, N, d)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("ramp", [3.0, 12.0, 40.0])
def test_forward_when_the_logits_keep_rising_along_the_key_list(ramp):
    """Keys whose logits grow with their index by up to `ramp` per 64-key tile in the exponent's base-2 units, and
    jump up and down around that trend: whatever value the kernel takes the weights of a row against early on is far
    too low later (by more than the f16 and, for the steepest ramp, the fp32 range), so the path that moves it and
    forms a tile's weights again has to run, many times per row.  Every query is kept, causal and not."""
    N, H, Hkv, d = 1536, 4, 2, 128
    Q, K, V = _plain_bf16_layer(77, N, H, Hkv, d)
    u = np.zeros(d, dtype=np.float32)
    u[:8] = 1.0
    scale = 1.0 / math.sqrt(d)
    # q.u = 8 a and k_n.u = 8 g(n) on top of the noise, u a unit step on 8 coordinates: logit trend 8 a g(n) scale nats
    a = 2.0
    rng = np.random.default_rng(78)
    g = (ramp * math.log(2.0) / 64.0) * np.arange(N) / (8 * a * scale) + rng.choice([0.0, 0.5, -0.5], N)
    Q = synth.round_to_bf16(Q * 0.25 + a * u)
    K = synth.round_to_bf16(K * 0.25 + g[None, None, :, None].astype(np.float32) * u)
    dQ, dK, dV = (to_device(x, "bf16") for x in (Q, K, V))
    full = [[np.arange(N, dtype=np.int32) for _ in range(H)]]
    q_idx, q_cnt = lists_to_padded(full, H, N)
    budget = torch.full((1,), N, dtype=torch.int32, device="cuda")
    for causal in (True, False):
        desc = ob.make_layer_desc(dQ, dK, 1, N - 8, 0, causal, scale)
        O, lse = ob.omni_sparse_attn_fwd(desc, dQ, dK, dV, q_idx, q_cnt, q_idx, budget, N)
        O2, lse2 = ob.omni_dense_attn_fwd(desc, dQ, dK, dV)
        torch.cuda.synchronize()
        Oo, Lo = oc.dense_attention(Q, K, V, causal, scale)
        for got_o, got_l in ((O, lse), (O2, lse2)):
            assert np.max(np.abs(to_host(got_o) - Oo)) <= TOL_OUT["bf16"]
            assert np.max(np.abs(to_host(got_l) - Lo)) <= 2e-3 * max(1.0, float(np.max(np.abs(Lo))) / 64)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("causal", [True, False])
def test_forward_returns_the_value_row_of_a_key_that_dominates(causal):
    """Every query's own key beats all others by more than 40 in the exponent: the softmax is one-hot to any working
    precision, so the output row is that key's V row -- bit for bit, whatever value the kernel takes the weights
    against and however it rounds them, because numerator and normaliser carry the same rounded weight."""
    N, H, Hkv, d = 1536, 4, 4, 128
    _, K, V = _plain_bf16_layer(55, N, H, Hkv, d)
    scale = 1.0 / math.sqrt(d)
    Q = synth.round_to_bf16(10.0 * K)                       # q_n . k_n scale ~ 113; q_n . k_m scale below 50
    S = np.einsum("hnd,hmd->hnm", Q[0].astype(np.float64), K[0].astype(np.float64)) * scale
    own = np.diagonal(S, axis1=1, axis2=2)
    off = S - 1e9 * np.eye(N)[None]
    if causal:
        off = np.where(np.tril(np.ones((N, N), bool))[None], off, -np.inf)
    assert np.min(own - off.max(-1)) > 40 * math.log(2.0) + 1          # the construction holds
    dQ, dK, dV = (to_device(x, "bf16") for x in (Q, K, V))
    desc = ob.make_layer_desc(dQ, dK, 1, N - 8, 0, causal, scale)
    O, lse = ob.omni_dense_attn_fwd(desc, dQ, dK, dV)
    full = [[np.arange(N, dtype=np.int32) for _ in range(H)]]
    q_idx, q_cnt = lists_to_padded(full, H, N)
    budget = torch.full((1,), N, dtype=torch.int32, device="cuda")
    O2, _ = ob.omni_sparse_attn_fwd(desc, dQ, dK, dV, q_idx, q_cnt, q_idx, budget, N)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(to_host(O), V)
    np.testing.assert_array_equal(to_host(O2), V)
    np.testing.assert_allclose(to_host(lse)[0], own, rtol=2e-6, atol=1e-4)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("vscale", [2.0 ** -12, 1.0, 2.0 ** 13])
def test_forward_value_range(vscale):
    """The second product runs in f16: V is converted exactly inside [2^-14, 65504].  Outputs follow V's scale with the
    same relative accuracy there; beyond it V saturates at 65504, which the last case pins against the oracle on the
    clamped values."""
    N, H, Hkv, d = 640, 4, 2, 64
    Q, K, V = _plain_bf16_layer(91, N, H, Hkv, d)
    V = synth.round_to_bf16(V * np.float32(vscale))
    scale = 1.0 / math.sqrt(d)
    dQ, dK = to_device(Q, "bf16"), to_device(K, "bf16")
    desc = ob.make_layer_desc(dQ, dK, 1, N - 8, 0, True, scale)
    O, _ = ob.omni_dense_attn_fwd(desc, dQ, dK, to_device(V, "bf16"))
    torch.cuda.synchronize()
    Oo, _ = oc.dense_attention(Q, K, V, True, scale)
    assert np.max(np.abs(to_host(O) - Oo)) <= TOL_OUT["bf16"] * vscale + 2e-7
    if vscale > 1:
        Vbig = V.copy()
        Vbig[0, :, 5::7, 3] = 3.0e5                     # beyond the f16 range: taken as 65504
        O, _ = ob.omni_dense_attn_fwd(desc, dQ, dK, to_device(Vbig, "bf16"))
        torch.cuda.synchronize()
        Oc, _ = oc.dense_attention(Q, K, np.minimum(Vbig, 65504.0), True, scale)
        got = to_host(O)
        assert np.all(np.isfinite(got))
        assert np.max(np.abs(got - Oc)) <= TOL_OUT["bf16"] * vscale + 2.0 ** -8 * 65504


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
@pytest.mark.parametrize("causal", [True, False])
def test_dense_attn_fwd_and_full_budget_sparse_equal_dense_definition(cfg, causal):
    c = case_for(cfg)
    desc = ob.make_layer_desc(c.dQ, c.dK, cfg.vis_begin, cfg.vis_end, cfg.sink_index, causal)
    O, lse = ob.omni_dense_attn_fwd(desc, c.dQ, c.dK, c.dV)
    torch.cuda.synchronize()
    Oo, Lo = oc.dense_attention(c.Q, c.K, c.V, causal, cfg.scale)
    tol = TOL_OUT[cfg.dtype]
    assert np.max(np.abs(to_host(O) - Oo)) <= tol
    assert np.max(np.abs(to_host(lse) - Lo)) <= (1e-4 if cfg.dtype == "f32" else 2e-3)
    # sparse call with every query kept and b = N is the same function
    N, H = cfg.n_tokens, cfg.n_q_heads
    full = [[np.arange(N, dtype=np.int32) for _ in range(H)] for _ in range(cfg.batch)]
    q_idx, q_cnt = lists_to_padded(full, H, N)
    budget = torch.full((cfg.batch,), N, dtype=torch.int32, device="cuda")
    O2, lse2 = ob.omni_sparse_attn_fwd(desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, q_idx, budget, N)
    torch.cuda.synchronize()
    assert np.max(np.abs(to_host(O2) - Oo)) <= tol


# ------------------------------------------------------------------ decode

def _decode_case(cfg, batch, n_ans=9):
    c = case_for(cfg)
    N = cfg.n_tokens
    cap = N + 16
    steps = synth.make_decode_steps(cfg, dict(side=c.side), n_ans + 1, batch=batch)
    Kc = np.zeros((batch, cfg.n_kv_heads, cap, cfg.head_dim), dtype=np.float32)
    Vc = np.zeros_like(Kc)
    for b in range(batch):
        Kc[b, :, :N], Vc[b, :, :N] = c.K[0], c.V[0]
        Kc[b, :, N:N + n_ans] = steps["k_new"][:n_ans, b].transpose(1, 0, 2)
        Vc[b, :, N:N + n_ans] = steps["v_new"][:n_ans, b].transpose(1, 0, 2)
    ctx = np.array([N + n_ans - (b % 3) for b in range(batch)], dtype=np.int32)
    q = steps["q"][n_ans]
    vis = oc.visual_subset([list(c.o_kvidx[0])] * batch, cfg.vis_begin, cfg.vis_end)
    probe = np.repeat(c.o_probe, batch, axis=0)
    return c, q, Kc, Vc, ctx, probe, vis


@pytest.mark.parametrize("cfg,batch", [(CFG_BF16, 1), (CFG_BF16, 3), (CFG_BF16_64, 2), (CFG_F32, 2), (CFG_F32_128, 1)],
                         ids=lambda x: getattr(x, "name", str(x)))
def test_slim_decode_and_dense_decode(cfg, batch):
    c, q, Kc, Vc, ctx, probe, vis = _decode_case(cfg, batch)
    tau = 0.08
    dq, dKc, dVc = (to_device(x, cfg.dtype) for x in (q, Kc, Vc))
    dctx = torch.from_numpy(ctx).cuda()
    b_cap = max(len(v) for per in vis for v in per)
    vis_idx, vis_cnt = lists_to_padded(vis, cfg.n_q_heads, b_cap)
    dprobe = torch.from_numpy(probe.astype(np.float32)).cuda()
    desc = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, tau)
    O, act = ob.omni_slim_decode(desc, dq, dKc, dVc, dctx, dprobe, vis_idx, vis_cnt, b_cap)
    torch.cuda.synchronize()
    Oo, acto, sc = oc.slim_decode(q, Kc, Vc, ctx, probe.astype(np.float32), vis, tau, cfg.vis_begin, cfg.vis_end, cfg.scale)
    act = to_host(act)
    clear = np.abs(sc - tau) > 1e-5          # heads whose score is not at the threshold must agree
    np.testing.assert_array_equal(act[clear], acto[clear])
    same = act == acto
    tol = TOL_OUT[cfg.dtype]
    assert np.max(np.abs(to_host(O)[same] - Oo[same])) <= tol
    assert 0 < acto.sum() and (not cfg.structured or acto.sum() < acto.size)
    Od = ob.omni_dense_decode(desc, dq, dKc, dVc, dctx)
    torch.cuda.synchronize()
    assert np.max(np.abs(to_host(Od) - oc.dense_decode(q, Kc, Vc, ctx, cfg.scale))) <= tol


@pytest.mark.parametrize("cfg,batch", [(CFG_BF16, 1), (CFG_BF16, 3), (CFG_BF16_64, 2), (CFG_F32, 2), (CFG_F32_128, 1)],
                         ids=lambda x: getattr(x, "name", str(x)))
def test_grouped_slim_decode(cfg, batch):
    """Group-union storage of the visual rows: the structure is the union of the per-head sets with the
    right membership bits, and the decode step on it gives the oracle's per-head result."""
    c, q, Kc, Vc, ctx, probe, vis = _decode_case(cfg, batch)
    tau = 0.08
    H, Hkv = cfg.n_q_heads, cfg.n_kv_heads
    G = H // Hkv
    b = len(c.o_kvidx[0][0])
    kv_idx, _ = lists_to_padded([list(c.o_kvidx[0])] * batch, H, b)
    budget = torch.full((batch,), b, dtype=torch.int32, device="cuda")
    ldesc = ob.make_layer_desc(c.dQ.expand(batch, -1, -1, -1).contiguous(), c.dK.expand(batch, -1, -1, -1).contiguous(),
                               cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
    grp_idx, grp_mask, grp_cnt = ob.omni_group_subset(ldesc, kv_idx, budget, b)
    torch.cuda.synchronize()
    gi, gm, gc = to_host(grp_idx), to_host(grp_mask).view(np.uint32), to_host(grp_cnt)
    for bb in range(batch):
        for g in range(Hkv):
            sets = [set(int(x) for x in vis[bb][g * G + j]) for j in range(G)]
            union = sorted(set().union(*sets))
            n = int(gc[bb, g])
            assert n == len(union)
            np.testing.assert_array_equal(gi[bb, g, :n], np.array(union, dtype=np.int32))
            want = np.array([sum((1 << j) for j in range(G) if t in sets[j]) for t in union], dtype=np.uint32)
            np.testing.assert_array_equal(gm[bb, g, :n], want)
    dq, dKc, dVc = (to_device(x, cfg.dtype) for x in (q, Kc, Vc))
    dctx = torch.from_numpy(ctx).cuda()
    dprobe = torch.from_numpy(probe.astype(np.float32)).cuda()
    desc = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, tau)
    O, act = ob.omni_slim_decode_grouped(desc, dq, dKc, dVc, dctx, dprobe, grp_idx, grp_mask, grp_cnt)
    torch.cuda.synchronize()
    Oo, acto, sc = oc.slim_decode(q, Kc, Vc, ctx, probe.astype(np.float32), vis, tau, cfg.vis_begin, cfg.vis_end, cfg.scale)
    act = to_host(act)
    clear = np.abs(sc - tau) > 1e-5
    np.testing.assert_array_equal(act[clear], acto[clear])
    same = act == acto
    assert np.max(np.abs(to_host(O)[same] - Oo[same])) <= TOL_OUT[cfg.dtype]


@pytest.mark.parametrize("cfg,batch", [(CFG_BF16, 1), (CFG_BF16, 3), (CFG_BF16_64, 2), (CFG_F32, 2)],
                         ids=lambda x: getattr(x, "name", str(x)))
def test_slim_decode_with_static_lists_reads_the_lists_merged_by_the_prepare_call(cfg, batch):
    """static_lists = 1: omni_slim_decode_prepare merges the per-head lists per KV group into the workspace and the
    decode calls that follow read them there.  Every call must give the bits of omni_slim_decode_grouped on the
    library's own group lists (and so the oracle's result), whatever the list arguments then hold; preparing again
    with other lists switches to those."""
    c, q, Kc, Vc, ctx, probe, vis = _decode_case(cfg, batch)
    tau = 0.08
    H = cfg.n_q_heads
    dq, dKc, dVc = (to_device(x, cfg.dtype) for x in (q, Kc, Vc))
    dctx = torch.from_numpy(ctx).cuda()
    dprobe = torch.from_numpy(probe.astype(np.float32)).cuda()
    b_cap = max(len(v) for per in vis for v in per)
    vis_idx, vis_cnt = lists_to_padded(vis, H, b_cap)
    desc = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, tau)
    sdesc = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, tau, static_lists=True)
    assert ob.workspace_bytes(ob.CALL_SLIM_DECODE, sdesc) > ob.workspace_bytes(ob.CALL_SLIM_DECODE, desc)
    view = torch.int16 if cfg.dtype == "bf16" else torch.int32

    def grouped_reference(lists):
        b = max(len(x) for per in lists for x in per)
        kv_idx, cnt = lists_to_padded(lists, H, b)
        ldesc = ob.make_layer_desc(c.dQ.expand(batch, -1, -1, -1).contiguous(), c.dK.expand(batch, -1, -1, -1).contiguous(),
                                   cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
        grp = ob.omni_group_subset_per_head(ldesc, kv_idx, cnt, b)
        return ob.omni_slim_decode_grouped(desc, dq, dKc, dVc, dctx, dprobe, *grp, ws=ob.Workspace())

    want_O, want_act = grouped_reference(vis)
    Oo, acto, sc = oc.slim_decode(q, Kc, Vc, ctx, probe.astype(np.float32), vis, tau, cfg.vis_begin, cfg.vis_end, cfg.scale)
    same = to_host(want_act) == acto
    assert np.max(np.abs(to_host(want_O)[same] - Oo[same])) <= TOL_OUT[cfg.dtype]
    ws = ob.Workspace()
    ws.get(ob.CALL_SLIM_DECODE, sdesc).fill_(0xFF)       # whatever the workspace held before
    ob.omni_slim_decode_prepare(sdesc, vis_idx, vis_cnt, b_cap, ws=ws)
    poison_idx, poison_cnt = torch.full_like(vis_idx, -7), torch.zeros_like(vis_cnt)
    for args in ((vis_idx, vis_cnt), (poison_idx, poison_cnt), (vis_idx, vis_cnt)):   # the decode calls read the workspace
        O, act = ob.omni_slim_decode(sdesc, dq, dKc, dVc, dctx, dprobe, *args, b_cap, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(O.view(view), want_O.view(view)) and torch.equal(act, want_act)
    # other lists: every second entry of every head
    thin = [[v[::2] for v in per] for per in vis]
    t_idx, t_cnt = lists_to_padded(thin, H, b_cap)
    want2_O, want2_act = grouped_reference(thin)
    ob.omni_slim_decode_prepare(sdesc, t_idx, t_cnt, b_cap, ws=ws)
    O, act = ob.omni_slim_decode(sdesc, dq, dKc, dVc, dctx, dprobe, t_idx, t_cnt, b_cap, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(O.view(view), want2_O.view(view)) and torch.equal(act, want2_act)
    assert not torch.equal(O.view(view), want_O.view(view))
    # the stateless call needs no preparation and gives the oracle's result too
    O0, act0 = ob.omni_slim_decode(desc, dq, dKc, dVc, dctx, dprobe, vis_idx, vis_cnt, b_cap, ws=ob.Workspace())
    torch.cuda.synchronize()
    assert np.max(np.abs(to_host(O0)[same] - Oo[same])) <= TOL_OUT[cfg.dtype]
    with pytest.raises(ob.OmniError):
        ob.omni_slim_decode_prepare(desc, vis_idx, vis_cnt, b_cap, ws=ws)      # not a static_lists descriptor


@pytest.mark.parametrize("cfg", [CFG_BF16, CFG_F32], ids=lambda c: c.name)
@pytest.mark.parametrize("case", ["all_lazy", "all_active", "empty_lists", "short_context", "one_row"])
def test_decode_degenerate_cases(cfg, case):
    """The decode step at its corners, on the per-head call (stateless and with static lists) and the group-list call:
    every head but head 0 lazy; every head active; heads that stored no visual row; a context that ends inside the
    visual range (listed rows at or beyond it do not exist yet); a context of one row."""
    batch = 2
    c, q, Kc, Vc, ctx, probe, vis = _decode_case(cfg, batch)
    H = cfg.n_q_heads
    tau = {"all_lazy": 0.9999, "all_active": -1.0}.get(case, 0.08)
    if case == "empty_lists":
        vis = [[v[:0] if (h % 3) else v for h, v in enumerate(per)] for per in vis]
        vis[1] = [v[:0] for v in vis[1]]                     # the second sequence stored nothing at all
    if case == "short_context":
        ctx = np.array([cfg.vis_begin + (cfg.vis_end - cfg.vis_begin) // 2, cfg.vis_begin + 3], dtype=np.int32)
    if case == "one_row":
        ctx = np.array([1, 1], dtype=np.int32)
    dq, dKc, dVc = (to_device(x, cfg.dtype) for x in (q, Kc, Vc))
    dctx = torch.from_numpy(ctx).cuda()
    dprobe = torch.from_numpy(probe.astype(np.float32)).cuda()
    b_cap = max(1, max(len(v) for per in vis for v in per))
    vis_idx, vis_cnt = lists_to_padded(vis, H, b_cap)
    Oo, acto, sc = oc.slim_decode(q, Kc, Vc, ctx, probe.astype(np.float32), vis, tau, cfg.vis_begin, cfg.vis_end, cfg.scale)
    if case == "all_lazy":
        assert acto[:, 1:].sum() == 0 and acto[:, 0].all()
    if case == "all_active":
        assert acto.all()
    ldesc = ob.make_layer_desc(c.dQ.expand(batch, -1, -1, -1).contiguous(), c.dK.expand(batch, -1, -1, -1).contiguous(),
                               cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
    grp = ob.omni_group_subset_per_head(ldesc, vis_idx, vis_cnt, b_cap)
    desc = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, tau)
    sdesc = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, tau, static_lists=True)
    ws_a, ws_b = ob.Workspace(), ob.Workspace()
    ob.omni_slim_decode_prepare(sdesc, vis_idx, vis_cnt, b_cap, ws=ws_b)
    results = [ob.omni_slim_decode(desc, dq, dKc, dVc, dctx, dprobe, vis_idx, vis_cnt, b_cap, ws=ws_a),
               ob.omni_slim_decode(sdesc, dq, dKc, dVc, dctx, dprobe, vis_idx, vis_cnt, b_cap, ws=ws_b),
               ob.omni_slim_decode_grouped(desc, dq, dKc, dVc, dctx, dprobe, *grp)]
    # the compacted store and its paged form (pages of 32 rows handed out in order) on the same group lists
    grp_idx, grp_mask, grp_cnt = grp
    Kcomp, Vcomp = ob.omni_compact_cache(desc, dKc, dVc, grp_idx, grp_cnt)
    page_rows, pages_cap = 32, -(-grp_idx.shape[-1] // 32)
    need = -(-to_host(grp_cnt) // page_rows)
    table = np.full((batch, cfg.n_kv_heads, pages_cap), -1, dtype=np.int32)
    nxt = 0
    for bb in range(batch):
        for g in range(cfg.n_kv_heads):
            table[bb, g, : need[bb, g]] = np.arange(nxt, nxt + need[bb, g])
            nxt += int(need[bb, g])
    Kpool = torch.full((max(nxt, 1), page_rows, cfg.head_dim), float("nan"), dtype=dKc.dtype, device="cuda")
    pool = ob.make_page_pool(Kpool, torch.full_like(Kpool, float("nan")), torch.from_numpy(table).cuda())
    ob.omni_compact_cache_paged(desc, dKc, dVc, grp_idx, grp_cnt, pool)
    results.append(ob.omni_slim_decode_compact(desc, dq, dKc, dVc, dctx, dprobe, Kcomp, Vcomp, grp_idx, grp_mask, grp_cnt))
    results.append(ob.omni_slim_decode_paged(desc, dq, dKc, dVc, dctx, dprobe, pool, grp_idx, grp_mask, grp_cnt))
    torch.cuda.synchronize()
    clear = np.abs(sc - tau) > 1e-5
    for O, act in results:
        act = to_host(act)
        np.testing.assert_array_equal(act[clear], acto[clear])
        same = act == acto
        got = to_host(O)
        assert np.all(np.isfinite(got))
        assert np.max(np.abs(got[same] - Oo[same])) <= TOL_OUT[cfg.dtype]


@pytest.mark.parametrize("cfg,batch", [(CFG_BF16, 1), (CFG_BF16, 3), (CFG_BF16_64, 2), (CFG_F32, 2), (CFG_F32_128, 1)],
                         ids=lambda x: getattr(x, "name", str(x)))
def test_compacted_cache_decode(cfg, batch):
    """The rows of the group lists copied side by side: the copy is exact, and the decode step that reads it gives
    the oracle's result while the visual part of the cache itself holds garbage (it is never read)."""
    c, q, Kc, Vc, ctx, probe, vis = _decode_case(cfg, batch)
    tau = 0.08
    H, Hkv = cfg.n_q_heads, cfg.n_kv_heads
    b = len(c.o_kvidx[0][0])
    kv_idx, _ = lists_to_padded([list(c.o_kvidx[0])] * batch, H, b)
    budget = torch.full((batch,), b, dtype=torch.int32, device="cuda")
    ldesc = ob.make_layer_desc(c.dQ.expand(batch, -1, -1, -1).contiguous(), c.dK.expand(batch, -1, -1, -1).contiguous(),
                               cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
    grp_idx, grp_mask, grp_cnt = ob.omni_group_subset(ldesc, kv_idx, budget, b)
    dq, dKc, dVc = (to_device(x, cfg.dtype) for x in (q, Kc, Vc))
    dctx = torch.from_numpy(ctx).cuda()
    dprobe = torch.from_numpy(probe.astype(np.float32)).cuda()
    desc = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, tau)
    Kcomp, Vcomp = ob.omni_compact_cache(desc, dKc, dVc, grp_idx, grp_cnt)
    torch.cuda.synchronize()
    gi, gc = to_host(grp_idx), to_host(grp_cnt)
    Kh, Vh = to_host(dKc), to_host(dVc)
    for bb in range(batch):
        for g in range(Hkv):
            n = int(gc[bb, g])
            np.testing.assert_array_equal(to_host(Kcomp)[bb, g, :n], Kh[bb, g, gi[bb, g, :n]])
            np.testing.assert_array_equal(to_host(Vcomp)[bb, g, :n], Vh[bb, g, gi[bb, g, :n]])
    # the caller may now drop the visual rows of the cache: fill them with values that would wreck any sum
    dKc[:, :, cfg.vis_begin:cfg.vis_end] = float("nan")
    dVc[:, :, cfg.vis_begin:cfg.vis_end] = float("nan")
    O, act = ob.omni_slim_decode_compact(desc, dq, dKc, dVc, dctx, dprobe, Kcomp, Vcomp, grp_idx, grp_mask, grp_cnt)
    torch.cuda.synchronize()
    Oo, acto, sc = oc.slim_decode(q, Kc, Vc, ctx, probe.astype(np.float32), vis, tau, cfg.vis_begin, cfg.vis_end, cfg.scale)
    act = to_host(act)
    clear = np.abs(sc - tau) > 1e-5
    np.testing.assert_array_equal(act[clear], acto[clear])
    same = act == acto
    got = to_host(O)
    assert np.all(np.isfinite(got))
    assert np.max(np.abs(got[same] - Oo[same])) <= TOL_OUT[cfg.dtype]


@pytest.mark.parametrize("cfg,batch,page_rows", [(CFG_BF16, 1, 16), (CFG_BF16, 3, 64), (CFG_BF16_64, 2, 1), (CFG_F32, 2, 32),
                                                 (CFG_F32_128, 1, 256)], ids=lambda x: getattr(x, "name", str(x)))
def test_paged_cache_decode(cfg, batch, page_rows):
    """The compacted store cut into pages of a shared pool, the pages of every (sequence, KV head) pair scattered
    over it in a seeded random order: every row lands in its page, the decode step equals the contiguous store's
    bit for bit and the oracle's to the bar; a pair whose last page is missing loses exactly those rows."""
    c, q, Kc, Vc, ctx, probe, vis = _decode_case(cfg, batch)
    tau = 0.08
    H, Hkv, D = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim
    b = len(c.o_kvidx[0][0])
    kv_idx, _ = lists_to_padded([list(c.o_kvidx[0])] * batch, H, b)
    budget = torch.full((batch,), b, dtype=torch.int32, device="cuda")
    ldesc = ob.make_layer_desc(c.dQ.expand(batch, -1, -1, -1).contiguous(), c.dK.expand(batch, -1, -1, -1).contiguous(),
                               cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
    grp_idx, grp_mask, grp_cnt = ob.omni_group_subset(ldesc, kv_idx, budget, b)
    dq, dKc, dVc = (to_device(x, cfg.dtype) for x in (q, Kc, Vc))
    dctx = torch.from_numpy(ctx).cuda()
    dprobe = torch.from_numpy(probe.astype(np.float32)).cuda()
    desc = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, tau)
    gi, gc = to_host(grp_idx), to_host(grp_cnt)
    u_cap = grp_idx.shape[-1]
    pages_cap = -(-u_cap // page_rows)
    need = [[-(-int(gc[bb, g]) // page_rows) for g in range(Hkv)] for bb in range(batch)]
    n_pages = sum(map(sum, need)) + 3                                  # a few pages nobody owns
    rng = np.random.default_rng(77 + page_rows)
    free = list(rng.permutation(n_pages))
    table = np.full((batch, Hkv, pages_cap), -1, dtype=np.int32)
    for bb in range(batch):
        for g in range(Hkv):
            for j in range(need[bb][g]):
                table[bb, g, j] = free.pop()
    dtable = torch.from_numpy(table).cuda()
    Kpool = torch.full((n_pages, page_rows, D), float("nan"), dtype=dKc.dtype, device="cuda")
    Vpool = torch.full_like(Kpool, float("nan"))
    pool = ob.make_page_pool(Kpool, Vpool, dtable)
    ob.omni_compact_cache_paged(desc, dKc, dVc, grp_idx, grp_cnt, pool)
    Kcomp, Vcomp = ob.omni_compact_cache(desc, dKc, dVc, grp_idx, grp_cnt)
    torch.cuda.synchronize()
    Kh, Vh, Kp, Vp = to_host(dKc), to_host(dVc), to_host(Kpool), to_host(Vpool)
    for bb in range(batch):
        for g in range(Hkv):
            n = int(gc[bb, g])
            u = np.arange(n)
            rows = table[bb, g, u // page_rows].astype(np.int64) * page_rows + u % page_rows
            np.testing.assert_array_equal(Kp.reshape(-1, D)[rows], Kh[bb, g, gi[bb, g, :n]])
            np.testing.assert_array_equal(Vp.reshape(-1, D)[rows], Vh[bb, g, gi[bb, g, :n]])
    owned = np.zeros(n_pages * page_rows, dtype=bool)
    for bb in range(batch):
        for g in range(Hkv):
            u = np.arange(int(gc[bb, g]))
            owned[table[bb, g, u // page_rows].astype(np.int64) * page_rows + u % page_rows] = True
    assert np.all(np.isnan(Kp.reshape(-1, D)[~owned]))                  # nothing written outside the owned rows
    dKc2, dVc2 = dKc.clone(), dVc.clone()
    dKc2[:, :, cfg.vis_begin:cfg.vis_end] = float("nan")
    dVc2[:, :, cfg.vis_begin:cfg.vis_end] = float("nan")
    O1, act1 = ob.omni_slim_decode_paged(desc, dq, dKc2, dVc2, dctx, dprobe, pool, grp_idx, grp_mask, grp_cnt)
    O2, act2 = ob.omni_slim_decode_compact(desc, dq, dKc2, dVc2, dctx, dprobe, Kcomp, Vcomp, grp_idx, grp_mask, grp_cnt)
    torch.cuda.synchronize()
    assert torch.equal(act1, act2)
    assert torch.equal(O1.view(torch.int16 if cfg.dtype == "bf16" else torch.int32),
                       O2.view(torch.int16 if cfg.dtype == "bf16" else torch.int32))
    Oo, acto, sc = oc.slim_decode(q, Kc, Vc, ctx, probe.astype(np.float32), vis, tau, cfg.vis_begin, cfg.vis_end, cfg.scale)
    same = to_host(act1) == acto
    got = to_host(O1)
    assert np.all(np.isfinite(got))
    assert np.max(np.abs(got[same] - Oo[same])) <= TOL_OUT[cfg.dtype]
    # drop the last page of pair (0, 0): the decode step then sees the list without that page's rows
    last = need[0][0] - 1
    if last >= 1:
        table2 = table.copy()
        table2[0, 0, last] = -1
        pool2 = ob.make_page_pool(Kpool, Vpool, torch.from_numpy(table2).cuda())
        O3, act3 = ob.omni_slim_decode_paged(desc, dq, dKc2, dVc2, dctx, dprobe, pool2, grp_idx, grp_mask, grp_cnt)
        torch.cuda.synchronize()
        G = H // Hkv
        gone = set(int(x) for x in gi[0, 0, last * page_rows: int(gc[0, 0])])
        vis3 = [[np.array([t for t in vis[bb][h] if not (bb == 0 and h < G and int(t) in gone)], dtype=np.int32)
                 for h in range(H)] for bb in range(batch)]
        Oo3, acto3, _ = oc.slim_decode(q, Kc, Vc, ctx, probe.astype(np.float32), vis3, tau, cfg.vis_begin, cfg.vis_end,
                                       cfg.scale)
        same3 = to_host(act3) == acto3
        assert np.max(np.abs(to_host(O3)[same3] - Oo3[same3])) <= TOL_OUT[cfg.dtype]


def test_visual_subset_matches_oracle():
    cfg = CFG_BF16
    c = case_for(cfg)
    b = int(c.o_bud["budget"][0])
    kv_idx, _ = lists_to_padded([list(c.o_kvidx[0])], cfg.n_q_heads, b)
    budget = torch.tensor([b], dtype=torch.int32, device="cuda")
    vis_idx, vis_cnt = ob.omni_visual_subset(c.desc, kv_idx, budget, b)
    torch.cuda.synchronize()
    want = oc.visual_subset([list(c.o_kvidx[0])], cfg.vis_begin, cfg.vis_end)
    got = padded_to_lists(vis_idx, vis_cnt)
    for h in range(cfg.n_q_heads):
        np.testing.assert_array_equal(got[0][h], want[0][h])


# ------------------------------------------------------------------ whole pipeline, free running

@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
@pytest.mark.parametrize("budget_mode", [0, 1, 2])
def test_free_running_pipeline_oracle_selection_on_the_gpu_scores_gives_the_gpu_sets(cfg, budget_mode):
    """The whole pipeline runs free on the GPU; the selection kernels are then checked on the arrays they really saw:
    the oracle's selection applied to the GPU-produced scores must return the GPU's sets bit for bit, the score arrays
    themselves are compared numerically, and attention is compared on every head on the GPU's own sets."""
    c = case_for(cfg)
    N, H = cfg.n_tokens, cfg.n_q_heads
    ph = budget_mode == 2
    probe, scores = ob.omni_score_queries(c.desc, c.dQ, c.dK)
    q_idx, q_cnt = ob.omni_select_queries(c.desc, scores, c.q_mode, c.q_param)
    r = ob.omni_kv_budget(c.desc, c.dQ, c.dK, c.recall_p, c.probe_block, budget_mode)
    kv_idx = ob.omni_select_kv(c.desc, r.key_scores, r.budget, N, _per_head=ph)
    O, lse = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, kv_idx, r.budget, N, _per_head=ph)
    torch.cuda.synchronize()
    s_gpu, a_gpu = to_host(scores), to_host(r.key_scores)
    np.testing.assert_allclose(s_gpu, c.o_scores, rtol=0, atol=1e-5)
    assert np.max(np.abs(a_gpu.astype(np.float64) - c.o_a)) <= 1e-4 * c.o_a.max()
    got_q = padded_to_lists(q_idx, q_cnt)
    kv_lists = check_selection_on_gpu_scores(oc, s_gpu, a_gpu, got_q, to_host(r.flattest), to_host(r.budget),
                                             to_host(kv_idx), c.q_mode, c.q_param, c.recall_p, budget_mode,
                                             cfg.vis_begin, cfg.vis_end)
    # informational: how far the free-running sets are from the oracle's own pipeline (numeric error of the scores)
    if budget_mode == 0:
        bo = int(c.o_bud["budget"][0])
        assert abs(len(kv_lists[0][0]) - bo) <= max(2, int(2e-3 * bo))
    # attention on every head, on the sets the GPU selected
    Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, got_q, kv_lists, cfg.causal, cfg.scale)
    _check_fwd(c, to_host(O), to_host(lse), Oo, Lo)


@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
@pytest.mark.parametrize("budget_mode", [0, 1, 2])
def test_fused_selection_call_writes_what_the_four_separate_calls_write(cfg, budget_mode):
    c = case_for(cfg)
    N, H = cfg.n_tokens, cfg.n_q_heads
    probe, scores = ob.omni_score_queries(c.desc, c.dQ, c.dK)
    q_idx, q_cnt = ob.omni_select_queries(c.desc, scores, c.q_mode, c.q_param)
    r = ob.omni_kv_budget(c.desc, c.dQ, c.dK, c.recall_p, c.probe_block, budget_mode)
    kv_idx = ob.omni_select_kv(c.desc, r.key_scores, r.budget, N, _per_head=budget_mode == 2)
    f = ob.omni_prefill_select(c.desc, c.dQ, c.dK, c.q_mode, c.q_param, c.recall_p, c.probe_block, budget_mode)
    torch.cuda.synchronize()
    assert torch.equal(f.probe_keys, probe) and torch.equal(f.scores, scores)
    assert torch.equal(f.q_cnt, q_cnt)
    for a, b in zip(padded_to_lists(f.q_idx, f.q_cnt), padded_to_lists(q_idx, q_cnt)):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)
    fb = f.budget
    assert torch.equal(fb.key_scores, r.key_scores) and torch.equal(fb.kurtosis, r.kurtosis)
    assert torch.equal(fb.flattest, r.flattest) and torch.equal(fb.budget, r.budget) and torch.equal(fb.recall, r.recall)
    bud = to_host(r.budget).reshape(cfg.batch, -1)
    got, want = to_host(f.kv_idx), to_host(kv_idx)
    for b in range(cfg.batch):
        for h in range(H):
            n = int(bud[b, h if budget_mode == 2 else 0])
            np.testing.assert_array_equal(got[b, h, :n], want[b, h, :n])


def test_fused_selection_call_with_a_capacity_below_the_budget():
    cfg = CFG_BF16
    c = case_for(cfg)
    cap = 200
    f = ob.omni_prefill_select(c.desc, c.dQ, c.dK, c.q_mode, c.q_param, c.recall_p, c.probe_block, 0, b_cap=cap)
    torch.cuda.synchronize()
    assert int(to_host(f.budget.budget)[0]) > cap                 # the budget itself is reported unclamped
    a = to_host(f.budget.key_scores)
    want = oc.select_kv(a, [cap])
    np.testing.assert_array_equal(to_host(f.kv_idx)[0], want[0])
    mass = np.sort(a[0].astype(np.float64), axis=-1)[:, ::-1][:, :cap].sum(-1) / cfg.n_tokens
    np.testing.assert_allclose(to_host(f.budget.recall)[0], mass, atol=1e-6)


def _same_selection(f, g, cfg, budget_mode):
    assert torch.equal(f.probe_keys, g.probe_keys) and torch.equal(f.scores, g.scores) and torch.equal(f.q_cnt, g.q_cnt)
    for a, b in zip(padded_to_lists(f.q_idx, f.q_cnt), padded_to_lists(g.q_idx, g.q_cnt)):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)
    fb, gb = f.budget, g.budget
    assert torch.equal(fb.key_scores, gb.key_scores) and torch.equal(fb.kurtosis, gb.kurtosis)
    assert torch.equal(fb.flattest, gb.flattest) and torch.equal(fb.budget, gb.budget) and torch.equal(fb.recall, gb.recall)
    cap = f.kv_idx.shape[-1]
    bud = to_host(gb.budget).reshape(cfg.batch, -1)
    got, want = to_host(f.kv_idx), to_host(g.kv_idx)
    for b in range(cfg.batch):
        for h in range(cfg.n_q_heads):
            n = min(int(bud[b, h if budget_mode == 2 else 0]), cap)
            np.testing.assert_array_equal(got[b, h, :n], want[b, h, :n], err_msg=f"kv list, batch {b} head {h}")


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
@pytest.mark.parametrize("budget_mode", [0, 1, 2])
def test_prefill_step_in_one_call_writes_what_selection_and_attention_write(cfg, budget_mode):
    """omni_sparse_prefill (key lists formed inside the attention's gather) against omni_prefill_select followed by
    omni_sparse_attn_fwd: every output bit for bit; and the output against the oracle on the lists it returned."""
    c = case_for(cfg)
    N = cfg.n_tokens
    g = ob.omni_prefill_select(c.desc, c.dQ, c.dK, c.q_mode, c.q_param, c.recall_p, c.probe_block, budget_mode)
    Og, Lg = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, g.q_idx, g.q_cnt, g.kv_idx, g.budget.budget, N,
                                     _per_head=budget_mode == 2)
    torch.cuda.synchronize()
    f, O, lse = ob.omni_sparse_prefill(c.desc, c.dQ, c.dK, c.dV, c.q_mode, c.q_param, c.recall_p, c.probe_block,
                                       budget_mode)
    torch.cuda.synchronize()
    _same_selection(f, g, cfg, budget_mode)
    assert torch.equal(O, Og)
    assert torch.equal(lse, Lg)
    bud = to_host(f.budget.budget).reshape(cfg.batch, -1)
    kv = to_host(f.kv_idx)
    kv_lists = [[kv[b, h, : int(bud[b, h if budget_mode == 2 else 0])] for h in range(cfg.n_q_heads)]
                for b in range(cfg.batch)]
    Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, padded_to_lists(f.q_idx, f.q_cnt), kv_lists, cfg.causal, cfg.scale)
    _check_fwd(c, to_host(O), to_host(lse), Oo, Lo)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cap", [1, 63, 64, 200, 777])
def test_prefill_step_in_one_call_with_a_capacity_below_the_budget(cap):
    cfg = CFG_BF16
    c = case_for(cfg)
    g = ob.omni_prefill_select(c.desc, c.dQ, c.dK, c.q_mode, c.q_param, c.recall_p, c.probe_block, 0, b_cap=cap)
    Og, Lg = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, g.q_idx, g.q_cnt, g.kv_idx, g.budget.budget, cap)
    torch.cuda.synchronize()
    f, O, lse = ob.omni_sparse_prefill(c.desc, c.dQ, c.dK, c.dV, c.q_mode, c.q_param, c.recall_p, c.probe_block, 0,
                                       b_cap=cap)
    torch.cuda.synchronize()
    _same_selection(f, g, cfg, 0)
    assert torch.equal(O, Og) and torch.equal(lse, Lg)
    n = min(cap, int(to_host(f.budget.budget)[0]))
    want = oc.select_kv(to_host(f.budget.key_scores), [n])
    np.testing.assert_array_equal(to_host(f.kv_idx)[0, :, :n], want[0])


def test_prefill_step_in_one_call_on_tied_key_scores():
    """Key scores with many equal values at the cut: the lists formed inside the gather take the first of them in index
    order, as omni_select_kv does.  Ties are made by giving groups of tokens the same key and query rows."""
    cfg = CFG_BF16
    c = case_for(cfg)
    N = cfg.n_tokens
    K2 = c.K.copy()
    Q2 = c.Q.copy()
    for n in range(8, N - 8, 8):                       # tokens n .. n+3 share their key rows
        K2[:, :, n + 1:n + 4] = K2[:, :, n:n + 1]
    dK2, dQ2 = to_device(K2, cfg.dtype), to_device(Q2, cfg.dtype)
    for mode in (0, 2):
        g = ob.omni_prefill_select(c.desc, dQ2, dK2, c.q_mode, c.q_param, 0.6, c.probe_block, mode)
        Og, Lg = ob.omni_sparse_attn_fwd(c.desc, dQ2, dK2, c.dV, g.q_idx, g.q_cnt, g.kv_idx, g.budget.budget, N,
                                         _per_head=mode == 2)
        f, O, lse = ob.omni_sparse_prefill(c.desc, dQ2, dK2, c.dV, c.q_mode, c.q_param, 0.6, c.probe_block, mode)
        torch.cuda.synchronize()
        _same_selection(f, g, cfg, mode)
        assert torch.equal(O, Og) and torch.equal(lse, Lg)
        a = to_host(g.budget.key_scores)[0]
        bud = to_host(g.budget.budget).reshape(-1)
        cut_ties = [int(np.sum(a[h] == np.sort(a[h])[::-1][int(bud[h if mode == 2 else 0]) - 1]))
                    for h in range(cfg.n_q_heads)]
        assert max(cut_ties) >= 2, "the input was meant to put equal scores at the cut"


# ------------------------------------------------------------------ block-granular KV selection

@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
@pytest.mark.parametrize("block", [64, 100])
def test_block_granular_selection_and_attention(cfg, block):
    """Queries and keys both pooled: block scores, budget in blocks, block lists, their token lists, and the
    sparse forward on them -- each stage against the oracle on the oracle's own inputs for that stage."""
    c = case_for(cfg)
    N, H = cfg.n_tokens, cfg.n_q_heads
    nb = math.ceil(N / block)
    want_a = oc.pooled_block_scores(c.Q, c.K, block, cfg.causal, cfg.scale)
    got_a = ob.omni_block_scores(c.desc, c.dQ, c.dK, block)
    torch.cuda.synchronize()
    assert np.max(np.abs(to_host(got_a) - want_a)) <= 1e-4 * want_a.max()
    np.testing.assert_allclose(to_host(got_a).sum(-1), float(nb), rtol=1e-4)
    # budget and block lists: decided on the oracle's fp32 block scores on both sides
    a32 = want_a.astype(np.float32)
    bdesc = ob.block_level_desc(c.desc, block)
    da = torch.from_numpy(a32).cuda()
    r = ob.omni_budget_from_scores(bdesc, da, 0.9, 0)
    want_b = oc.kv_budget(a32, 0.9, 0)
    np.testing.assert_array_equal(to_host(r.budget), want_b["budget"])
    np.testing.assert_array_equal(to_host(r.flattest), want_b["flattest"])
    nbud = int(want_b["budget"][0])
    blk_idx = ob.omni_select_kv(bdesc, da, r.budget, nb)
    want_blk = oc.select_kv(a32, want_b["budget"])
    got_blk = to_host(blk_idx)
    for h in range(H):
        np.testing.assert_array_equal(got_blk[0, h, :nbud], want_blk[0][h])
    # token lists
    kv_idx, budget = ob.omni_expand_blocks(c.desc, blk_idx, r.budget, block)
    torch.cuda.synchronize()
    assert int(to_host(budget)[0]) == nbud * block
    want_tok = oc.expand_blocks(want_blk, block, N)
    got_tok = to_host(kv_idx)
    for h in range(H):
        row = got_tok[0, h, : nbud * block]
        np.testing.assert_array_equal(row[row < N], want_tok[0][h])
        assert np.all(np.diff(row.astype(np.int64)) > 0) or np.all(row[row >= N] == row[row >= N][0])
    # attention on the block lists (kept queries of the token-level case)
    q_idx, q_cnt = lists_to_padded(c.o_qidx, H, N)
    O, lse = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, kv_idx, budget, kv_idx.shape[-1])
    torch.cuda.synchronize()
    Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, c.o_qidx, want_tok, cfg.causal, cfg.scale)
    assert np.max(np.abs(to_host(O) - Oo)) <= TOL_OUT[cfg.dtype]
    fin = np.isfinite(Lo)
    assert np.array_equal(np.isfinite(to_host(lse)), fin)
    assert np.max(np.abs(to_host(lse)[fin] - Lo[fin])) <= (1e-4 if cfg.dtype == "f32" else 2e-2)


CFG_BF16_NC = synth.C2_16K.scaled(name="bf16_noncausal", frames=4, tok_per_frame=240, n_text=64, n_q_heads=8, n_kv_heads=2,
                                  causal=False, seed=31)          # 1024 tokens: a multiple of every block size below


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", [CFG_BF16, CFG_BF16_64, CFG_BF16_NC], ids=lambda c: c.name)
@pytest.mark.parametrize("block,frac", [(64, 0.4), (128, 0.5), (256, 1.0), (192, 0.3)])
def test_block_attention_in_place_equals_gathered_path_and_oracle(cfg, block, frac):
    """The forward pass that walks block lists inside one token-ordered copy of K/V per KV head: bit-for-bit the
    result of expanding the lists to tokens and gathering, and within the bf16 bar of the oracle."""
    c = case_for(cfg)
    N, H = cfg.n_tokens, cfg.n_q_heads
    if not cfg.causal and N % block:
        pytest.skip("without the causal mask the call wants whole blocks")
    nb = math.ceil(N / block)
    nsel = max(1, int(round(frac * nb)))
    rng = np.random.default_rng(1000 + block)
    lists = [[np.sort(rng.choice(nb, nsel, replace=False)).astype(np.int32) for _ in range(H)]]
    lists[0][0] = np.sort(np.concatenate([rng.choice(nb - 1, nsel - 1, replace=False), [nb - 1]])).astype(np.int32)
    blk_idx, _ = lists_to_padded(lists, H, nb)
    blk_budget = torch.tensor([nsel], dtype=torch.int32, device="cuda")
    q_idx, q_cnt = lists_to_padded(c.o_qidx, H, N)
    O1, lse1 = ob.omni_block_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, blk_idx, blk_budget, block)
    kv_idx, budget = ob.omni_expand_blocks(c.desc, blk_idx, blk_budget, block)
    O2, lse2 = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, kv_idx, budget, kv_idx.shape[-1])
    torch.cuda.synchronize()
    assert torch.equal(O1.view(torch.int16), O2.view(torch.int16))
    assert torch.equal(lse1.view(torch.int32), lse2.view(torch.int32))
    want_tok = oc.expand_blocks(lists, block, N)
    Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, c.o_qidx, want_tok, cfg.causal, cfg.scale)
    assert np.max(np.abs(to_host(O1) - Oo)) <= TOL_OUT["bf16"]
    fin = np.isfinite(Lo)
    assert np.array_equal(np.isfinite(to_host(lse1)), fin)
    assert np.max(np.abs(to_host(lse1)[fin] - Lo[fin])) <= 2e-2


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", [CFG_BF16, CFG_BF16_64, CFG_BF16_NC], ids=lambda c: c.name)
@pytest.mark.parametrize("block,frac", [(64, 0.4), (128, 0.5), (256, 1.0), (192, 0.3)])
@pytest.mark.parametrize("split_len", [0, 2])
def test_block_attention_backward_in_place_equals_gathered_path_and_oracle(cfg, block, frac, split_len):
    """The backward pass that walks block lists inside one token-ordered copy of K/V per KV head: bit-for-bit the
    gradients of expanding the lists to tokens and gathering, and within the gradient bar of the oracle.  split_len 2
    forces the long-context path of the key kernels (a key tile shared by several workgroups)."""
    c = case_for(cfg)
    N, H = cfg.n_tokens, cfg.n_q_heads
    if not cfg.causal and N % block:
        pytest.skip("without the causal mask the call wants whole blocks")
    nb = math.ceil(N / block)
    nsel = max(1, int(round(frac * nb)))
    rng = np.random.default_rng(2000 + block)
    lists = [[np.sort(rng.choice(nb, nsel, replace=False)).astype(np.int32) for _ in range(H)]]
    lists[0][0] = np.sort(np.concatenate([rng.choice(nb - 1, nsel - 1, replace=False), [nb - 1]])).astype(np.int32)
    blk_idx, _ = lists_to_padded(lists, H, nb)
    blk_budget = torch.tensor([nsel], dtype=torch.int32, device="cuda")
    q_idx, q_cnt = lists_to_padded(c.o_qidx, H, N)
    tok = oc.expand_blocks(lists, block, N)
    dO_np = synth.make_grad_output(cfg)
    O_st, lse_o, want = oracle_train(oc, cfg.dtype, c.Q, c.K, c.V, dO_np, c.o_qidx, tok, cfg.causal, cfg.scale)
    O, lse, dO = to_device(O_st, cfg.dtype), torch.from_numpy(lse_o).cuda(), to_device(dO_np, cfg.dtype)
    kv_idx, budget = ob.omni_expand_blocks(c.desc, blk_idx, blk_budget, block)
    ob.debug_key_split_len(split_len)
    try:
        g1 = ob.omni_block_attn_bwd(c.desc, c.dQ, c.dK, c.dV, O, dO, lse, q_idx, q_cnt, blk_idx, blk_budget, block)
        g2 = ob.omni_sparse_attn_bwd(c.desc, c.dQ, c.dK, c.dV, O, dO, lse, q_idx, q_cnt, kv_idx, budget, kv_idx.shape[-1])
        torch.cuda.synchronize()
    finally:
        ob.debug_key_split_len(0)
    for name, x, y in zip(("dQ", "dK", "dV"), g1, g2):
        assert torch.equal(x.view(torch.int16), y.view(torch.int16)), name
    _check_grads(cfg, g1, want, c.o_qidx, tok)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", [CFG_BF16, CFG_F32], ids=lambda c: c.name)
def test_block_lists_train_through_their_token_lists(cfg):
    """Training on block lists: expanded to token lists they go through the same forward and backward, and the
    gradients are the oracle's for those sets (pad entries of a partial last block collect nothing)."""
    c = case_for(cfg)
    N, H, block = cfg.n_tokens, cfg.n_q_heads, 64
    nb = math.ceil(N / block)
    nsel = max(2, nb // 2)
    rng = np.random.default_rng(83)
    lists = [[np.sort(np.concatenate([[0, nb - 1], 1 + rng.choice(nb - 2, nsel - 2, replace=False)])).astype(np.int32)
              for _ in range(H)]]
    blk_idx, _ = lists_to_padded(lists, H, nsel)
    blk_budget = torch.tensor([nsel], dtype=torch.int32, device="cuda")
    kv_idx, budget = ob.omni_expand_blocks(c.desc, blk_idx, blk_budget, block)
    q_idx, q_cnt = lists_to_padded(c.o_qidx, H, N)
    dO_np = synth.make_grad_output(cfg)
    dO = to_device(dO_np, cfg.dtype)
    b_cap = kv_idx.shape[-1]
    tok = oc.expand_blocks(lists, block, N)
    O_st, lse_o, want = oracle_train(oc, cfg.dtype, c.Q, c.K, c.V, dO_np, c.o_qidx, tok, cfg.causal, cfg.scale)
    O, lse = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, kv_idx, budget, b_cap)
    _check_fwd(c, to_host(O), to_host(lse), O_st.astype(np.float64), lse_o.astype(np.float64))
    grads = ob.omni_sparse_attn_bwd(c.desc, c.dQ, c.dK, c.dV, to_device(O_st, cfg.dtype), dO, torch.from_numpy(lse_o).cuda(),
                                    q_idx, q_cnt, kv_idx, budget, b_cap)
    torch.cuda.synchronize()
    _check_grads(cfg, grads, want, c.o_qidx, tok)


@pytest.mark.usefixtures("attention_route")
def test_sparse_forward_with_more_heads_than_the_queued_scheduler_places():
    """Batch 150 x 8 heads = 1200 (batch, head) pairs: above 1024 the work list falls back to one queue.  Every batch
    entry holds the same sequence, so every one must give the oracle's output for it."""
    cfg = CFG_BF16_64.scaled(name="bf16_d64_many", n_q_heads=8, n_kv_heads=2, frames=2, tok_per_frame=100, n_text=21, seed=13)
    c = case_for(cfg)
    N, H, B = cfg.n_tokens, cfg.n_q_heads, 150
    dQ, dK, dV = (x.expand(B, -1, -1, -1).contiguous() for x in (c.dQ, c.dK, c.dV))
    desc = ob.make_layer_desc(dQ, dK, cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
    b = len(c.o_kvidx[0][0])
    q_idx, q_cnt = lists_to_padded([c.o_qidx[0]] * B, H, N)
    kv_idx, _ = lists_to_padded([list(c.o_kvidx[0])] * B, H, b)
    budget = torch.full((B,), b, dtype=torch.int32, device="cuda")
    O, lse = ob.omni_sparse_attn_fwd(desc, dQ, dK, dV, q_idx, q_cnt, kv_idx, budget, b)
    torch.cuda.synchronize()
    Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, c.o_qidx, [list(c.o_kvidx[0])], cfg.causal, cfg.scale)
    Og, Lg = to_host(O), to_host(lse)
    assert np.max(np.abs(Og - Oo)) <= TOL_OUT["bf16"]                 # broadcasts over the batch
    fin = np.isfinite(Lo[0])
    assert np.array_equal(np.isfinite(Lg), np.broadcast_to(fin, Lg.shape))
    assert np.max(np.abs(Lg[:, fin] - Lo[0][fin])) <= 2e-3
    assert np.array_equal(Og[0], Og[-1]) and np.array_equal(Og[0], Og[B // 2])


@pytest.mark.usefixtures("attention_route")
def test_block_attention_in_place_edge_budgets():
    """Block budget 0: every kept query sees no key (zero output, lse = -inf).  A budget above blk_cap is clamped to
    it.  Both as the gathered path does it."""
    cfg = CFG_BF16
    c = case_for(cfg)
    N, H, block = cfg.n_tokens, cfg.n_q_heads, 128
    nb = math.ceil(N / block)
    cap = 5
    rng = np.random.default_rng(71)
    lists = [[np.sort(rng.choice(nb, cap, replace=False)).astype(np.int32) for _ in range(H)]]
    blk_idx, _ = lists_to_padded(lists, H, cap)
    q_idx, q_cnt = lists_to_padded(c.o_qidx, H, N)
    zero = torch.zeros(1, dtype=torch.int32, device="cuda")
    O0, lse0 = ob.omni_block_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, blk_idx, zero, block)
    torch.cuda.synchronize()
    assert not to_host(O0).any() and np.all(to_host(lse0) == -np.inf)
    big = torch.full((1,), cap + 7, dtype=torch.int32, device="cuda")
    O1, lse1 = ob.omni_block_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, blk_idx, big, block)
    kv_idx, budget = ob.omni_expand_blocks(c.desc, blk_idx, big, block)
    O2, lse2 = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, kv_idx, budget, kv_idx.shape[-1])
    torch.cuda.synchronize()
    assert int(to_host(budget)[0]) == cap * block
    assert torch.equal(O1.view(torch.int16), O2.view(torch.int16)) and torch.equal(lse1.view(torch.int32), lse2.view(torch.int32))
    Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, c.o_qidx, oc.expand_blocks(lists, block, N), cfg.causal, cfg.scale)
    assert np.max(np.abs(to_host(O1) - Oo)) <= TOL_OUT["bf16"]


# ------------------------------------------------------------------ attention backward

def _oracle_train(c, q_lists, kv_lists, dO_np, causal=None):
    cfg = c.cfg
    return oracle_train(oc, cfg.dtype, c.Q, c.K, c.V, dO_np, q_lists, kv_lists, cfg.causal if causal is None else causal,
                        cfg.scale)


def _run_bwd(c, q_lists, kv_lists, dO_np, O_st, lse_o, desc=None):
    """The backward call on the oracle's stored forward output and log-sum-exp (both sides read the same inputs)."""
    cfg = c.cfg
    N = cfg.n_tokens
    desc = desc or c.desc
    q_idx, q_cnt = lists_to_padded(q_lists, cfg.n_q_heads, N)
    b = max(len(x) for x in kv_lists[0])
    kv_idx, _ = lists_to_padded(kv_lists, cfg.n_q_heads, b)
    budget = torch.tensor([len(kv_lists[bb][0]) for bb in range(cfg.batch)], dtype=torch.int32, device="cuda")
    dO = to_device(dO_np, cfg.dtype)
    O, lse = to_device(O_st, cfg.dtype), torch.from_numpy(lse_o).cuda()
    dQ, dK, dV = ob.omni_sparse_attn_bwd(desc, c.dQ, c.dK, c.dV, O, dO, lse, q_idx, q_cnt, kv_idx, budget, b)
    torch.cuda.synchronize()
    return dQ, dK, dV


def _run_fwd_bwd(c, q_lists, kv_lists, dO_np, desc=None):
    """Forward and backward chained on the GPU (the backward reads the GPU's own O and lse)."""
    cfg = c.cfg
    N = cfg.n_tokens
    desc = desc or c.desc
    q_idx, q_cnt = lists_to_padded(q_lists, cfg.n_q_heads, N)
    b = max(len(x) for x in kv_lists[0])
    kv_idx, _ = lists_to_padded(kv_lists, cfg.n_q_heads, b)
    budget = torch.tensor([len(kv_lists[bb][0]) for bb in range(cfg.batch)], dtype=torch.int32, device="cuda")
    dO = to_device(dO_np, cfg.dtype)
    O, lse = ob.omni_sparse_attn_fwd(desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, kv_idx, budget, b)
    dQ, dK, dV = ob.omni_sparse_attn_bwd(desc, c.dQ, c.dK, c.dV, O, dO, lse, q_idx, q_cnt, kv_idx, budget, b)
    torch.cuda.synchronize()
    return dQ, dK, dV


def _check_grads(cfg, got, want, q_lists, kv_lists):
    # fp32: 1e-4.  bf16: 2e-2, widened where the element's own rounding scale is larger (helpers.grad_bar)
    rss = getattr(want, "rss", None) or (None, None, None)
    for name, g, w, r in zip(("dQ", "dK", "dV"), got, want, rss):
        err = np.abs(to_host(g) - w)
        over = err - grad_bar(w, cfg.dtype, r)
        i = np.unravel_index(np.argmax(over), over.shape)
        assert over[i] <= 0, f"{name}: abs err {err[i]} at {i}, reference {w[i]}, max abs err {err.max()}"
    # rows outside the kept / selected sets are exactly zero
    N, G = cfg.n_tokens, cfg.n_q_heads // cfg.n_kv_heads
    dQ, dK, dV = (to_host(x) for x in got)
    for b in range(cfg.batch):
        for h in range(cfg.n_q_heads):
            out = np.setdiff1d(np.arange(N), q_lists[b][h])
            assert np.all(dQ[b, h, out] == 0)
        for g in range(cfg.n_kv_heads):
            used = np.unique(np.concatenate([kv_lists[b][h] for h in range(g * G, (g + 1) * G)]))
            out = np.setdiff1d(np.arange(N), used)
            assert np.all(dK[b, g, out] == 0) and np.all(dV[b, g, out] == 0)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", ALL_CFGS, ids=lambda c: c.name)
def test_sparse_attn_bwd_on_oracle_selection(cfg):
    c = case_for(cfg)
    dO = synth.make_grad_output(cfg)
    kv_lists = [list(c.o_kvidx[b]) for b in range(cfg.batch)]
    O_st, lse_o, want = _oracle_train(c, c.o_qidx, kv_lists, dO)
    got = _run_bwd(c, c.o_qidx, kv_lists, dO, O_st, lse_o)
    _check_grads(cfg, got, want, c.o_qidx, kv_lists)
    # bitwise reproducible
    again = _run_bwd(c, c.o_qidx, kv_lists, dO, O_st, lse_o)
    for x, y in zip(got, again):
        assert torch.equal(x, y)
    # chained on the GPU's own forward the gradients move by what the few last-bit differences between the two stored
    # outputs do to rowsum(dO * O): well inside the bar
    chained = _run_fwd_bwd(c, c.o_qidx, kv_lists, dO)
    for name, x, y, w, r in zip(("dQ", "dK", "dV"), chained, got, want, want.rss or (None,) * 3):
        assert np.all(np.abs(to_host(x) - to_host(y)) <= grad_bar(w, cfg.dtype, r)), name


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", [CFG_BF16, CFG_F32_128], ids=lambda c: c.name)
@pytest.mark.parametrize("causal", [True, False])
def test_sparse_attn_bwd_full_sets_is_dense_attention_gradient(cfg, causal):
    c = case_for(cfg)
    N, H = cfg.n_tokens, cfg.n_q_heads
    desc = ob.make_layer_desc(c.dQ, c.dK, cfg.vis_begin, cfg.vis_end, cfg.sink_index, causal)
    full = [[np.arange(N, dtype=np.int32) for _ in range(H)] for _ in range(cfg.batch)]
    # every query of every head of a group feeds the sink key here: its gradient rows are the large ones (|dK| > 8)
    dO = synth.make_grad_output(cfg)
    O_st, lse_o, want = _oracle_train(c, full, full, dO, causal)
    got = _run_bwd(c, full, full, dO, O_st, lse_o, desc)
    _check_grads(cfg, got, want, full, full)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", [CFG_BF16_64, CFG_F32], ids=lambda c: c.name)
def test_sparse_attn_bwd_edge_sets(cfg):
    c = case_for(cfg)
    N, H = cfg.n_tokens, cfg.n_q_heads
    rng = np.random.default_rng(19)
    dO = synth.make_grad_output(cfg)
    q_lists = [[np.arange(N, dtype=np.int32)] + [np.sort(rng.choice(N, int(rng.integers(1, 150)), replace=False)).astype(np.int32)
                                                for _ in range(H - 1)]]
    q_lists[0][1] = np.arange(0, 5, dtype=np.int32)            # precedes every key of head 1: no gradient at all
    for b_sel in (1, 64, 129, 200):
        kv_lists = [[np.sort(rng.choice(np.arange(8, N), b_sel, replace=False)).astype(np.int32) for _ in range(H)]]
        O_st, lse_o, want = _oracle_train(c, q_lists, kv_lists, dO)
        got = _run_bwd(c, q_lists, kv_lists, dO, O_st, lse_o)
        _check_grads(cfg, got, want, q_lists, kv_lists)
        assert np.all(to_host(got[0])[0, 1] == 0)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", [CFG_BF16, CFG_BF16_64], ids=lambda c: c.name)
@pytest.mark.parametrize("split_len", [1, 3])
def test_sparse_attn_bwd_with_key_tiles_shared_between_workgroups(cfg, split_len):
    """Long-context path of the key kernels (several workgroups per key tile, partial planes added in order),
    forced on a short input by lowering the split length."""
    c = case_for(cfg)
    dO = synth.make_grad_output(cfg)
    kv_lists = [list(c.o_kvidx[b]) for b in range(cfg.batch)]
    O_st, lse_o, want = _oracle_train(c, c.o_qidx, kv_lists, dO)
    ob.debug_key_split_len(split_len)
    try:
        got = _run_bwd(c, c.o_qidx, kv_lists, dO, O_st, lse_o)
        again = _run_bwd(c, c.o_qidx, kv_lists, dO, O_st, lse_o)
    finally:
        ob.debug_key_split_len(0)
    _check_grads(cfg, got, want, c.o_qidx, kv_lists)
    for x, y in zip(got, again):
        assert torch.equal(x, y)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("one_call", [False, True], ids=["two_calls", "one_call"])
def test_prefill_step_replays_from_a_hip_graph(one_call):
    """No call of the step allocates, synchronises or clears memory from the host, so a caller may capture it.
    Replays are interleaved with eager work and each one must reproduce the eager result bit for bit."""
    cfg = CFG_BF16
    c = case_for(cfg)
    N = cfg.n_tokens
    eager_sel = ob.omni_prefill_select(c.desc, c.dQ, c.dK, c.q_mode, c.q_param, c.recall_p, c.probe_block, 0)
    eager_O, eager_lse = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, eager_sel.q_idx, eager_sel.q_cnt,
                                                 eager_sel.kv_idx, eager_sel.budget.budget, N)
    torch.cuda.synchronize()
    sel = ob.omni_prefill_select(c.desc, c.dQ, c.dK, c.q_mode, c.q_param, c.recall_p, c.probe_block, 0)
    O, lse = torch.empty_like(eager_O), torch.empty_like(eager_lse)

    def step():
        if one_call:
            ob.omni_sparse_prefill(c.desc, c.dQ, c.dK, c.dV, c.q_mode, c.q_param, c.recall_p, c.probe_block, 0, out=sel,
                                   O=O, lse=lse)
            return
        ob.omni_prefill_select(c.desc, c.dQ, c.dK, c.q_mode, c.q_param, c.recall_p, c.probe_block, 0, out=sel)
        ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, sel.q_idx, sel.q_cnt, sel.kv_idx, sel.budget.budget, N, O, lse)

    step()                                    # workspaces exist before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for replay in range(3):
        O.zero_()
        lse.zero_()
        sel.kv_idx.zero_()
        scratch = torch.randn(1 << 20, device="cuda").sum()      # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(O, eager_O) and torch.equal(lse, eager_lse), f"replay {replay}"
        assert torch.equal(sel.q_cnt, eager_sel.q_cnt) and torch.equal(sel.budget.budget, eager_sel.budget.budget)
        b = int(eager_sel.budget.budget[0])
        assert torch.equal(sel.kv_idx[..., :b], eager_sel.kv_idx[..., :b])
        assert torch.isfinite(scratch)


def test_decode_step_replays_from_a_hip_graph():
    """A decode step (context length advanced on the device, then the group-list call) captured once and replayed
    with a new query and a longer context each time: every replay equals the eager call on the same inputs."""
    cfg, batch = CFG_BF16, 2
    c, q, Kc, Vc, ctx, probe, vis = _decode_case(cfg, batch)
    H = cfg.n_q_heads
    b = len(c.o_kvidx[0][0])
    kv_idx, _ = lists_to_padded([list(c.o_kvidx[0])] * batch, H, b)
    budget = torch.full((batch,), b, dtype=torch.int32, device="cuda")
    ldesc = ob.make_layer_desc(c.dQ.expand(batch, -1, -1, -1).contiguous(), c.dK.expand(batch, -1, -1, -1).contiguous(),
                               cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
    grp_idx, grp_mask, grp_cnt = ob.omni_group_subset(ldesc, kv_idx, budget, b)
    dKc, dVc = (to_device(x, cfg.dtype) for x in (Kc, Vc))
    dprobe = torch.from_numpy(probe.astype(np.float32)).cuda()
    rng = np.random.default_rng(61)
    queries = [to_device(synth.round_to_bf16((q * (1.0 + 0.1 * k) + 0.05 * rng.standard_normal(q.shape)).astype(np.float32)),
                         cfg.dtype) for k in range(3)]
    q_static = queries[0].clone()
    ctx0 = torch.from_numpy(ctx).cuda() - 4                    # four rows short of what the cache holds
    ctx_static = ctx0.clone()
    desc = ob.make_decode_desc(q_static, dKc, cfg.vis_begin, cfg.vis_end, 0.08)
    O, act = torch.empty_like(q_static), torch.empty(batch, H, dtype=torch.uint8, device="cuda")

    def step():
        ctx_static.add_(1)
        ob.omni_slim_decode_grouped(desc, q_static, dKc, dVc, ctx_static, dprobe, grp_idx, grp_mask, grp_cnt, O, act)

    step()                                    # the workspace exists before the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    ctx_static.copy_(ctx0)
    for k in range(3):
        q_static.copy_(queries[k])
        O.zero_()
        scratch = torch.randn(1 << 20, device="cuda").sum()      # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want_ctx = ctx0 + (k + 1)
        assert torch.equal(ctx_static, want_ctx)
        O_e, act_e = ob.omni_slim_decode_grouped(desc, queries[k], dKc, dVc, want_ctx, dprobe, grp_idx, grp_mask, grp_cnt)
        torch.cuda.synchronize()
        assert torch.equal(O, O_e) and torch.equal(act, act_e), f"replay {k}"
        assert torch.isfinite(scratch)


def test_calls_on_two_streams_with_their_own_workspaces():
    """Every call is ordered by its stream only and keeps its scratch in the caller's workspace: a prefill step and a
    training step issued on two streams at once (default priority, one workspace each) give what they give alone."""
    ca, cb = case_for(CFG_BF16), case_for(CFG_BF16_64)
    Na, Nb = CFG_BF16.n_tokens, CFG_BF16_64.n_tokens
    dOb = to_device(synth.make_grad_output(CFG_BF16_64), "bf16")

    def step_a(ws):
        sel = ob.omni_prefill_select(ca.desc, ca.dQ, ca.dK, ca.q_mode, ca.q_param, ca.recall_p, ca.probe_block, 0, ws=ws)
        return ob.omni_sparse_attn_fwd(ca.desc, ca.dQ, ca.dK, ca.dV, sel.q_idx, sel.q_cnt, sel.kv_idx, sel.budget.budget, Na,
                                       ws=ws)

    def step_b(ws):
        sel = ob.omni_prefill_select(cb.desc, cb.dQ, cb.dK, cb.q_mode, cb.q_param, cb.recall_p, cb.probe_block, 2, ws=ws)
        O, lse = ob.omni_sparse_attn_fwd(cb.desc, cb.dQ, cb.dK, cb.dV, sel.q_idx, sel.q_cnt, sel.kv_idx, sel.budget.budget,
                                         Nb, ws=ws, _per_head=True)
        return ob.omni_sparse_attn_bwd(cb.desc, cb.dQ, cb.dK, cb.dV, O, dOb, lse, sel.q_idx, sel.q_cnt, sel.kv_idx,
                                       sel.budget.budget, Nb, ws=ws, _per_head=True)

    wa, wb = ob.Workspace(), ob.Workspace()
    alone_a, alone_b = step_a(wa), step_b(wb)
    torch.cuda.synchronize()
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(3):
        with torch.cuda.stream(sa):
            got_a = step_a(wa)
        with torch.cuda.stream(sb):
            got_b = step_b(wb)
        with torch.cuda.stream(sa):
            got_a2 = step_a(wa)
        torch.cuda.synchronize()
        for x, y in zip(alone_a + alone_b, got_a + got_b):
            assert torch.equal(x, y)
        for x, y in zip(alone_a, got_a2):
            assert torch.equal(x, y)


# ------------------------------------------------------------------ batch > 1

CFG_B2 = synth.C2_16K.scaled(name="bf16_batch2", batch=2, frames=4, tok_per_frame=252, n_text=70, n_q_heads=8, n_kv_heads=2,
                             seed=23)


@pytest.mark.parametrize("budget_mode", [0, 2])
def test_prefill_step_in_one_call_on_a_batch_of_two(budget_mode):
    test_prefill_step_in_one_call_writes_what_selection_and_attention_write(CFG_B2, budget_mode)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("budget_mode", [0, 2])
def test_two_sequences_in_a_batch_have_their_own_sets_budgets_and_gradients(budget_mode):
    cfg = CFG_B2
    c = case_for(cfg)
    N, H = cfg.n_tokens, cfg.n_q_heads
    per_head = budget_mode == 2
    want_bud = oc.kv_budget(c.o_a32, c.recall_p, budget_mode)
    assert not np.array_equal(want_bud["budget"][0], want_bud["budget"][1])      # the two sequences really differ
    kv_lists = oc.select_kv(c.o_a32, want_bud["budget"])
    kv_lists = [list(x) for x in kv_lists]
    # selection, teacher-forced on the oracle's score arrays: exact
    a = torch.from_numpy(c.o_a32).cuda()
    r = ob.omni_budget_from_scores(c.desc, a, c.recall_p, budget_mode)
    np.testing.assert_array_equal(to_host(r.budget), want_bud["budget"])
    kv_idx = ob.omni_select_kv(c.desc, a, r.budget, N, _per_head=per_head)
    got = to_host(kv_idx)
    for b in range(2):
        for h in range(H):
            np.testing.assert_array_equal(got[b, h, : len(kv_lists[b][h])], kv_lists[b][h])
    sc = torch.from_numpy(c.o_scores32).cuda()
    q_idx, q_cnt = ob.omni_select_queries(c.desc, sc, c.q_mode, c.q_param)
    for b, (x, y) in enumerate(zip(padded_to_lists(q_idx, q_cnt), c.o_qidx)):
        for h in range(H):
            np.testing.assert_array_equal(x[h], y[h], err_msg=f"batch {b} head {h}")
    # attention and gradients on those sets
    dO_np = synth.make_grad_output(cfg)
    dO = to_device(dO_np, cfg.dtype)
    O, lse = ob.omni_sparse_attn_fwd(c.desc, c.dQ, c.dK, c.dV, q_idx, q_cnt, kv_idx, r.budget, N, _per_head=per_head)
    Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, c.o_qidx, kv_lists, cfg.causal, cfg.scale)
    _check_fwd(c, to_host(O), to_host(lse), Oo, Lo)
    O_st, lse_o, want = _oracle_train(c, c.o_qidx, kv_lists, dO_np)
    grads = ob.omni_sparse_attn_bwd(c.desc, c.dQ, c.dK, c.dV, to_device(O_st, cfg.dtype), dO, torch.from_numpy(lse_o).cuda(),
                                    q_idx, q_cnt, kv_idx, r.budget, N, _per_head=per_head)
    torch.cuda.synchronize()
    _check_grads(cfg, grads, want, c.o_qidx, kv_lists)
    # free-running fused selection: same budgets up to the probe's numeric error, on both sequences
    f = ob.omni_prefill_select(c.desc, c.dQ, c.dK, c.q_mode, c.q_param, c.recall_p, c.probe_block, budget_mode)
    torch.cuda.synchronize()
    bg = to_host(f.budget.budget).astype(np.int64)
    assert np.all(np.abs(bg - want_bud["budget"]) <= np.maximum(2, (2e-3 * want_bud["budget"]).astype(np.int64)))


def test_two_sequences_of_different_lengths_in_one_padded_batch():
    """Sequences of 1859 and 1060 tokens, own visual ranges, in tensors padded to 1859 rows (NaN in the padding).
    Selection runs per sequence on a batch-1 descriptor that points into the padded tensors (strides are explicit) and
    gives the bits it gives on the sequence alone; attention forward and backward run once over the padded batch:
    the lists carry the lengths."""
    cfa = CFG_BF16
    cfb = CFG_BF16.scaled(name="bf16_d128_short", frames=5, tok_per_frame=200, n_text=60, seed=77)
    ca, cb = case_for(cfa), case_for(cfb)
    Na, Nb, H, Hkv, D = cfa.n_tokens, cfb.n_tokens, cfa.n_q_heads, cfa.n_kv_heads, cfa.head_dim
    assert Nb < Na
    nan = float("nan")
    Q = torch.full((2, H, Na, D), nan, dtype=torch.bfloat16, device="cuda")
    K = torch.full((2, Hkv, Na, D), nan, dtype=torch.bfloat16, device="cuda")
    V = torch.full_like(K, nan)
    Q[0], K[0], V[0] = ca.dQ[0], ca.dK[0], ca.dV[0]
    Q[1, :, :Nb], K[1, :, :Nb], V[1, :, :Nb] = cb.dQ[0], cb.dK[0], cb.dV[0]
    # selection of the short sequence through a view of the padded tensors
    desc_b = ob.make_layer_desc(Q[1:2, :, :Nb], K[1:2, :, :Nb], cfb.vis_begin, cfb.vis_end, cfb.sink_index, cfb.causal)
    sel_view = ob.omni_prefill_select(desc_b, Q[1:2, :, :Nb], K[1:2, :, :Nb], cb.q_mode, cb.q_param, cb.recall_p, cb.probe_block, 0)
    sel_own = ob.omni_prefill_select(cb.desc, cb.dQ, cb.dK, cb.q_mode, cb.q_param, cb.recall_p, cb.probe_block, 0)
    torch.cuda.synchronize()
    assert torch.equal(sel_view.q_cnt, sel_own.q_cnt) and torch.equal(sel_view.budget.budget, sel_own.budget.budget)
    for x, y in zip(padded_to_lists(sel_view.q_idx, sel_view.q_cnt)[0], padded_to_lists(sel_own.q_idx, sel_own.q_cnt)[0]):
        np.testing.assert_array_equal(x, y)                   # entries past a head's count are not written
    bb = int(sel_own.budget.budget[0])
    assert torch.equal(sel_view.kv_idx[..., :bb], sel_own.kv_idx[..., :bb])
    # attention over the padded batch on the oracle's sets of each sequence
    b_cap = max(len(ca.o_kvidx[0][0]), len(cb.o_kvidx[0][0]))
    q_idx, q_cnt = lists_to_padded([ca.o_qidx[0], cb.o_qidx[0]], H, Na)
    kv_idx, _ = lists_to_padded([list(ca.o_kvidx[0]), list(cb.o_kvidx[0])], H, b_cap)
    budget = torch.tensor([len(ca.o_kvidx[0][0]), len(cb.o_kvidx[0][0])], dtype=torch.int32, device="cuda")
    desc = ob.make_layer_desc(Q, K, cfa.vis_begin, cfa.vis_end, cfa.sink_index, cfa.causal)
    dOa = synth.make_grad_output(cfa)
    dOb = synth.make_grad_output(cfb)
    dO = torch.full_like(Q, nan)
    dO[0] = to_device(dOa, "bf16")[0]
    dO[1, :, :Nb] = to_device(dOb, "bf16")[0]
    O, lse = ob.omni_sparse_attn_fwd(desc, Q, K, V, q_idx, q_cnt, kv_idx, budget, b_cap)
    # the backward reads the oracle's stored forward of each sequence (NaN in the padding of both arrays)
    trained = [_oracle_train(c, c.o_qidx, [list(c.o_kvidx[0])], d) for c, d in ((ca, dOa), (cb, dOb))]
    O_in = torch.full_like(Q, nan)
    lse_in = torch.full((2, H, Na), nan, dtype=torch.float32, device="cuda")
    O_in[0], lse_in[0] = to_device(trained[0][0], "bf16")[0], torch.from_numpy(trained[0][1]).cuda()[0]
    O_in[1, :, :Nb], lse_in[1, :, :Nb] = to_device(trained[1][0], "bf16")[0], torch.from_numpy(trained[1][1]).cuda()[0]
    dQ, dK, dV = ob.omni_sparse_attn_bwd(desc, Q, K, V, O_in, dO, lse_in, q_idx, q_cnt, kv_idx, budget, b_cap)
    torch.cuda.synchronize()
    for c, cfg, n, i, (O_st, lse_o, want) in ((ca, cfa, Na, 0, trained[0]), (cb, cfb, Nb, 1, trained[1])):
        kv_lists = [list(c.o_kvidx[0])]
        _check_fwd(c, to_host(O[i:i + 1, :, :n]), to_host(lse[i:i + 1, :, :n]), O_st.astype(np.float64),
                   lse_o.astype(np.float64))
        _check_grads(cfg, (dQ[i:i + 1, :, :n], dK[i:i + 1, :, :n], dV[i:i + 1, :, :n]), want, c.o_qidx, kv_lists)
    # the padding of the short sequence: zero output and zero gradients, never NaN
    for x in (O, dQ, dK, dV):
        assert not to_host(x[1, :, Nb:]).any()
    assert np.all(to_host(lse[1, :, Nb:]) == -np.inf)


@pytest.mark.parametrize("budget_mode", [0, 2])
def test_selection_of_a_padded_batch_in_one_call_with_per_sequence_lengths(budget_mode):
    """omni_prefill_select_varlen on three sequences (1859, 1060 and 537 tokens, own visual ranges) padded to 1859 rows
    with NaN: every output of a sequence is bit for bit what omni_prefill_select gives on the sequence alone, and the
    attention call consumes the batch's lists as they are."""
    cfa = CFG_BF16
    cfb = CFG_BF16.scaled(name="bf16_d128_short", frames=5, tok_per_frame=200, n_text=60, seed=77)
    cfc = CFG_BF16.scaled(name="bf16_d128_shorter", frames=5, tok_per_frame=100, n_text=37, seed=78)
    cases = [case_for(cfa), case_for(cfb), case_for(cfc)]
    cfgs = [cfa, cfb, cfc]
    Np, H, Hkv, D = cfa.n_tokens, cfa.n_q_heads, cfa.n_kv_heads, cfa.head_dim
    nan = float("nan")
    Q = torch.full((3, H, Np, D), nan, dtype=torch.bfloat16, device="cuda")
    K = torch.full((3, Hkv, Np, D), nan, dtype=torch.bfloat16, device="cuda")
    V = torch.full_like(K, nan)
    for i, (c, cfg) in enumerate(zip(cases, cfgs)):
        n = cfg.n_tokens
        Q[i, :, :n], K[i, :, :n], V[i, :, :n] = c.dQ[0], c.dK[0], c.dV[0]
    desc = ob.make_layer_desc(Q, K, cfa.vis_begin, cfa.vis_end, cfa.sink_index, cfa.causal)
    ca = cases[0]
    sel = ob.omni_prefill_select_varlen(desc, Q, K, [c.n_tokens for c in cfgs], [c.vis_begin for c in cfgs],
                                        [c.vis_end for c in cfgs], ca.q_mode, ca.q_param, ca.recall_p, ca.probe_block,
                                        budget_mode)
    torch.cuda.synchronize()
    ph = budget_mode == 2
    for i, (c, cfg) in enumerate(zip(cases, cfgs)):
        n = cfg.n_tokens
        own = ob.omni_prefill_select(c.desc, c.dQ, c.dK, c.q_mode, c.q_param, c.recall_p, c.probe_block, budget_mode,
                                     ws=ob.Workspace())
        torch.cuda.synchronize()
        assert torch.equal(sel.probe_keys[i], own.probe_keys[0])
        assert torch.equal(sel.scores[i, :, :n], own.scores[0])
        assert torch.equal(sel.budget.key_scores[i, :, :n], own.budget.key_scores[0])
        assert torch.equal(sel.budget.kurtosis[i], own.budget.kurtosis[0])
        assert torch.equal(sel.budget.flattest[i], own.budget.flattest[0])
        assert torch.equal(sel.budget.budget[i], own.budget.budget[0])
        assert torch.equal(sel.budget.recall[i], own.budget.recall[0])
        assert torch.equal(sel.q_cnt[i], own.q_cnt[0])
        cnt, bud = to_host(own.q_cnt)[0], to_host(own.budget.budget)[0]
        for h in range(H):
            assert torch.equal(sel.q_idx[i, h, : cnt[h]], own.q_idx[0, h, : cnt[h]])
            bh = int(bud[h] if ph else bud)
            assert torch.equal(sel.kv_idx[i, h, :bh], own.kv_idx[0, h, :bh])
    # attention over the padded batch straight from the batch's lists; the shortest sequence against the oracle
    O, lse = ob.omni_sparse_attn_fwd(desc, Q, K, V, sel.q_idx, sel.q_cnt, sel.kv_idx, sel.budget.budget, Np, _per_head=ph)
    torch.cuda.synchronize()
    i, c, cfg = 2, cases[2], cfgs[2]
    n = cfg.n_tokens
    q_lists = [padded_to_lists(sel.q_idx[i:i + 1], sel.q_cnt[i:i + 1])[0]]
    bud = to_host(sel.budget.budget)[i]
    kv = to_host(sel.kv_idx)[i]
    kv_lists = [[kv[h, : int(bud[h] if ph else bud)] for h in range(H)]]
    Oo, Lo = oc.sparse_attn_fwd(c.Q, c.K, c.V, q_lists, kv_lists, cfg.causal, cfg.scale)
    _check_fwd(c, to_host(O[i:i + 1, :, :n]), to_host(lse[i:i + 1, :, :n]), Oo, Lo)
    assert not to_host(O[i, :, n:]).any() and np.all(to_host(lse[i, :, n:]) == -np.inf)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_padded_batch_with_sequences_of_two_tokens_and_of_the_full_length(dtype):
    """omni_prefill_select_varlen at its corners: a sequence of two tokens (sink + one visual token), one of 65, one
    that fills the padded length; NaN in the padding.  Per sequence bit for bit the single-sequence call."""
    Np, H, Hkv, d = 333, 4, 2, 64
    lens, v0s, v1s = [2, 65, Np], [1, 3, 10], [2, 60, Np - 20]
    rng = np.random.default_rng(4242)
    mk = lambda *shape: rng.standard_normal(shape).astype(np.float32)
    Qh, Kh = mk(3, H, Np, d), mk(3, Hkv, Np, d)
    if dtype == "bf16":
        Qh, Kh = synth.round_to_bf16(Qh), synth.round_to_bf16(Kh)
    for i, n in enumerate(lens):
        Qh[i, :, n:], Kh[i, :, n:] = np.nan, np.nan
    Q, K = to_device(Qh, dtype), to_device(Kh, dtype)
    desc = ob.make_layer_desc(Q, K, 1, 2, 0, True)
    for mode in (0, 2):
        sel = ob.omni_prefill_select_varlen(desc, Q, K, lens, v0s, v1s, 1, 0.5, 0.7, 32, mode)
        torch.cuda.synchronize()
        for i, n in enumerate(lens):
            Qi, Ki = Q[i:i + 1, :, :n].contiguous(), K[i:i + 1, :, :n].contiguous()
            di = ob.make_layer_desc(Qi, Ki, v0s[i], v1s[i], 0, True)
            own = ob.omni_prefill_select(di, Qi, Ki, 1, 0.5, 0.7, 32, mode, ws=ob.Workspace())
            torch.cuda.synchronize()
            assert torch.equal(sel.scores[i, :, :n], own.scores[0]) and torch.equal(sel.q_cnt[i], own.q_cnt[0])
            assert torch.equal(sel.budget.key_scores[i, :, :n], own.budget.key_scores[0])
            assert torch.equal(sel.budget.budget[i], own.budget.budget[0])
            assert torch.equal(sel.budget.flattest[i], own.budget.flattest[0])
            cnt, bud = to_host(own.q_cnt)[0], to_host(own.budget.budget)[0]
            for h in range(H):
                assert torch.equal(sel.q_idx[i, h, : cnt[h]], own.q_idx[0, h, : cnt[h]])
                bh = int(bud[h] if mode == 2 else bud)
                assert 1 <= bh <= n
                assert torch.equal(sel.kv_idx[i, h, :bh], own.kv_idx[0, h, :bh])
            # and the single-sequence call against the oracle's selection on its own score arrays
            check_selection_on_gpu_scores(oc, to_host(own.scores), to_host(own.budget.key_scores),
                                          padded_to_lists(own.q_idx, own.q_cnt), to_host(own.budget.flattest),
                                          to_host(own.budget.budget), to_host(own.kv_idx), 1, 0.5, 0.7, mode, v0s[i], v1s[i])


# ------------------------------------------------------------------ strides

@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", [CFG_BF16, CFG_F32], ids=lambda c: c.name)
def test_token_major_memory_layout_gives_the_same_bits(cfg):
    """Q, K, V as a projection leaves them in memory ([batch, token, head, dim], viewed as [batch, head, token, dim]):
    every call reads and writes through the descriptor's strides and reproduces the head-major results bit for bit."""
    c = case_for(cfg)
    N = cfg.n_tokens
    tm = lambda t: t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    Q2, K2, V2 = tm(c.dQ), tm(c.dK), tm(c.dV)
    assert Q2.stride(1) == cfg.head_dim and Q2.stride(2) == cfg.n_q_heads * cfg.head_dim
    desc2 = ob.make_layer_desc(Q2, K2, cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
    dO = to_device(synth.make_grad_output(cfg), cfg.dtype)
    dO2 = tm(dO)

    def run(desc, Q, K, V, g):
        sel = ob.omni_prefill_select(desc, Q, K, c.q_mode, c.q_param, c.recall_p, c.probe_block, 0)
        O, lse = ob.omni_sparse_attn_fwd(desc, Q, K, V, sel.q_idx, sel.q_cnt, sel.kv_idx, sel.budget.budget, N)
        grads = ob.omni_sparse_attn_bwd(desc, Q, K, V, O, g, lse, sel.q_idx, sel.q_cnt, sel.kv_idx, sel.budget.budget, N)
        Od, _ = ob.omni_dense_attn_fwd(desc, Q, K, V)
        torch.cuda.synchronize()
        return sel, O, lse, grads, Od

    s1, O1, l1, g1, d1 = run(c.desc, c.dQ, c.dK, c.dV, dO)
    s2, O2, l2, g2, d2 = run(desc2, Q2, K2, V2, dO2)
    assert O2.stride() == Q2.stride() and g2[1].stride() == K2.stride()          # outputs laid out like their inputs
    assert torch.equal(s1.scores, s2.scores) and torch.equal(s1.budget.key_scores, s2.budget.key_scores)
    assert torch.equal(s1.q_cnt, s2.q_cnt) and torch.equal(s1.budget.budget, s2.budget.budget)
    assert torch.equal(O1, O2) and torch.equal(l1, l2) and torch.equal(d1, d2)
    for x, y in zip(g1, g2):
        assert torch.equal(x, y)


@pytest.mark.parametrize("cfg,batch", [(CFG_BF16, 2), (CFG_F32, 2)], ids=lambda x: getattr(x, "name", str(x)))
def test_decode_on_a_token_major_cache_gives_the_same_bits(cfg, batch):
    """The KV cache as [batch, token, head, dim] in memory (viewed head-major): every decode call reads it through
    the descriptor's strides and gives the head-major cache's result bit for bit."""
    c, q, Kc, Vc, ctx, probe, vis = _decode_case(cfg, batch)
    H = cfg.n_q_heads
    b = len(c.o_kvidx[0][0])
    kv_idx, _ = lists_to_padded([list(c.o_kvidx[0])] * batch, H, b)
    budget = torch.full((batch,), b, dtype=torch.int32, device="cuda")
    ldesc = ob.make_layer_desc(c.dQ.expand(batch, -1, -1, -1).contiguous(), c.dK.expand(batch, -1, -1, -1).contiguous(),
                               cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
    grp_idx, grp_mask, grp_cnt = ob.omni_group_subset(ldesc, kv_idx, budget, b)
    vis_idx, vis_cnt = ob.omni_visual_subset(ldesc, kv_idx, budget, b)
    dq, dKc, dVc = (to_device(x, cfg.dtype) for x in (q, Kc, Vc))
    tm = lambda t: t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    K2, V2 = tm(dKc), tm(dVc)
    assert K2.stride(1) == cfg.head_dim and K2.stride(2) == cfg.n_kv_heads * cfg.head_dim
    dctx = torch.from_numpy(ctx).cuda()
    dprobe = torch.from_numpy(probe.astype(np.float32)).cuda()
    d1 = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, 0.08)
    d2 = ob.make_decode_desc(dq, K2, cfg.vis_begin, cfg.vis_end, 0.08)

    def run(desc, Kx, Vx):
        out = [ob.omni_slim_decode(desc, dq, Kx, Vx, dctx, dprobe, vis_idx, vis_cnt, vis_idx.shape[-1])[0],
               ob.omni_slim_decode_grouped(desc, dq, Kx, Vx, dctx, dprobe, grp_idx, grp_mask, grp_cnt)[0],
               ob.omni_dense_decode(desc, dq, Kx, Vx, dctx)]
        Kcomp, Vcomp = ob.omni_compact_cache(desc, Kx, Vx, grp_idx, grp_cnt)
        out.append(ob.omni_slim_decode_compact(desc, dq, Kx, Vx, dctx, dprobe, Kcomp, Vcomp, grp_idx, grp_mask, grp_cnt)[0])
        torch.cuda.synchronize()
        return out, Kcomp

    o1, kc1 = run(d1, dKc, dVc)
    o2, kc2 = run(d2, K2, V2)
    for x, y in zip(o1, o2):
        assert torch.equal(x, y)
    n = int(grp_cnt.min())
    assert torch.equal(kc1[:, :, :n], kc2[:, :, :n])


# ------------------------------------------------------------------ visual tokens in the middle of the sequence

@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("cfg", [CFG_BF16, CFG_F32], ids=lambda c: c.name)
def test_visual_range_between_two_text_segments_and_a_sink_that_is_not_token_0(cfg):
    """[system text][visual tokens][question]: the visual range, the sink and the rows a decode step always reads
    are descriptor arguments; the oracle is called with the same ones."""
    c, q, Kc, Vc, ctx, _, _ = _decode_case(cfg, 2)
    N, H = cfg.n_tokens, cfg.n_q_heads
    v0, v1, sink = 69, N - 131, 2
    desc = ob.make_layer_desc(c.dQ, c.dK, v0, v1, sink, cfg.causal)
    o_probe = oc.probe_keys(c.K, v0, v1, sink)
    o_scores = oc.score_queries(c.Q, o_probe, cfg.scale)
    probe, scores = ob.omni_score_queries(desc, c.dQ, c.dK)
    torch.cuda.synchronize()
    np.testing.assert_allclose(to_host(probe), o_probe, rtol=0, atol=2e-5)
    np.testing.assert_allclose(to_host(scores), o_scores, rtol=0, atol=2e-5)
    s32 = o_scores.astype(np.float32)
    for mode, param in ((0, 0.08), (1, 0.3)):
        want = oc.select_queries(s32, mode, param, v0, v1)
        q_idx, q_cnt = ob.omni_select_queries(desc, torch.from_numpy(s32).cuda(), mode, param)
        got = padded_to_lists(q_idx, q_cnt)
        for h in range(H):
            np.testing.assert_array_equal(got[0][h], want[0][h], err_msg=f"mode {mode} head {h}")
            assert np.all(np.isin(np.arange(0, v0), got[0][h])) and np.all(np.isin(np.arange(v1, N), got[0][h]))
    # decode: stored visual rows are the selected keys inside [v0, v1); rows below v0 and from v1 on are always read
    batch = 2
    b = len(c.o_kvidx[0][0])
    vis = oc.visual_subset([list(c.o_kvidx[0])] * batch, v0, v1)
    kv_idx, _ = lists_to_padded([list(c.o_kvidx[0])] * batch, H, b)
    budget = torch.full((batch,), b, dtype=torch.int32, device="cuda")
    ldesc = ob.make_layer_desc(c.dQ.expand(batch, -1, -1, -1).contiguous(), c.dK.expand(batch, -1, -1, -1).contiguous(),
                               v0, v1, sink, cfg.causal)
    vis_idx, vis_cnt = ob.omni_visual_subset(ldesc, kv_idx, budget, b)
    for bb in range(batch):
        for h in range(H):
            np.testing.assert_array_equal(padded_to_lists(vis_idx, vis_cnt)[bb][h], vis[bb][h])
    grp_idx, grp_mask, grp_cnt = ob.omni_group_subset(ldesc, kv_idx, budget, b)
    dq, dKc, dVc = (to_device(x, cfg.dtype) for x in (q, Kc, Vc))
    dctx = torch.from_numpy(ctx).cuda()
    probe_b = np.repeat(o_probe, batch, axis=0).astype(np.float32)
    dprobe = torch.from_numpy(probe_b).cuda()
    tau = 0.08
    ddesc = ob.make_decode_desc(dq, dKc, v0, v1, tau)
    Oo, acto, sc = oc.slim_decode(q, Kc, Vc, ctx, probe_b, vis, tau, v0, v1, cfg.scale)
    clear = np.abs(sc - tau) > 1e-5
    Kcomp, Vcomp = ob.omni_compact_cache(ddesc, dKc, dVc, grp_idx, grp_cnt)
    outs = {
        "per-head": ob.omni_slim_decode(ddesc, dq, dKc, dVc, dctx, dprobe, vis_idx, vis_cnt, b),
        "grouped": ob.omni_slim_decode_grouped(ddesc, dq, dKc, dVc, dctx, dprobe, grp_idx, grp_mask, grp_cnt),
        "compact": ob.omni_slim_decode_compact(ddesc, dq, dKc, dVc, dctx, dprobe, Kcomp, Vcomp, grp_idx, grp_mask, grp_cnt),
    }
    torch.cuda.synchronize()
    for name, (O, act) in outs.items():
        act = to_host(act)
        np.testing.assert_array_equal(act[clear], acto[clear], err_msg=name)
        same = act == acto
        assert np.max(np.abs(to_host(O)[same] - Oo[same])) <= TOL_OUT[cfg.dtype], name


# ------------------------------------------------------------------ decode: every head-group tiling

@pytest.mark.parametrize("G,hkv,d", [(7, 2, 128), (8, 1, 128), (6, 2, 64), (3, 2, 128), (5, 1, 64), (16, 1, 128)])
def test_decode_with_other_group_sizes(G, hkv, d):
    """Heads per KV group decide how many heads a workgroup serves at once (8, 7, 4, 2 or 1) and whether the scores
    come from the matrix cores: all three decode calls and the plain one on each tiling."""
    cfg = synth.C2_16K.scaled(name=f"dec_g{G}", frames=3, tok_per_frame=211, n_text=45, n_q_heads=G * hkv, n_kv_heads=hkv,
                              head_dim=d, seed=60 + G)
    batch = 2
    c, q, Kc, Vc, ctx, probe, vis = _decode_case(cfg, batch)
    tau = 0.08
    H = cfg.n_q_heads
    b = len(c.o_kvidx[0][0])
    kv_idx, _ = lists_to_padded([list(c.o_kvidx[0])] * batch, H, b)
    budget = torch.full((batch,), b, dtype=torch.int32, device="cuda")
    ldesc = ob.make_layer_desc(c.dQ.expand(batch, -1, -1, -1).contiguous(), c.dK.expand(batch, -1, -1, -1).contiguous(),
                               cfg.vis_begin, cfg.vis_end, cfg.sink_index, cfg.causal)
    vis_idx, vis_cnt = ob.omni_visual_subset(ldesc, kv_idx, budget, b)
    grp_idx, grp_mask, grp_cnt = ob.omni_group_subset(ldesc, kv_idx, budget, b)
    dq, dKc, dVc = (to_device(x, cfg.dtype) for x in (q, Kc, Vc))
    dctx = torch.from_numpy(ctx).cuda()
    dprobe = torch.from_numpy(probe.astype(np.float32)).cuda()
    desc = ob.make_decode_desc(dq, dKc, cfg.vis_begin, cfg.vis_end, tau)
    Kcomp, Vcomp = ob.omni_compact_cache(desc, dKc, dVc, grp_idx, grp_cnt)
    outs = {
        "per-head": ob.omni_slim_decode(desc, dq, dKc, dVc, dctx, dprobe, vis_idx, vis_cnt, b),
        "grouped": ob.omni_slim_decode_grouped(desc, dq, dKc, dVc, dctx, dprobe, grp_idx, grp_mask, grp_cnt),
        "compact": ob.omni_slim_decode_compact(desc, dq, dKc, dVc, dctx, dprobe, Kcomp, Vcomp, grp_idx, grp_mask, grp_cnt),
    }
    Od = ob.omni_dense_decode(desc, dq, dKc, dVc, dctx)
    torch.cuda.synchronize()
    Oo, acto, sc = oc.slim_decode(q, Kc, Vc, ctx, probe.astype(np.float32), vis, tau, cfg.vis_begin, cfg.vis_end, cfg.scale)
    clear = np.abs(sc - tau) > 1e-5
    for name, (O, act) in outs.items():
        act = to_host(act)
        np.testing.assert_array_equal(act[clear], acto[clear], err_msg=name)
        same = act == acto
        assert np.max(np.abs(to_host(O)[same] - Oo[same])) <= TOL_OUT[cfg.dtype], name
    assert np.max(np.abs(to_host(Od) - oc.dense_decode(q, Kc, Vc, ctx, cfg.scale))) <= TOL_OUT[cfg.dtype]


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("rows", [64, 65, 96 * 64, 96 * 64 + 1, 200 * 64 + 5])
def test_decode_at_the_edges_of_how_a_head_is_combined(rows, dtype, d):
    """One slice, 96 slices and one more (where d = 128 goes to two workgroups a head), several trips; the last slices hold no
    row of a shorter sequence."""
    g = torch.Generator(device="cuda").manual_seed(rows)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)  # noqa: E731
    q, K, V = rand(2, 2, d), rand(2, 1, rows, d), rand(2, 1, rows, d)
    ctx = torch.tensor([rows, max(1, rows // 3)], dtype=torch.int32, device="cuda")
    O = ob.omni_dense_decode(ob.make_decode_desc(q, K, 0, 0, 0.0), q, K, V, ctx)
    for b in range(2):
        n = int(ctx[b])
        p = torch.softmax(q[b].double() @ K[b, 0, :n].double().T * d ** -0.5, -1)
        assert float((O[b].double() - p @ V[b, 0, :n].double()).abs().max()) <= TOL_OUT[dtype]


# ------------------------------------------------------------------ odd layouts of the visual range and the sink

@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("layout", ["all_visual", "sink_not_first", "two_visual_tokens", "text_on_both_sides",
                                    "visual_at_the_end"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_selection_and_attention_on_odd_layouts(layout, dtype):
    """Where the visual tokens and the sink sit is the caller's business: the whole sequence visual (the sink inside
    the range), a sink that is not token 0, a visual range of two tokens, text on both sides, visual tokens up to the
    last position.  Scores, kept queries, key scores, budgets and lists against the oracle (lists on the GPU's own
    score arrays, bit for bit), then attention on those sets."""
    N, H, Hkv, d = 700, 6, 2, 64
    v0, v1, sink = {"all_visual": (0, N, 0), "sink_not_first": (9, 600, 5), "two_visual_tokens": (300, 302, 0),
                    "text_on_both_sides": (200, 450, 0), "visual_at_the_end": (64, N, 0)}[layout]
    rng = np.random.default_rng(300 + sorted(["all_visual", "sink_not_first", "two_visual_tokens", "text_on_both_sides",
                                              "visual_at_the_end"]).index(layout))
    mk = lambda *shape: rng.standard_normal(shape).astype(np.float32)
    Q, K, V = mk(1, H, N, d), mk(1, Hkv, N, d), mk(1, Hkv, N, d)
    K[0, :, sink] *= 1.5
    if dtype == "bf16":
        Q, K, V = (synth.round_to_bf16(x) for x in (Q, K, V))
    scale = d ** -0.5
    dQ, dK, dV = (to_device(x, dtype) for x in (Q, K, V))
    desc = ob.make_layer_desc(dQ, dK, v0, v1, sink, True, scale)
    tau, p, pb = 0.45, 0.8, 64
    for mode in (0, 2):
        sel, O, lse = ob.omni_sparse_prefill(desc, dQ, dK, dV, 0, tau, p, pb, mode)
        torch.cuda.synchronize()
        probe = oc.probe_keys(K, v0, v1, sink)
        o_scores = oc.score_queries(Q, probe, scale)
        s_gpu, a_gpu = to_host(sel.scores), to_host(sel.budget.key_scores)
        assert np.max(np.abs(s_gpu - o_scores)) <= 2e-5
        o_a = oc.pooled_key_scores(Q, K, pb, True, scale)
        assert np.max(np.abs(a_gpu - o_a)) <= 1e-4 * o_a.max()
        got_q = padded_to_lists(sel.q_idx, sel.q_cnt)
        kv_lists = check_selection_on_gpu_scores(oc, s_gpu, a_gpu, got_q, to_host(sel.budget.flattest),
                                                 to_host(sel.budget.budget), to_host(sel.kv_idx), 0, tau, p, mode, v0, v1)
        kept = sum(len(x) for x in got_q[0])
        assert H * (N - (v1 - v0)) <= kept <= H * N                  # non-visual queries are always kept
        assert len(got_q[0][0]) == N                                 # head 0 keeps every query
        Oo, Lo = oc.sparse_attn_fwd(Q, K, V, got_q, kv_lists, True, scale)
        assert np.max(np.abs(to_host(O) - Oo)) <= TOL_OUT[dtype]
        fin = np.isfinite(Lo)
        assert np.array_equal(np.isfinite(to_host(lse)), fin)
        assert np.max(np.abs(to_host(lse)[fin] - Lo[fin])) <= (1e-4 if dtype == "f32" else 2e-3)


@pytest.mark.parametrize("nv", [1, 64, 65, 8191, 32768, 32769])
@pytest.mark.parametrize("d", [64, 128])
def test_decode_on_lists_as_they_are_around_the_short_slices(nv, d):
    """One KV group of seven heads, 256 slices at most: slices of 1 to 128 tokens take spans of 128 and search all lists, those of
    129 spans of 1024; a head that stores everything, one that stores nothing, stored rows beyond the context.  The rows at
    the edges of slices, spans and context weigh so much that one of them missing or too many is seen, and so is a slice: the
    reference without it is outside the bar."""
    H, cap, rng = 7, nv + 40, np.random.default_rng(nv)
    g = torch.Generator(device="cuda").manual_seed(nv)
    K, V = (torch.randn(1, 1, cap, d, generator=g, device="cuda") for _ in range(2))
    q = torch.randn(1, H, d, generator=g, device="cuda").bfloat16()
    probe = torch.randn(1, 1, 2, d, generator=g, device="cuda")
    per = -(-nv // 256)
    edges = sorted(t for t in {0, 1, 63, 64, 127, 128, per - 1, per, 2 * per - 1, 2 * per, 1023, 1024, nv // 2, nv - 6, nv - 5, nv - 1}
                   if 0 <= t < nv)
    # the same logit for every head, log(rows / 64 + 1): a weight of about a hundredth each
    dual = torch.linalg.pinv(q[0].double()).sum(1) * np.log(cap / 64 + 1) * d ** 0.5
    K[0, 0, edges] = dual.float()
    K, V = K.bfloat16(), V.bfloat16()
    keep = rng.random((H, nv)) < rng.random((H, 1))
    keep[0], keep[1] = True, False
    lists = [[np.flatnonzero(keep[h]).astype(np.int32) for h in range(H)]]
    vis_idx, vis_cnt = lists_to_padded(lists, H, nv)

    def reference(h, rows):
        if not len(rows):
            return torch.zeros(2, d, dtype=torch.float64, device="cuda")
        v = V[0, 0, rows].double()
        w = torch.softmax(K[0, 0, rows].double() @ q[0, h].double() * d ** -0.5, -1)
        return torch.stack([w @ v, (w.square() @ v.square()).sqrt()])

    for ctx in (nv + 33, max(1, nv - 5)):
        desc = ob.make_decode_desc(q, K, 0, nv, 0.2)
        O, active = ob.omni_slim_decode(desc, q, K, V, torch.tensor([ctx], dtype=torch.int32, device="cuda"), probe, vis_idx,
                                        vis_cnt, nv)
        for h in range(H):
            z = probe[0, 0].double() @ q[0, h].double() * d ** -0.5
            act = h == 0 or float(torch.sigmoid(z[1] - z[0])) > 0.2
            assert bool(active[0, h]) == act
            seen = np.ones(ctx, dtype=bool)
            seen[:min(nv, ctx)] = keep[h, :ctx] if act else False
            want, rss = reference(h, np.flatnonzero(seen))
            # weights rounded to 8 bits, as in grad_bar, and the result stored in 8 bits
            bar = GRAD_RSS * rss + 0.5 * torch.from_numpy(bf16_ulp(want.cpu().numpy())).cuda()
            assert bool(((O[0, h].double() - want).abs() <= bar).all())
            for t in edges:                                # the bar tells a row from no row
                rows = np.flatnonzero(seen ^ (np.arange(ctx) == t)) if t < ctx else np.append(np.flatnonzero(seen), t)
                assert not bool(((reference(h, rows)[0] - want).abs() <= bar).all())
            for first in (0, nv // 2 // per * per, (nv - 1) // per * per) if h == 0 else ():      # and a slice from none
                rows = np.flatnonzero(seen & ((np.arange(ctx) < first) | (np.arange(ctx) >= min(nv, first + per))))
                assert first >= ctx or not bool(((reference(h, rows)[0] - want).abs() <= bar).all())


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_kernel_timing_records_the_launches_that_the_header_names(dtype, attention_route):
    """Which ids a call records, and how often: a program that times one id must not get another kernel, or nothing."""
    long, N, H, Hkv, d = attention_route == "long", 300, 4, 2, 64
    g = torch.Generator(device="cuda").manual_seed(1)
    rand = lambda h: torch.randn(1, h, N, d, generator=g, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32)  # noqa: E731
    Q, K, V, dO = rand(H), rand(Hkv), rand(Hkv), rand(H)
    desc = ob.make_layer_desc(Q, K, 0, N - 9, 0, True)

    def launches(call):
        call()
        ob.profile_enable(True)
        out = call()
        got = {name: ob.profile_read(name)[1] for name in ob.PROF_KERNELS}
        ob.profile_enable(False)
        return out, {name: n for name, n in got.items() if n}

    try:
        _, n = launches(lambda: ob.omni_score_queries(desc, Q, K))
        assert n == {"score": 1}
        sel, n = launches(lambda: ob.omni_prefill_select(desc, Q, K, 0, 0.3, 0.9, 64, 0))
        assert n == {"pool_q": 1, "probe_lse": 1, "probe_sum": 1}
        lists = (sel.q_idx, sel.q_cnt, sel.kv_idx, sel.budget.budget, N)
        (O, lse), n = launches(lambda: ob.omni_sparse_attn_fwd(desc, Q, K, V, *lists))
        assert n == {"attn_fwd": 1, "pack_kv": 1, **({"clear_out": 1} if long else {})}
        _, n = launches(lambda: ob.omni_sparse_attn_bwd(desc, Q, K, V, O, dO, lse, *lists))
        assert n == {"bwd_dkdv": 1, "bwd_reduce": 1, "pack_kv": 1, **({"clear_out": 1} if long or dtype == "bf16" else {}),
                     **({"bwd_dq": 1} if long and dtype == "f32" else {})}
    finally:
        ob.profile_enable(False)
