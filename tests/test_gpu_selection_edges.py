"""The cut search and the list writers on score vectors where they can go wrong: lengths at the edges of a trip, of a
chunk and of a wavefront; more elements in one bin than the list in LDS holds; long runs of equal scores; few elements
left to rank; negative, zero, infinite and NaN scores.  The oracle's selection on the same float32 arrays is the answer,
bit for bit for the index sets and budgets."""
import numpy as np
import pytest
import torch

from oracle import omni_oracle as oc
from paper_2511_12201_amd import binding as ob
from tests.helpers import check_selection_on_gpu_scores, padded_to_lists

pytestmark = pytest.mark.gpu


def _scores(kind, rng, H, N):
    if kind == "lognormal":
        a = np.exp(1.5 * rng.standard_normal((1, H, N)))
    elif kind == "narrow":              # one bin of the first digit holds everything
        a = 1.0 + 0.2 * rng.random((1, H, N))
    elif kind == "equal":
        a = np.full((1, H, N), 0.75)
    elif kind == "steps":               # runs of equal scores, the cut inside one
        a = np.floor(4 * rng.random((1, H, N))) + 0.5
    else:                               # "zeros": more than half of the scores carry no mass
        a = np.maximum(rng.standard_normal((1, H, N)) - 0.5, 0.0)
        a[..., 0] = 1.0
    return np.ascontiguousarray(a * (N / a.sum(-1, keepdims=True)), dtype=np.float32)


def _desc(H, N, v0, v1):
    q = torch.empty(1, H, N, 64, dtype=torch.bfloat16, device="cuda")
    return ob.make_layer_desc(q, q, v0, v1, 0, True)


@pytest.mark.parametrize("kind", ["lognormal", "narrow", "equal", "steps", "zeros"])
@pytest.mark.parametrize("N", [1, 2, 63, 65, 1023, 1025, 8193, 20001])
def test_budget_and_lists_on_scores_in_hand(N, kind):
    H, rng = 3, np.random.default_rng(N)
    a = _scores(kind, rng, H, N)
    s = rng.random((1, H, N)).astype(np.float32) if kind != "equal" else np.full((1, H, N), 0.3, np.float32)
    v0, v1 = (0, 1) if N < 3 else (1, N - 1)
    d, da, ds = _desc(H, N, v0, v1), torch.from_numpy(a).cuda(), torch.from_numpy(s).cuda()
    for mode, p, q_mode, q_param in ((0, 0.95, 0, 0.3), (1, 0.5, 1, 0.37), (2, 1.0, 1, 1.0), (2, 0.2, 0, 0.9)):
        r = ob.omni_budget_from_scores(d, da, p, mode)
        kv = (ob.omni_select_kv_per_head if mode == 2 else ob.omni_select_kv)(d, da, r.budget, N)
        q_idx, q_cnt = ob.omni_select_queries(d, ds, q_mode, q_param)
        torch.cuda.synchronize()
        bud = r.budget.cpu().numpy()
        check_selection_on_gpu_scores(oc, s, a, padded_to_lists(q_idx, q_cnt), r.flattest.cpu().numpy(), bud,
                                      kv.cpu().numpy(), q_mode, q_param, p, mode, v0, v1)
        for h in range(H):
            top = np.sort(a[0, h].astype(np.float64))[::-1][: int(bud[0, h] if mode == 2 else bud[0])]
            # masses are truncated to 2^-40 each, the recall is stored in fp32
            assert abs(float(r.recall[0, h]) - top.sum() / N) <= 2.0 ** -23


@pytest.mark.parametrize("N", [8191, 8192, 8193, 16384, 33000])
def test_cuts_among_scores_that_no_sample_shows(N):
    """Nearly all scores within a thousandth of each other, a hundred far above and a hundred far below at positions between those
    that the bins are laid out by: cuts on both sides of every such group, and budgets of their mass."""
    H, rng = 2, np.random.default_rng(N)
    a = (1.0 + 1e-3 * rng.random((1, H, N))).astype(np.float32)
    seen = N * np.arange(1024) // 1024
    at = rng.choice(np.setdiff1d(np.arange(N), seen) if N > 8192 else np.arange(N), 200, replace=False)
    a[0, :, at[:100]] = np.exp2(20 * rng.random((100, 1))).astype(np.float32)
    a[0, :, at[100:]] = np.exp2(-20 * rng.random((100, 1)) - 1).astype(np.float32)
    d, da = _desc(H, N, 0, N), torch.from_numpy(a).cuda()
    for b in (1, 50, 99, 100, 101, N // 2, N - 101, N - 100, N - 99, N - 1):
        kv = ob.omni_select_kv(d, da, torch.tensor([b], dtype=torch.int32, device="cuda"), N).cpu().numpy()
        for h in range(H):
            np.testing.assert_array_equal(kv[0, h, :b], np.sort(np.lexsort((np.arange(N), -a[0, h]))[:b]))
    for p in (1e-3, 0.5, 0.9, 0.999):
        c = np.ascontiguousarray(a * (N / a.sum(-1, keepdims=True, dtype=np.float64)), dtype=np.float32)
        r = ob.omni_budget_from_scores(d, torch.from_numpy(c).cuda(), p, 2)
        for h in range(H):
            b = int(r.budget[0, h])
            assert b == oc.budget_of(c[0, h], p, N)
            assert abs(float(r.recall[0, h]) - np.sort(c[0, h].astype(np.float64))[::-1][:b].sum() / N) <= 2.0 ** -23


@pytest.mark.parametrize("m", [1, 64, 65, 255, 256, 257, 1025])
@pytest.mark.parametrize("N", [2000, 8192, 8193, 8194, 8195, 16385, 24579])
def test_cuts_in_a_bin_that_holds_a_given_number_of_scores(N, m):
    """m neighbouring scores, some of them equal, far from all others: as many as are ranked against each other in one go, fewer and
    more, in vectors whose last load is whole, moved back by one, two or three elements, or not there."""
    H, rng = 2, np.random.default_rng(N + m)
    a = np.exp(2 * rng.standard_normal((1, H, N)))
    a[(a > 1.0) & (a < 4.0)] *= 4.0
    at = np.stack([rng.choice(N, m, replace=False) for _ in range(H)])
    for h in range(H):
        a[0, h, at[h]] = 2.0 + 2.0 ** -18 * (rng.integers(0, 2 * m, m) // 2)
    a = a.astype(np.float32)
    d = _desc(H, N, 0, N)
    for h in range(H):
        above = int((a[0, h] >= 2.5).sum())
        for b in sorted({above + 1, above + (m + 1) // 2, above + m, min(N, above + m + 1)}):
            kv = ob.omni_select_kv(d, torch.from_numpy(a).cuda(), torch.tensor([b], dtype=torch.int32, device="cuda"), N)
            np.testing.assert_array_equal(kv[0, h, :b].cpu().numpy(), np.sort(np.lexsort((np.arange(N), -a[0, h]))[:b]))
        c = np.ascontiguousarray(a * (N / a.sum(-1, keepdims=True, dtype=np.float64)), dtype=np.float32)
        top = np.sort(c[0, h].astype(np.float64))[::-1][: above + (m + 1) // 2]
        p = float((top.sum() - 0.5 * top[-1]) / N)      # a cut amid the group, half an element away from the next
        r = ob.omni_budget_from_scores(d, torch.from_numpy(c).cuda(), p, 2)
        assert int(r.budget[0, h]) == oc.budget_of(c[0, h], p, N)


def test_lists_with_infinite_negative_and_nan_scores():
    """The order of the keys is that of the floats, NaN above infinity; counts and ties follow it."""
    N, H = 3000, 2
    rng = np.random.default_rng(5)
    a = rng.standard_normal((1, H, N)).astype(np.float32)
    a[0, :, 10:20], a[0, :, 20:40], a[0, :, 40:60] = np.inf, -np.inf, np.nan
    a[0, 1, 100:1500] = -3.0e38
    d, da = _desc(H, N, 0, N), torch.from_numpy(a).cuda()
    u = a.view(np.uint32).astype(np.int64)
    key = np.where(u >> 31, 0xFFFFFFFF - u, u + 0x80000000)
    for b in (1, 25, 30, 700, 1600, 2985, N):
        kv = ob.omni_select_kv(d, da, torch.tensor([b], dtype=torch.int32, device="cuda"), N).cpu().numpy()
        for h in range(H):
            order = np.lexsort((np.arange(N), -key[0, h]))
            np.testing.assert_array_equal(kv[0, h, :b], np.sort(order[:b]))


@pytest.mark.parametrize("B", [64, 65])
def test_shared_budget_with_fewer_and_more_heads_than_the_search_of_all_takes(B):
    """256 heads and 260: the budgets, flattest heads and recalls of every sequence are those of the sequence alone, bit for bit."""
    H, N, rng = 4, 300, np.random.default_rng(B)
    a = torch.from_numpy(np.concatenate([_scores("lognormal", rng, H, N) for _ in range(B)])).cuda()
    q = torch.empty(B, H, N, 64, dtype=torch.bfloat16, device="cuda")
    d = ob.make_layer_desc(q, q, 0, N, 0, True)
    r = ob.omni_budget_from_scores(d, a, 0.9, 0)
    kv = ob.omni_select_kv(d, a, r.budget, N)
    one = ob.make_layer_desc(q[:1], q[:1], 0, N, 0, True)
    for b in (0, 1, B // 2, B - 1):
        s = ob.omni_budget_from_scores(one, a[b:b + 1], 0.9, 0)
        for x, y in ((r.budget, s.budget), (r.flattest, s.flattest), (r.kurtosis, s.kurtosis), (r.recall, s.recall)):
            assert torch.equal(x[b], y[0])
        n = int(s.budget[0])
        assert n == oc.budget_of(a[b, int(s.flattest[0])].cpu().numpy(), 0.9, N)
        assert torch.equal(kv[b, :, :n], ob.omni_select_kv(one, a[b:b + 1], s.budget, N)[0, :, :n])


@pytest.mark.parametrize("N", [700, 8193, 20001])
@pytest.mark.parametrize("value", [float("inf"), 3.0e38, 2.0e7, "just", "just_not"])
def test_budget_where_one_score_outweighs_the_target(N, value):
    """A score that reaches recall * N by itself is the whole budget; so it is with several of them, in every head that has one;
    the other heads' budgets do not move.  At the target exactly, and one step of the float grid below."""
    H, rng = 3, np.random.default_rng(N)
    a, p = _scores("lognormal", rng, H, N), 0.75
    target = np.float32(p * N)                          # exact in float32
    v = {"just": target, "just_not": np.nextafter(target, np.float32(0))}.get(value, value)
    d = _desc(H, N, 0, N)
    plain = ob.omni_budget_from_scores(d, torch.from_numpy(a).cuda(), p, 2).budget.cpu().numpy()
    for at in ([N // 3], [0, N // 2, N - 1]):
        b = a.copy()
        b[0, 1, at] = v
        r = ob.omni_budget_from_scores(d, torch.from_numpy(b).cuda(), p, 2).budget
        want = oc.budget_of(b[0, 1], p, N)
        assert want == (2 if value == "just_not" else 1)
        assert r[0].tolist() == [plain[0, 0], want, plain[0, 2]]
        kv = ob.omni_select_kv_per_head(d, torch.from_numpy(b).cuda(), r, N)
        assert kv[0, 1, :want].tolist()[0] in at or want == 2
        assert int(ob.omni_budget_from_scores(d, torch.from_numpy(b).cuda(), p, 1).budget[0]) == plain[0, [0, 2]].max()


@pytest.mark.parametrize("block", [1, 64])
@pytest.mark.parametrize("causal", [True, False])
def test_block_scores_with_keys_that_are_not_finite(block, causal):
    """A key at -inf on a coordinate where every query is positive has no weight in any row, and the other scores are those of
    64-bit softmaxes without it; a NaN key makes every row that sees it NaN.  700 blocks: several per thread."""
    N, H, d = 700, 2, 64
    g = torch.Generator(device="cuda").manual_seed(1)
    Q = torch.randn(1, H, N, d, generator=g, device="cuda").bfloat16()
    K = torch.randn(1, 1, N, d, generator=g, device="cuda").bfloat16()
    Q[..., 0] = Q[..., 0].abs() + 0.1
    desc = ob.make_layer_desc(Q, K, 0, N, 0, causal)
    nb = -(-N // block)
    ends = torch.arange(block, N + block, block, device="cuda").clamp(max=N)
    width = torch.diff(ends, prepend=ends.new_zeros(1)).double()
    pool = lambda x: torch.stack([x[..., j * block: (j + 1) * block, :].double().mean(-2) for j in range(nb)], -2)  # noqa: E731
    K2 = K.clone()
    K2[..., 0, 0] = -float("inf")
    z = pool(Q)[0] @ pool(K2)[0, 0].T * d ** -0.5 + width.log()
    if causal:
        z = z.masked_fill(torch.ones(nb, nb, dtype=torch.bool, device="cuda").triu(1), -float("inf"))
    first = 1 if causal else 0                                   # causal: the first row sees that key only
    want = width[first:] @ torch.softmax(z[:, first:], -1) * (nb / N)
    got = ob.omni_block_scores(desc, Q, K2, block)[0]
    if causal:
        assert bool(torch.isnan(got[:, 0]).all())                              # as the first row's softmax
        got, want = got[:, 1:], want[:, 1:]
    else:
        assert not got[:, 0].any()
    assert float((got.double() - want).abs().max()) <= 1e-4 * float(want.max())       # the key scores' bar
    K2[..., 0, 0] = float("nan")
    assert bool(torch.isnan(ob.omni_block_scores(desc, Q, K2, block)).all())


def _same_selection(x, y, lengths):
    for i, n in enumerate(lengths):
        assert torch.equal(x.scores[i, :, :n], y.scores[i, :, :n])
        assert torch.equal(x.budget.key_scores[i, :, :n], y.budget.key_scores[i, :, :n])
        assert torch.equal(x.q_idx[i, 1, : int(x.q_cnt[i, 1])], y.q_idx[i, 1, : int(x.q_cnt[i, 1])])
        assert torch.equal(x.kv_idx[i, :, : int(x.budget.budget[i])], y.kv_idx[i, :, : int(x.budget.budget[i])])
    for u, v in ((x.q_cnt, y.q_cnt), (x.budget.budget, y.budget.budget), (x.budget.recall, y.budget.recall),
                 (x.budget.kurtosis, y.budget.kurtosis), (x.probe_keys, y.probe_keys)):
        assert torch.equal(u, v)


class _ScratchFor(ob.Workspace):
    """A workspace of just the size that the library asks for a batch of `batch`, whatever the call would like."""
    def __init__(self, batch):
        super().__init__()
        self.batch = batch

    def get(self, call_id, desc, param=0):
        some = ob.LayerDesc.from_buffer_copy(desc)
        some.batch, some.vis_begin, some.vis_end = self.batch, 0, 1
        n = ob.workspace_bytes(call_id, some, param)
        self.raw = torch.empty(n + 256, dtype=torch.uint8, device="cuda")
        at = -self.raw.data_ptr() % 256
        return self.raw[at: at + n]


@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("probe_block", [32, 700])
def test_padded_batch_with_scratch_for_some_of_its_sequences_gives_the_same(batch, probe_block):
    """Three sequences on exactly the scratch that is asked for one or two (a full group and a rest), by a descriptor whose own
    visual range is a single token: the outputs of the batch in one go."""
    B, H, Hkv, N, D = 3, 4, 2, 700, 64
    g = torch.Generator(device="cuda").manual_seed(3)
    Q = torch.randn(B, H, N, D, generator=g, device="cuda").bfloat16()
    K = torch.randn(B, Hkv, N, D, generator=g, device="cuda").bfloat16()
    d = ob.make_layer_desc(Q, K, 0, 1, 0, True)
    args = ([700, 333, 40], [0, 5, 1], [690, 300, 33], 1, 0.4, 0.8, probe_block, 1)
    x, y = (ob.omni_prefill_select_varlen(d, Q, K, *args, ws=w) for w in (ob.Workspace(), _ScratchFor(batch)))
    torch.cuda.synchronize()
    _same_selection(x, y, args[0])


@pytest.mark.parametrize("mode", [0, 2])
def test_padded_batch_of_more_sequences_than_one_set_of_launches_takes(mode):
    """35 sequences: a full group of 32 and a rest of 3, each as it is alone."""
    B, H, Hkv, N, D = 35, 2, 1, 130, 64
    g = torch.Generator(device="cuda").manual_seed(4)
    Q = torch.randn(B, H, N, D, generator=g, device="cuda").bfloat16()
    K = torch.randn(B, Hkv, N, D, generator=g, device="cuda").bfloat16()
    n = [130 - 3 * b for b in range(B)]
    v1 = [max(1, x - 5) for x in n]
    x = ob.omni_prefill_select_varlen(ob.make_layer_desc(Q, K, 0, N, 0, True), Q, K, n, [0] * B, v1, 1, 0.4, 0.8, 32, mode)
    for b in (0, 1, 31, 32, 33, 34):
        q, k = Q[b:b + 1, :, :n[b]].contiguous(), K[b:b + 1, :, :n[b]].contiguous()
        y = ob.omni_prefill_select(ob.make_layer_desc(q, k, 0, v1[b], 0, True), q, k, 1, 0.4, 0.8, 32, mode)
        assert torch.equal(x.scores[b, :, :n[b]], y.scores[0]) and torch.equal(x.budget.key_scores[b, :, :n[b]], y.budget.key_scores[0])
        assert torch.equal(x.q_cnt[b], y.q_cnt[0]) and torch.equal(x.budget.budget[b], y.budget.budget[0])
        for h in range(H):
            c, m = int(y.q_cnt[0, h]), int(y.budget.budget[0, h] if mode == 2 else y.budget.budget[0])
            assert torch.equal(x.q_idx[b, h, :c], y.q_idx[0, h, :c]) and torch.equal(x.kv_idx[b, h, :m], y.kv_idx[0, h, :m])


def test_padded_batch_with_scratch_for_one_sequence_gives_the_same():
    """A workspace for one sequence takes a batch one sequence at a time: the outputs of the batch in one go."""
    B, H, Hkv, N, D = 3, 4, 2, 700, 64
    g = torch.Generator(device="cuda").manual_seed(3)
    Q = torch.randn(B, H, N, D, generator=g, device="cuda").bfloat16()
    K = torch.randn(B, Hkv, N, D, generator=g, device="cuda").bfloat16()
    d = ob.make_layer_desc(Q, K, 0, N - 9, 0, True)
    one = ob.make_layer_desc(Q[:1], K[:1], 0, N - 9, 0, True)
    args = ([700, 333, 40], [0, 5, 1], [690, 300, 33], 1, 0.4, 0.8, 32, 1)

    class Small(ob.Workspace):
        def get(self, call_id, desc, param=0):
            return super().get(call_id, one, param)

    x, y = (ob.omni_prefill_select_varlen(d, Q, K, *args, ws=w) for w in (ob.Workspace(), Small()))
    torch.cuda.synchronize()
    for i, n in enumerate(args[0]):
        assert torch.equal(x.scores[i, :, :n], y.scores[i, :, :n])
        assert torch.equal(x.budget.key_scores[i, :, :n], y.budget.key_scores[i, :, :n])
        assert torch.equal(x.q_idx[i, 1, : int(x.q_cnt[i, 1])], y.q_idx[i, 1, : int(x.q_cnt[i, 1])])
        assert torch.equal(x.kv_idx[i, :, : int(x.budget.budget[i])], y.kv_idx[i, :, : int(x.budget.budget[i])])
    for u, v in ((x.q_cnt, y.q_cnt), (x.budget.budget, y.budget.budget), (x.budget.recall, y.budget.recall),
                 (x.budget.kurtosis, y.budget.kurtosis), (x.probe_keys, y.probe_keys)):
        assert torch.equal(u, v)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [(14, 2), (2, 2)])
@pytest.mark.parametrize("N,block", [(1, 256), (40, 256), (300, 16), (300, 256), (4096, 128), (4096, 256), (4097, 256), (9000, 256)])
def test_selection_of_short_and_long_sequences_gives_what_the_separate_calls_give(N, block, heads, d, causal):
    """The launches that a short selection shares (rows and key chunks few enough; block 128 at 4096 tokens and seven heads a
    group is past the line) against the passes one by one, which keep launches of their own: bit for bit."""
    H, Hkv = heads
    g = torch.Generator(device="cuda").manual_seed(N + d)
    Q, K = (torch.randn(2, h, N, d, generator=g, device="cuda").bfloat16() for h in (H, Hkv))
    v0, v1 = (0, N) if N < 3 else (1, N - 1)
    desc = ob.make_layer_desc(Q, K, v0, v1, 0, causal)
    out = ob.omni_prefill_select(desc, Q, K, 0, 0.3, 0.9, block, 0)
    probe, scores = ob.omni_score_queries(desc, Q, K)
    b = ob.omni_kv_budget(desc, Q, K, 0.9, block, 0)
    for x, y in ((out.probe_keys, probe), (out.scores, scores), (out.budget.key_scores, b.key_scores),
                 (out.budget.budget, b.budget), (out.budget.kurtosis, b.kurtosis), (out.budget.recall, b.recall)):
        assert torch.equal(x, y)


def _same_selection_as_the_separate_calls(desc, Q, K, q_mode, q_param, recall_p, block, mode, b_cap):
    """Every output of the fused call, the lists up to their counts, against the four calls one after the other: bit for bit (the
    recall counts the keys taken, so it is compared where the capacity takes them all)."""
    H, N = desc.n_q_heads, desc.n_tokens
    out = ob.omni_prefill_select(desc, Q, K, q_mode, q_param, recall_p, block, mode, b_cap)
    probe, scores = ob.omni_score_queries(desc, Q, K)
    q_idx, q_cnt = ob.omni_select_queries(desc, scores, q_mode, q_param)
    b = ob.omni_kv_budget(desc, Q, K, recall_p, block, mode)
    kv_idx = (ob.omni_select_kv_per_head if mode == 2 else ob.omni_select_kv)(desc, b.key_scores, b.budget, b_cap)
    got = out.budget
    for x, y in ((out.probe_keys, probe), (out.scores, scores), (out.q_cnt, q_cnt), (got.key_scores, b.key_scores),
                 (got.budget, b.budget), (got.flattest, b.flattest), (got.kurtosis, b.kurtosis)):
        assert torch.equal(x, y)
    per_head = b.budget if mode == 2 else b.budget[:, None].expand(-1, H)
    assert torch.equal(got.recall[per_head <= b_cap], b.recall[per_head <= b_cap])
    at = torch.arange(N, device="cuda")
    assert torch.equal(torch.where(at < q_cnt[..., None], out.q_idx, -1), torch.where(at < q_cnt[..., None], q_idx, -1))
    listed = at[:b_cap] < per_head[..., None]
    assert torch.equal(torch.where(listed, out.kv_idx, -1), torch.where(listed, kv_idx, -1))
    return out


@pytest.mark.parametrize("cap", ["all", "few"])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("N", [300, 4096, 8192, 8193, 9000])
def test_selection_in_one_call_forms_the_lists_of_the_separate_calls(N, mode, cap):
    """The fused call takes a head's list from the cut that its own budget's search left (budgets of one head in modes 0 and 1,
    of all in mode 2; past 8192 tokens that cut lies where the list's own goes), the separate calls search it again.  Every
    key stands four times in a row, so that ties straddle the cuts, and a capacity below the budgets moves them."""
    H, Hkv, D = 6, 2, 64
    g = torch.Generator(device="cuda").manual_seed(N)
    Q = torch.randn(2, H, N, D, generator=g, device="cuda").bfloat16()
    K = torch.randn(2, Hkv, N // 4 + 1, D, generator=g, device="cuda").bfloat16().repeat_interleave(4, 2)[:, :, :N].contiguous()
    desc = ob.make_layer_desc(Q, K, 1, N - 9, 0, False)
    out = _same_selection_as_the_separate_calls(desc, Q, K, 1, 0.31, 0.83, 256, mode, N if cap == "all" else N // 3)
    if cap == "few":
        assert int(out.budget.budget.max()) > N // 3
    else:                                       # the cut stands among equal scores
        n = int(out.budget.budget.flatten()[0])
        a = out.budget.key_scores[0, 0].sort(descending=True).values
        assert n % 4 == 0 or float(a[n - 1]) == float(a[n])


@pytest.mark.parametrize("batch", [4, 5])
def test_selection_of_a_short_batch_on_both_sides_of_the_size_of_its_queries(batch):
    """Up to 2^25 elements of Q a short selection reads them twice and shares its launches (4 sequences of 14 heads, 4096
    tokens, d = 128), beyond they are read once."""
    H, Hkv, N, D = 14, 2, 4096, 128
    assert (batch * H * N * D <= 1 << 25) == (batch == 4)
    g = torch.Generator(device="cuda").manual_seed(batch)
    Q, K = (torch.randn(batch, h, N, D, generator=g, device="cuda").bfloat16() for h in (H, Hkv))
    _same_selection_as_the_separate_calls(ob.make_layer_desc(Q, K, 1, N - 1, 0, True), Q, K, 0, 0.3, 0.9, 256, 0, N)


def test_keys_of_a_vector_beyond_two_to_the_thirty_scores():
    """One head's scores are 4 bytes each: byte offsets past element 2^30 do not fit 32 bits.  Peaks and ties at the cut lie on
    both sides of it, in the last elements too."""
    N = (1 << 30) + 5001
    g = torch.Generator(device="cuda").manual_seed(0)
    a = torch.rand(1, 1, N, generator=g, device="cuda")
    at = torch.cat([torch.tensor([0, 5, (1 << 30) - 1, 1 << 30, N - 1]), torch.randint(6, N - 1, (995,)),
                    torch.randint((1 << 30) + 1, N - 1, (400,))]).unique().cuda()
    peak, tie = at[::2], at[1::2]
    a[0, 0, peak] = 2 + torch.rand(len(peak), generator=g, device="cuda")
    a[0, 0, tie] = 1.5
    n_tie = len(tie) // 2 + 1
    budget = len(peak) + n_tie
    d = _desc(1, 64, 0, 64)
    d.n_tokens = d.vis_end = N
    kv = ob.omni_select_kv(d, a, torch.tensor([budget], dtype=torch.int32, device="cuda"), budget)
    want = torch.cat([peak, tie[:n_tie]]).sort().values
    assert torch.equal(kv[0, 0].long(), want)
