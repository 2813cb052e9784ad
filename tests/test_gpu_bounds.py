"""The pass that turns the kept-query and key lists into visible counts, slots, cleared rows and work items: token counts
at the edges of its 64-token windows and 256-row items, empty and full lists, outputs that start as NaN."""
import numpy as np
import pytest
import torch

from oracle import omni_oracle as oc
from paper_2511_12201_amd import binding as ob
from paper_2511_12201_amd import synth
from tests.helpers import GRAD_RSS, bf16_ulp, grad_bar, lists_to_padded, to_device, to_host

pytestmark = pytest.mark.gpu


def _lists(rng, H, N):
    """Kept queries: all, none, one, and random shares; keys: random sets of per-head sizes 0 .. N."""
    pick = lambda n: np.sort(rng.choice(N, n, replace=False)).astype(np.int32)  # noqa: E731
    q = [np.arange(N, dtype=np.int32), pick(0), pick(1), pick(-(-N // 3))]
    k = [pick(n) for n in (-(-N // 2), N, 0, min(N, 70))]
    return [q[:H]], [k[:H]]


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("N", [1, 63, 64, 65, 255, 257, 600])
@pytest.mark.parametrize("causal", [True, False])
def test_rows_slots_and_items_at_window_edges(N, dtype, d, causal):
    H, Hkv, rng = 4, 2, np.random.default_rng(N + d)
    mk = lambda h, s=1.0: s * rng.standard_normal((1, h, N, d)).astype(np.float32)  # noqa: E731
    Q, K, V, dO = mk(H), mk(Hkv), mk(Hkv), mk(H, d ** -0.5)
    if dtype == "bf16":
        Q, K, V, dO = (synth.round_to_bf16(x) for x in (Q, K, V, dO))
    q_lists, kv_lists = _lists(rng, H, N)
    q_idx, q_cnt = lists_to_padded(q_lists, H, N)
    kv_idx, budget = lists_to_padded(kv_lists, H, N)
    tq, tk, tv, tg = (to_device(x, dtype) for x in (Q, K, V, dO))
    desc = ob.make_layer_desc(tq, tk, 0, N, 0, causal)
    nan = lambda x: torch.full_like(x, float("nan"))  # noqa: E731
    O, lse = nan(tq), torch.full((1, H, N), float("nan"), device="cuda")
    ob.omni_sparse_attn_fwd_per_head(desc, tq, tk, tv, q_idx, q_cnt, kv_idx, budget, N, O, lse)
    dQ, dK, dV = ob.omni_sparse_attn_bwd_per_head(desc, tq, tk, tv, O, tg, lse, q_idx, q_cnt, kv_idx, budget, N, nan(tq),
                                                  nan(tk), nan(tv))
    torch.cuda.synchronize()
    scale = d ** -0.5
    Oo, Lo = oc.sparse_attn_fwd(Q, K, V, q_lists, kv_lists, causal, scale)
    tol = 1e-4 if dtype == "f32" else 2e-2             # the bars of the parity tests
    assert np.max(np.abs(to_host(O) - Oo)) <= tol
    got = to_host(lse)
    np.testing.assert_array_equal(np.isfinite(got), np.isfinite(Lo))
    fin = np.isfinite(Lo)
    if fin.any():
        assert np.max(np.abs(got[fin] - Lo[fin])) <= (1e-4 if dtype == "f32" else 2e-3)
    dropped = np.ones((1, H, N), dtype=bool)
    for h in range(H):
        dropped[0, h, q_lists[0][h]] = False
    assert not to_host(O)[dropped].any() and not to_host(dQ)[dropped].any() and np.all(got[dropped] == -np.inf)
    stored = to_host(O)
    want = oc.sparse_attn_bwd(Q, K, V, dO, q_lists, kv_lists, causal, scale, O=stored)
    rss = oc.sparse_attn_bwd_term_rss(Q, K, V, dO, q_lists, kv_lists, causal, scale, O=stored)
    for x, w, r in zip((dQ, dK, dV), want, rss):
        assert np.all(np.abs(to_host(x) - w) <= grad_bar(w, dtype, r))


def _check_layer(dtype, d, N, q_lists, kv_lists, causal, backward=True):
    """Forward (and backward) of four heads on these lists against the oracle, outputs that start as NaN."""
    H, Hkv, rng = 4, 2, np.random.default_rng(N + d)
    mk = lambda h, s=1.0: s * rng.standard_normal((1, h, N, d)).astype(np.float32)  # noqa: E731
    Q, K, V, dO = mk(H), mk(Hkv), mk(Hkv), mk(H, d ** -0.5)
    if dtype == "bf16":
        Q, K, V, dO = (synth.round_to_bf16(x) for x in (Q, K, V, dO))
    q_idx, q_cnt = lists_to_padded(q_lists, H, N)
    kv_idx, budget = lists_to_padded(kv_lists, H, N)
    tq, tk, tv, tg = (to_device(x, dtype) for x in (Q, K, V, dO))
    desc = ob.make_layer_desc(tq, tk, 0, N, 0, causal)
    nan = lambda x: torch.full_like(x, float("nan"))  # noqa: E731
    O, lse = nan(tq), torch.full((1, H, N), float("nan"), device="cuda")
    ob.omni_sparse_attn_fwd_per_head(desc, tq, tk, tv, q_idx, q_cnt, kv_idx, budget, N, O, lse)
    scale = d ** -0.5
    Oo, Lo = oc.sparse_attn_fwd(Q, K, V, q_lists, kv_lists, causal, scale)
    assert np.max(np.abs(to_host(O) - Oo)) <= (1e-4 if dtype == "f32" else 2e-2)      # the bars of the parity tests
    got, fin = to_host(lse), np.isfinite(Lo)
    np.testing.assert_array_equal(np.isfinite(got), fin)
    assert np.max(np.abs(got[fin] - Lo[fin])) <= (1e-4 if dtype == "f32" else 2e-3)
    if not backward:
        return
    grads = ob.omni_sparse_attn_bwd_per_head(desc, tq, tk, tv, O, tg, lse, q_idx, q_cnt, kv_idx, budget, N, nan(tq), nan(tk),
                                             nan(tv))
    torch.cuda.synchronize()
    want = oc.sparse_attn_bwd(Q, K, V, dO, q_lists, kv_lists, causal, scale, O=to_host(O))
    rss = oc.sparse_attn_bwd_term_rss(Q, K, V, dO, q_lists, kv_lists, causal, scale, O=to_host(O))
    for x, w, r in zip(grads, want, rss):
        assert np.all(np.abs(to_host(x) - w) <= grad_bar(w, dtype, r))


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("N", [65, 600])
def test_lists_in_any_order_without_the_causal_mask(N, dtype, d):
    """Nothing has to be searched then: kept queries and keys may come in any order."""
    rng = np.random.default_rng(N)
    q_lists, kv_lists = _lists(rng, 4, N)
    mix = lambda lists: [[rng.permutation(x) for x in lists[0]]]  # noqa: E731
    _check_layer(dtype, d, N, mix(q_lists), mix(kv_lists), False)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("N", [65, 600])
@pytest.mark.parametrize("causal", [True, False])
def test_forward_on_ascending_lists_that_repeat_an_index(N, dtype, d, causal):
    """A kept query listed twice is computed twice, a key listed twice counts twice; also more repeats than a window of 64
    entries holds."""
    rng = np.random.default_rng(N)
    twice = lambda n: np.sort(rng.integers(0, N, n)).astype(np.int32)  # noqa: E731
    run = lambda n, at: np.sort(np.concatenate([np.full(n // 2, at), rng.integers(0, N, n - n // 2)])).astype(np.int32)  # noqa: E731
    q_lists = [[np.arange(N, dtype=np.int32), twice(N), run(N, N // 2), run(N // 3, 3)]]
    kv_lists = [[twice(N), run(N, N // 3), twice(N // 2), run(N, 0)]]
    _check_layer(dtype, d, N, q_lists, kv_lists, causal, backward=False)


def _hand_out_order(cost, head, queues, cus):
    """(order of the item ids, queue ends): the rule of the work list, from exact costs."""
    H, total = int(head.max()) + 1 if len(head) else 1, int(cost.sum())
    per_head = np.bincount(head, cost, minlength=H).astype(np.int64)
    if queues == 1 or H > 1024 or 2 * int(per_head.max()) * queues > 3 * total:
        return np.lexsort((np.arange(len(cost)), -cost)), np.full(8, len(cost))
    queue, pos, load, held, shift = np.zeros(H, int), np.zeros(H, int), [0] * 8, [0] * 8, 0
    while total >> shift >= 1 << 27:
        shift += 1
    for h in sorted(range(H), key=lambda x: (-per_head[x], x)):
        q = min(range(8), key=lambda r: (load[r], r))
        queue[h], pos[h] = q, held[q]
        held[q] += 1
        load[q] += int(per_head[h]) >> shift
    if 10 * total < 34 * int(cost.max()) * cus:            # long items against a CU's work: whatever their head
        pos[:] = 0
    return np.lexsort((np.arange(len(cost)), -cost, pos[head], queue[head])), np.cumsum(np.bincount(queue[head], minlength=8))


def _work_list_lists(kind, rng):
    """(N, kept queries and keys per head)."""
    pick = lambda N, n: np.sort(rng.choice(N, n, replace=False)).astype(np.int32)  # noqa: E731
    if kind == "edges":                                      # counts around one and several items, empty heads, empty key lists
        N = 1100
        return N, [pick(N, n) for n in (N, 0, 1, 127, 128, 129, 255, 256, 257, 0, 512, 513)], \
            [pick(N, n) for n in (600, 5, 0, N, 64, 65, 1, 700, 333, 0, 2, N)]
    if kind == "even":                                       # no head outweighs a queue
        N = 2000
        return N, [pick(N, 600 + 13 * h) for h in range(24)], [pick(N, 900 - h) for h in range(24)]
    if kind == "long":                                       # the work of a CU is several longest items: head after head
        N = 65536
        return N, [np.arange(N, dtype=np.int32)] + [pick(N, 21000 + 11 * h) for h in range(27)], [pick(N, 35000)] * 28
    if kind == "hundreds":                                   # as many heads as a large batch has, of very different lengths
        N = 2100
        return N, [pick(N, int(n)) for n in rng.integers(0, N + 1, 900)], [pick(N, 1 + 2 * h) for h in range(900)]
    N = 300                                                  # "many": more heads than queues place
    return N, [pick(N, int(n)) for n in rng.integers(0, N + 1, 1100)], [pick(N, 200)] * 1100


@pytest.mark.parametrize("kind", ["edges", "even", "long", "hundreds", "many"])
@pytest.mark.parametrize("queues", [1, 8])
@pytest.mark.parametrize("tile_rows", [128, 256])
@pytest.mark.parametrize("causal", [True, False])
def test_work_list_of_the_device(kind, queues, tile_rows, causal):
    """Items, costs and hand-out order that the device builds from index lists: those of the rule replayed from exact counts."""
    N, q, k = _work_list_lists(kind, np.random.default_rng(7))
    H, cap = len(q), max(1, max(len(x) for x in k))
    q_idx, q_cnt = lists_to_padded([q], H, N)
    kv_idx, budget = lists_to_padded([k], H, cap)
    desc = ob.LayerDesc(batch=1, n_q_heads=H, n_kv_heads=H, head_dim=64, n_tokens=N, vis_begin=0, vis_end=N, sink_index=0,
                        causal=int(causal), dtype=ob.OMNI_BF16, softmax_scale=0.125, q_stride=(H * N * 64, N * 64, 64),
                        kv_stride=(H * N * 64, N * 64, 64))
    items, order, starts, ends = ob.debug_device_work_list(desc, q_idx, q_cnt, kv_idx, budget, tile_rows, queues)
    head, tile, cost = [], [], []
    for h in range(H):
        for t in range(-(-len(q[h]) // tile_rows)):
            last = q[h][min((t + 1) * tile_rows, len(q[h])) - 1]
            seen = np.searchsorted(k[h], last, side="right") if causal else len(k[h])
            head.append(h), tile.append(t), cost.append(-(-int(seen) // 64))
    packed, cost, head = np.array(head) << 16 | np.array(tile), np.array(cost), np.array(head)
    np.testing.assert_array_equal(items[:, 0], packed)
    np.testing.assert_array_equal(items[:, 1], cost)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    by, at = _hand_out_order(cost, head, queues, cus)
    np.testing.assert_array_equal(order, packed[by])
    np.testing.assert_array_equal(ends, at)
    np.testing.assert_array_equal(starts, np.concatenate([[0], at[:-1]]))


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d", [64, 128])
def test_forward_on_both_sides_of_the_short_sequence_rule(d, causal, full):
    """Shapes just below and just above the line between the two bf16 forward kernels (batch * heads * N^2 * d, twice
    that without the mask, against 6.5e10), on the same random lists, or on lists of everything; a whole number of 32-row
    items and one row more."""
    H, Hkv, B = 16, 1, 8
    line = int((6.5e10 / (B * H * d * (1 if causal else 2))) ** 0.5)
    for N in (line // 32 * 32, line // 32 * 32 + 33):
        rng = np.random.default_rng(N)
        g = torch.Generator(device="cuda").manual_seed(N)
        rand = lambda h: torch.randn(B, h, N, d, generator=g, device="cuda").bfloat16()  # noqa: E731
        Q, K, V = rand(H), rand(Hkv), rand(Hkv)
        desc = ob.make_layer_desc(Q, K, 0, N, 0, causal)
        sizes = [(N, N)] * 4 if full else [(N, 65), (N // 5, N // 3), (33, N), (31, 1)]
        q_lists = [[np.sort(rng.choice(N, sizes[h % 4][0], replace=False)) for h in range(H)] for _ in range(B)]
        k_lists = [[np.sort(rng.choice(N, sizes[h % 4][1], replace=False)) for h in range(H)] for _ in range(B)]
        q_idx, q_cnt = lists_to_padded(q_lists, H, N)
        kv_idx, budget = lists_to_padded(k_lists, H, N)
        O, lse = ob.omni_sparse_attn_fwd_per_head(desc, Q, K, V, q_idx, q_cnt, kv_idx, budget, N)
        for b, h in ((0, 0), (B - 1, 1), (3, 2), (5, 3)):
            q, k = torch.from_numpy(q_lists[b][h]).cuda(), torch.from_numpy(k_lists[b][h]).cuda()
            z = Q[b, h, q].double() @ K[b, 0, k].double().T * d ** -0.5
            if causal:
                z = z.masked_fill(k[None] > q[:, None], -float("inf"))
            want = torch.nan_to_num(torch.softmax(z, -1)) @ V[b, 0, k].double()
            assert float((O[b, h, q].double() - want).abs().max()) <= 2e-2
            m = torch.logsumexp(z, -1)
            fin = torch.isfinite(m)
            assert torch.equal(torch.isfinite(lse[b, h, q]), fin)
            assert float((lse[b, h, q][fin] - m[fin]).abs().max()) <= 2e-3


def _check_block_and_list_gradients(B, H, N, d, causal, full, block=64):
    """Block lists in place give the bits of their token lists, and the gradients of the first and the last sequence are those
    of 64-bit sums over the listed pairs."""
    rng = np.random.default_rng(N + d)
    g = torch.Generator(device="cuda").manual_seed(N)
    rand = lambda h, s=1.0: (s * torch.randn(B, h, N, d, generator=g, device="cuda")).bfloat16()  # noqa: E731
    Q, K, V, dO = rand(H), rand(1), rand(1), rand(H, d ** -0.5)
    desc = ob.make_layer_desc(Q, K, 0, N, 0, causal)
    nb = N // block
    nsel = nb if full else nb // 3
    blocks = [[np.sort(rng.choice(nb, nsel, replace=False)) for _ in range(H)] for _ in range(B)]
    kept = (N, N, N, N) if full else (N, N // 5, 33, 31)
    rows = [[np.sort(rng.choice(N, kept[h % 4], replace=False)) for h in range(H)] for _ in range(B)]
    q_idx, q_cnt = lists_to_padded(rows, H, N)
    blk_idx, _ = lists_to_padded(blocks, H, nb)
    blk_budget = torch.full((B,), nsel, dtype=torch.int32, device="cuda")
    kv_idx, budget = ob.omni_expand_blocks(desc, blk_idx, blk_budget, block)
    O, lse = ob.omni_block_attn_fwd(desc, Q, K, V, q_idx, q_cnt, blk_idx, blk_budget, block)
    O2, lse2 = ob.omni_sparse_attn_fwd(desc, Q, K, V, q_idx, q_cnt, kv_idx, budget, kv_idx.shape[-1])
    assert torch.equal(O, O2) and torch.equal(lse, lse2)
    got = ob.omni_block_attn_bwd(desc, Q, K, V, O, dO, lse, q_idx, q_cnt, blk_idx, blk_budget, block)
    got2 = ob.omni_sparse_attn_bwd(desc, Q, K, V, O, dO, lse, q_idx, q_cnt, kv_idx, budget, kv_idx.shape[-1])
    for x, y in zip(got, got2):
        assert torch.equal(x, y)
    for b in {0, B - 1}:
        k64, v64 = K[b, 0].double(), V[b, 0].double()
        want = [torch.zeros(H, N, d, dtype=torch.float64, device="cuda")] + [torch.zeros_like(k64) for _ in range(2)]
        rss = [torch.zeros_like(x) for x in want]
        for h in range(H):
            q = torch.from_numpy(rows[b][h]).cuda()
            k = (torch.from_numpy(blocks[b][h]).cuda()[:, None] * block + torch.arange(block, device="cuda")).flatten()
            z = Q[b, h, q].double() @ k64[k].T * d ** -0.5
            if causal:
                z = z.masked_fill(k[None] > q[:, None], -float("inf"))
            P = torch.nan_to_num(torch.softmax(z, -1))
            go = dO[b, h, q].double()
            dS = P * (go @ v64[k].T - (go * O[b, h, q].double()).sum(-1, keepdim=True)) * d ** -0.5
            for out, f in ((want, lambda x: x), (rss, torch.square)):
                out[0][h, q] = f(dS) @ f(k64[k])
                out[1][k] += f(dS).T @ f(Q[b, h, q].double())
                out[2][k] += f(P).T @ f(go)
        for x, w, r in zip((got[0][b], got[1][b, 0], got[2][b, 0]), want, rss):
            ulp = torch.from_numpy(bf16_ulp(w.cpu().numpy())).cuda()
            bar = torch.clamp(GRAD_RSS * r.sqrt() + 0.5 * ulp, min=2e-2)      # grad_bar
            assert bool(((x.double() - w).abs() <= bar).all())


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d", [64, 128])
def test_gradients_on_both_sides_of_the_short_sequence_rules(d, causal, full):
    """The backward on either forward's output: shapes just below and just above the line between the forward kernels
    (6.5e10), and at sizes below it (4.0e10)."""
    H, B, block = 16, 4, 64
    for line in (4.0e10, 6.5e10):
        N0 = int((line / (B * H * d * (1 if causal else 2))) ** 0.5) // block * block
        for N in (N0, N0 + block):
            _check_block_and_list_gradients(B, H, N, d, causal, full)


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,H,N,d", [(1, 8, 3200, 128), (1, 8, 3264, 128), (2, 4, 4992, 64), (2, 4, 5056, 64), (1, 9, 64, 128),
                                     (3, 3, 64, 64), (1, 1, 64, 64), (1, 2, 8256, 128)])
def test_gradients_on_both_sides_of_the_few_row_rule(B, H, N, d, causal, full):
    """Eight heads and 26000 rows of d = 128, 40000 of d = 64: below, the dQ items are 32 rows whose wavefronts share the keys,
    above (more rows, or more heads) 256 rows."""
    _check_block_and_list_gradients(B, H, N, d, causal, full)


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("kept", [1, 64, 513, 2049])
def test_key_gradients_when_a_few_long_key_tiles_are_split(kept):
    """One head keeps every query (its key tiles are shared between workgroups), the others few: dK and dV of the split
    tiles against 64-bit sums, at counts around whole query tiles and splits."""
    H, Hkv, N, d = 4, 1, 2304, 64
    g = torch.Generator(device="cuda").manual_seed(kept)
    rand = lambda h, s=1.0: (s * torch.randn(1, h, N, d, generator=g, device="cuda")).bfloat16()  # noqa: E731
    Q, K, V, dO = rand(H), rand(Hkv), rand(Hkv), rand(H, d ** -0.5)
    rng = np.random.default_rng(kept)
    q_lists = [[np.arange(N)] + [np.sort(rng.choice(N, kept, replace=False)) for _ in range(H - 1)]]
    k_lists = [[np.sort(rng.choice(N, n, replace=False)) for n in (1500, 257, 1, 700)]]
    q_idx, q_cnt = lists_to_padded(q_lists, H, N)
    kv_idx, budget = lists_to_padded(k_lists, H, N)
    desc = ob.make_layer_desc(Q, K, 0, N, 0, True)
    O, lse = ob.omni_sparse_attn_fwd_per_head(desc, Q, K, V, q_idx, q_cnt, kv_idx, budget, N)
    got = ob.omni_sparse_attn_bwd_per_head(desc, Q, K, V, O, dO, lse, q_idx, q_cnt, kv_idx, budget, N)
    torch.cuda.synchronize()
    args = [to_host(x) for x in (Q, K, V, dO)] + [q_lists, k_lists, True, d ** -0.5]
    want = oc.sparse_attn_bwd(*args, O=to_host(O))
    rss = oc.sparse_attn_bwd_term_rss(*args, O=to_host(O))
    for x, w, r in zip(got, want, rss):
        assert np.all(np.abs(to_host(x) - w) <= grad_bar(w, "bf16", r))


@pytest.mark.usefixtures("attention_route")
@pytest.mark.parametrize("dtype,d", [("bf16", 64), ("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("N", [64, 65, 300])
def test_what_the_scratch_held_before_does_not_show(N, dtype, d):
    """The slot map is written for listed tokens only: whatever the scratch says of the others, slots in range among it, their
    gradients are zero and all others the same to the last bit."""
    rng = np.random.default_rng(N)
    q_lists, kv_lists = _lists(rng, 4, N)
    g = torch.Generator(device="cuda").manual_seed(N)
    rand = lambda h, s=1.0: to_device((s * torch.randn(1, h, N, d, generator=g, device="cuda")).cpu().numpy(), dtype)  # noqa: E731
    Q, K, V, dO = rand(4), rand(2), rand(2), rand(4, d ** -0.5)
    desc = ob.make_layer_desc(Q, K, 0, N, 0, True)
    q_idx, q_cnt = lists_to_padded(q_lists, 4, N)
    kv_idx, budget = lists_to_padded(kv_lists, 4, N)
    lists, results = (q_idx, q_cnt, kv_idx, budget, N), []
    for fill in (0, 1, -1, None):
        ws = ob.Workspace()
        for call in (ob.CALL_SPARSE_ATTN_FWD, ob.CALL_SPARSE_ATTN_BWD):
            words = ws.get(call, desc, N)
            words = words[:words.numel() // 4 * 4].view(torch.int32)
            words.copy_(torch.arange(len(words), device="cuda") % N if fill is None else torch.full_like(words, fill))
        O, lse = ob.omni_sparse_attn_fwd_per_head(desc, Q, K, V, *lists, ws=ws)
        results.append((O, lse, *ob.omni_sparse_attn_bwd_per_head(desc, Q, K, V, O, dO, lse, *lists, ws=ws)))
    for other in results[1:]:
        assert all(torch.equal(x, y) for x, y in zip(results[0], other))
    for group, x in ((g, x) for x in results[0][3:] for g in range(2)):
        unlisted = np.setdiff1d(np.arange(N), np.concatenate(kv_lists[0][2 * group:2 * group + 2]))
        assert not x[0, group, torch.from_numpy(unlisted).cuda()].any()
