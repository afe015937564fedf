"""Routes that a call takes by its sizes give the results of the general ones (GPU)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2509_00388_amd import binding as gk
from tests.test_gpu_parity import key_order, rows_with_nan

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)


def select_scratch(p):
    cp = p.c()
    return int(gk.load_library().graphkv_select_workspace_bytes(ctypes.byref(cp)))


# (a segment is 8192 entries: rows that fill their last one, that leave one entry for it, the longest row)
@pytest.mark.parametrize("P,k", [(32769, 1), (40960, 40959), (40961, 2000), (131008, 32768), (1 << 18, 4000)])
def test_long_rows_shared_out(P, k):
    """The budgeted selection of few long rows by many workgroups, against one workgroup a row (which is what
    a call without workspace takes) and against the order of the keys."""
    say(f"selection shared out P={P} k={k}")
    rng = np.random.default_rng(P + k)
    w = 3
    s = rows_with_nan(P, k, P ^ k)
    s = np.concatenate([s, rng.standard_normal((5, P)).astype(np.float32)])
    s[10, ::3] = 0.0
    s[10, 1::3] = -0.0
    s[11] = rng.integers(0, 40, P)                                  # ties in every segment
    s[12, rng.choice(P, size=min(P, k + 5), replace=False)] = 9.0   # the cut among equal values
    s[13] = 1.0 + np.arange(P, dtype=np.float32) * np.float32(1e-7)  # neighbouring values, all in few bins
    s = s[:max(1, 256 // -(-P // 8192))]
    H = s.shape[0]
    p = gk.Params(n_kv_heads=H, n_q_heads=H, head_dim=8, n_tokens=P + w, window=w, budget=k + w)
    assert select_scratch(p) > 0
    x = torch.from_numpy(s).cuda()
    none = torch.empty(256, dtype=torch.uint8, device="cuda")
    one = gk.graphkv_select(p, x, torch.full((H, k + w), -7, dtype=torch.int32, device="cuda"), none).cpu().numpy()
    for _ in range(2):
        ws = torch.randint(0, 256, (select_scratch(p),), dtype=torch.uint8, device="cuda")
        idx = gk.graphkv_select(p, x, torch.full((H, k + w), -7, dtype=torch.int32, device="cuda"), ws).cpu().numpy()
        assert np.array_equal(idx, one)
    for h in range(H):
        assert np.array_equal(idx[h, :k], key_order(s[h], k)), f"row {h}"
        assert np.array_equal(idx[h, k:], np.arange(P, P + w))


def test_long_rows_shared_out_in_a_whole_pass():
    """A layer of a long prompt: its final selection is shared out, that of the same layer in a batch whose heads
    fill the chip is not."""
    say("whole pass with a long row, alone and in a batch")
    L, H, N, d, w, B = 65, 4, 33000, 8, 4, 700
    g = torch.Generator("cuda").manual_seed(5)
    K = torch.randn(L, H, N, d, generator=g, device="cuda")
    V = torch.randn(L, H, N, d, generator=g, device="cuda")
    p = gk.Params(n_kv_heads=H, n_q_heads=H, head_dim=d, n_tokens=N, window=w, budget=B, dtype=gk.FP32,
                  scorer=gk.SCORER_KNORM)
    Ks, Vs, idx = gk.graphkv_compress_batched(p, L, None, K, V, None)
    for l in (0, L - 1):
        K1, V1, i1 = gk.graphkv_compress(p, K[l], V[l], None)
        at = slice(l * H * B, (l + 1) * H * B)
        assert torch.equal(i1.flatten(), idx[at])
        assert torch.equal(K1.view(-1, d), Ks[at]) and torch.equal(V1.view(-1, d), Vs[at])
        ref = K[l, :, :N - w].double().norm(dim=2).neg().topk(B - w, dim=1).indices.sort(dim=1).values
        assert (i1[:, :B - w] == ref).float().mean() > 0.99


# (an update of up to 4096 triples rides along with the next selection, a larger one does not; more than 256 sources are
# matched in a launch of their own; 300 neighbours are more than the quick selection of a redone row takes)
@pytest.mark.parametrize("N,S,m,signal", [(8300, 64, 32, 0), (8224, 40, 90, 0), (9000, 64, 16, 1), (16416, 20, 200, 2),
                                          (8300, 64, 80, 0), (8300, 300, 8, 2), (33100, 8, 300, 0), (33100, 16, 24, 0)])
@pytest.mark.parametrize("T", [1, 3])
def test_redone_heads_in_few_and_in_many(N, S, m, signal, T):
    """Layers in which one head's candidate lists overflow for certain: half of its keys are one vector, of the lowest
    norm, so that they are the sources and every list has thousands of equal edges.  Which nodes it keeps is known:
    the sources' neighbours are the m lowest of those nodes (m + 1 with the sources that are among them), and what
    is left of them, lowest first, is best.  The same with the head's layer alone, and for the other heads."""
    say(f"redone heads, few and many N={N} S={S} m={m} signal={signal} T={T}")
    L, H, d, w, B = 40, 3, 128, 32, 300
    P = N - w
    g = torch.Generator("cuda").manual_seed(N + S)
    K = torch.randn(L, H, N, d, generator=g, device="cuda")
    same = torch.rand(L, P, generator=g, device="cuda") < 0.5
    same[:, 0] = True
    K[:, 1, :P] = torch.where(same[..., None], 0.25 * K[:, 1, :1], K[:, 1, :P])
    kind = torch.randint(0, 64, (L, N), generator=g, device="cuda")
    K[:, 2] = 0.4 * K[:, 2] + torch.randn(L, 64, d, generator=g, device="cuda").gather(1, kind[..., None].expand(-1, -1, d))
    K = K.to(torch.bfloat16)
    V = torch.randn(L, H, N, d, generator=g, device="cuda").to(torch.bfloat16)
    p = gk.Params(n_kv_heads=H, n_q_heads=H, head_dim=d, n_tokens=N, window=w, budget=B, n_sources=S, n_neighbors=m,
                  rounds=T, signal=signal, scorer=gk.SCORER_KNORM)

    def batch(K):
        sc = torch.empty(L, H, P, device="cuda")
        gk.graphkv_profile_begin()
        out = gk.graphkv_compress_batched(p, L, None, K, V, None, scores_out=sc)
        torch.cuda.synchronize()
        return out, sc, gk.graphkv_profile_end()["redo_rows"]

    plain = K[:, :1].expand(-1, H, -1, -1).contiguous()
    batch(plain)
    nothing = batch(plain)[2]
    (Ks, Vs, idx), sc, redone = batch(K)
    assert redone[1] == nothing[1] == T and redone[0] > 4 * nothing[0], (redone, nothing)
    generic = gk.Params(**{**p.__dict__, "impl": gk.IMPL_GENERIC})
    for l in (0, 7, L - 1):
        s1, s2 = (torch.empty(H, P, device="cuda") for _ in range(2))
        K1, V1, i1 = gk.graphkv_compress(p, K[l], V[l], None, scores_out=s1)
        at = slice(l * H * B, (l + 1) * H * B)
        assert torch.equal(i1.flatten(), idx[at]) and torch.equal(s1, sc[l])
        assert torch.equal(K1.view(-1, d).view(torch.int16), Ks[at].view(torch.int16))
        if signal != 1:   # (an enhanced signal keeps the neighbours instead)
            left = same[l].nonzero().flatten()[m + 1:]
            assert torch.equal(i1[1, :B - w].long(), left[:B - w])
            assert torch.equal(V1[1, :B - w].view(torch.int16), V[l, 1][left[:B - w]].view(torch.int16))
        # the scalar kernels, whose edges round otherwise: the same nodes but for near-ties
        _, _, i2 = gk.graphkv_compress(generic, K[l], V[l], None, scores_out=s2)
        for h in range(H):
            assert len(set(i1[h].tolist()) ^ set(i2[h].tolist())) <= 4, f"layer {l} head {h}"
        assert torch.isclose(s1, s2, rtol=1e-3, atol=0.0).float().mean() > 0.99   # (evicted nodes: equal infinities)


# (rows of 16 bytes, of exactly 128, of a little more, of exactly 256, of several pieces and a rest)
@pytest.mark.parametrize("fp32,d", [(0, 8), (0, 64), (0, 72), (1, 32), (1, 40), (1, 64), (1, 168), (0, 200)])
@pytest.mark.parametrize("G,w,S", [(1, 16, 5), (2, 24, 40), (4, 33, 70)])
def test_tiled_products_by_row_length(fp32, d, G, w, S):
    """Scores and edges of the tiled matrix products against 64 bits for every length of a row that is staged
    differently, with one, two and four row blocks and tiles that end in the middle."""
    say(f"tiled products fp32={fp32} d={d} rows={G * w} S={S}")
    H, N = 2, 777
    g = torch.Generator("cuda").manual_seed(100 * d + S)
    td = torch.float32 if fp32 else torch.bfloat16
    K = torch.randn(H, N, d, generator=g, device="cuda").to(td)
    Q = torch.randn(H * G, w, d, generator=g, device="cuda").to(td)
    P = N - w
    p = gk.Params(n_kv_heads=H, n_q_heads=H * G, head_dim=d, n_tokens=N, window=w, pool_kernel=5, budget=w + 1, n_sources=S,
                  n_neighbors=P - 1, rounds=1, dtype=gk.FP32 if fp32 else gk.BF16)
    sc = gk.graphkv_score(p, K, Q)
    l = (Q.double().view(H, G * w, d) @ K.double().transpose(1, 2).contiguous()) / d ** 0.5
    hidden = torch.arange(N, device="cuda")[None] > (P + torch.arange(w, device="cuda").repeat(G))[:, None]
    votes = l.masked_fill(hidden, -torch.inf).softmax(2)[:, :, :P].sum(1)
    ref = torch.nn.functional.avg_pool1d(votes[:, None], 5, 1, 2)[:, 0] / G
    # 32-bit logits of size up to |l| are off by 2e-7 |l| d^0.5 at most, their exponentials by as much
    assert ((sc - ref).abs() <= 2e-5 * ref).all()
    src = torch.empty(1, H, S, dtype=torch.int32, device="cuda")
    nbr = torch.empty(1, H, S, P - 1, dtype=torch.int32, device="cuda")
    e = torch.empty(1, H, S, P - 1, device="cuda")
    gk.graphkv_propagate(p, K, sc.clone(), src, nbr, e)
    Kn = torch.nn.functional.normalize(K[:, :P].double(), dim=2)
    for h in range(H):   # m = P - 1: every edge but a source's own
        full = Kn[h][src[0, h].long()] @ Kn[h].T
        assert ((full.gather(1, nbr[0, h].long()) - e[0, h]).abs() <= 2e-5).all()


@pytest.mark.parametrize("P,B,fp32,d", [(900, 256, 0, 128), (900, 257, 0, 128), (3000, 128, 1, 128), (3000, 129, 1, 128),
                                        (40, 7, 0, 8), (32768, 4096, 0, 8), (32768, 4097, 0, 8), (32769, 100, 0, 8)])
def test_few_retained_rows_are_gathered_by_the_selection(P, B, fp32, d):
    """Heads with up to 64 KiB of retained rows are copied by the workgroup that selected them: both sides of that
    limit, of the row length up to which the kernel serves, and budgets that differ from layer to layer."""
    say(f"gather by the selection P={P} B={B} fp32={fp32} d={d}")
    L, H, w = 3, 2, 3
    N = P + w
    budgets = [B, max(w + 1, B - 3), max(w + 1, B // 2)]
    g = torch.Generator("cuda").manual_seed(P + B)
    td = torch.float32 if fp32 else torch.bfloat16
    K, V = (torch.randn(L, H, N, d, generator=g, device="cuda").to(td) for _ in range(2))
    p = gk.Params(n_kv_heads=H, n_q_heads=H, head_dim=d, n_tokens=N, window=w, budget=B, n_sources=3, n_neighbors=2,
                  rounds=1, dtype=gk.FP32 if fp32 else gk.BF16, scorer=gk.SCORER_KNORM)
    Ks, Vs, idx = gk.graphkv_compress_batched(p, L, budgets, K, V, None)
    row = 0
    for l, b in enumerate(budgets):
        for h in range(H):
            i = idx[row:row + b].long()
            assert (i[1:] > i[:-1]).all() and torch.equal(i[-w:], torch.arange(P, N, device="cuda"))
            assert torch.equal(Ks[row:row + b], K[l, h][i]) and torch.equal(Vs[row:row + b], V[l, h][i])
            row += b


@pytest.mark.parametrize("H,N,S,scorer", [(8, 16384, 64, 1), (8, 16384, 192, 1), (8, 32768, 128, 1), (8, 16384, 192, 0)])
def test_new_lists_of_later_rounds_cost_no_more_than_the_first(H, N, S, scorer):
    """Few heads whose sources are exchanged from round to round (key norms lie close together; more sources than
    are promoted): a later round's bound, filter and select passes take no longer than those of the first round,
    which are over all sources (and half as much again for what a clock shows; selected from by one workgroup a
    head they took three times as long), whether they are one launch or several."""
    say(f"new lists of later rounds H={H} N={N} S={S} scorer={scorer}")
    d, w, T = 128, 32, 3
    g = torch.Generator("cuda").manual_seed(S)
    centre = torch.randn(H, 256, d, generator=g, device="cuda")
    kind = torch.randint(0, 256, (H, N, 1), generator=g, device="cuda").expand(-1, -1, d)
    K = centre.gather(1, kind) + 0.3 * torch.randn(H, N, d, generator=g, device="cuda")
    K[:, :, :4] *= 8.0
    K = K.to(torch.bfloat16)
    Q = (0.5 * K[:, :w] + torch.randn(H, w, d, generator=g, device="cuda")).to(torch.bfloat16)
    p = gk.Params(n_kv_heads=H, n_q_heads=H, head_dim=d, n_tokens=N, window=w, budget=w + 500, n_sources=S, n_neighbors=32,
                  rounds=T, scorer=scorer, dtype=gk.BF16)
    first = later = np.inf
    for _ in range(4):
        gk.graphkv_profile_begin()
        gk.graphkv_compress(p, K, K, Q)
        torch.cuda.synchronize()
        took = gk.graphkv_profile_end()

        def ms(*kernels):
            return sum(took[k][0] for k in kernels if k in took)   # (bound and filter may be one launch)

        first = min(first, ms("cosine_bound", "cosine_filter", "nbr_select"))
        later = min(later, ms("cosine_bound_new", "cosine_filter_new", "nbr_select_later") / (T - 1))
    say(f"  first round {first:.3f} ms, a later one {later:.3f} ms")
    assert later < 1.5 * first + 0.01


@pytest.mark.parametrize("P,S,m", [(152, 152, 20), (300, 100, 40), (900, 128, 30)])
def test_update_in_front_of_the_selection_takes_long_chains(P, S, m):
    """Few nodes that many sources reach, up to 4096 triples: the update that the final selection does first takes
    no longer than the update and the selection of their own (and a fifth more for what a clock shows; with the ends
    of the chains several to a thread it took half as much again)."""
    say(f"long chains P={P} S={S} m={m}")
    H, w, d = 4, 32, 128
    g = torch.Generator("cuda").manual_seed(P)
    K = torch.randn(H, P + w, d, generator=g, device="cuda").to(torch.bfloat16)
    p = gk.Params(n_kv_heads=H, n_q_heads=H, head_dim=d, n_tokens=P + w, window=w, budget=w + P // 2, n_sources=S, n_neighbors=m,
                  rounds=1, scorer=gk.SCORER_KNORM)
    s = gk.graphkv_score_knorm(p, K)
    both = update = select = np.inf
    for _ in range(6):
        gk.graphkv_profile_begin()
        kept = gk.graphkv_compress(p, K, K, None)[2]
        torch.cuda.synchronize()
        both = min(both, gk.graphkv_profile_end()["topk_final"][0])
        gk.graphkv_profile_begin()
        alone = gk.graphkv_select(p, gk.graphkv_propagate(p, K, s.clone()))
        torch.cuda.synchronize()
        took = gk.graphkv_profile_end()
        update, select = min(update, took["decay"][0]), min(select, took["topk_final"][0])
    say(f"  together {1e3 * both:.1f} us, update {1e3 * update:.1f}, selection {1e3 * select:.1f}")
    assert torch.equal(kept, alone)
    assert both < 1.2 * (update + select)


# (row groups of 32 per workgroup: one and two in a single round, three with the next-ranked nodes along, two workgroups of
# three; the last key block short, or starting early at the end of the head; keys beyond 256 MiB, which stay out of the caches)
@pytest.mark.parametrize("P,w,S,m,T,H", [(2080, 1, 32, 4, 1, 128), (2175, 5, 33, 9, 1, 128), (4097, 1, 64, 32, 2, 36),
                                         (8191, 32, 129, 20, 2, 8), (2049, 63, 65, 16, 2, 64), (2050, 2, 8, 5, 1, 512),
                                         # bounds put together from 10, 8, 6 and 3 parts of the sample, in the filter pass
                                         # (a head a workgroup), of the last rank taken from maxima and of the first counted
                                         (8190, 1, 96, 32, 1, 12), (8191, 1, 65, 7, 1, 16), (4099, 3, 100, 64, 3, 24),
                                         (2100, 4, 128, 32, 1, 40), (2200, 4, 40, 32, 2, 260), (8190, 1, 40, 133, 1, 28),
                                         (8190, 1, 40, 134, 1, 28), (8190, 1, 40, 134, 2, 280)])
def test_filter_pass_row_groups_and_key_blocks(P, w, S, m, T, H):
    """The filter pass against the dense edge block, bit for bit: many heads take the one, the same heads alone the
    other.  Among the sources a zero key; among the nodes zero keys, keys of norms that leave the range of the matrix
    cores' test of the bounds, keys close to all sources of a kind, blocks in which every key is a candidate."""
    say(f"filter pass P={P} w={w} S={S} m={m} T={T} H={H}")
    d, few, N = 128, 4, P + w
    assert H * S * P >= 1 << 23 > few * S * P
    g = torch.Generator("cuda").manual_seed(P + S)
    kind = torch.randint(0, 16, (few, N, 1), generator=g, device="cuda")
    cent = torch.randn(few, 16, d, generator=g, device="cuda")
    K = cent.gather(1, kind.expand(-1, -1, d)) + 0.7 * torch.randn(few, N, d, generator=g, device="cuda")
    K[:, 64:96] = cent[:, 3:4] + 0.05 * torch.randn(few, 32, d, generator=g, device="cuda")
    s = torch.rand(few, P, generator=g, device="cuda") + 0.1
    K[1, P - 1] = 0.0
    K[1, 7] = 0.0
    s[1, 7] = 5.0                                                   # a source all of whose edges are 0
    for j, norm in ((100, 1e-18), (101, 1e18), (102, 3e17), (P - 2, 1e-12), (P - 3, 1e12)):
        K[2, j] *= norm / 10.0
        s[2, j] = 3.0 if j == 102 else s[2, j]
    K = K.to(torch.bfloat16)
    rep = -(-H // few)
    kw = dict(head_dim=d, n_tokens=N, window=w, n_sources=S, n_neighbors=m, rounds=T)

    def run(heads, K, s):
        p = gk.Params(n_kv_heads=heads, n_q_heads=heads, **kw)
        dbg = [torch.full((T, heads, S, n) if n else (T, heads, S), -1, dtype=t, device="cuda")
               for n, t in ((0, torch.int32), (m, torch.int32), (m, torch.float32))]
        out = gk.graphkv_propagate(p, K, s.clone(), *dbg)
        return (out, *dbg)

    dense = run(few, K, s)
    many = run(rep * few, K.repeat(rep, 1, 1), s.repeat(rep, 1))
    assert torch.equal(many[0].view(rep, few, P), dense[0].expand(rep, -1, -1))
    for a, b in zip(many[1:], dense[1:]):
        assert torch.equal(a.view(T, rep, *b.shape[1:]), b[:, None].expand(-1, rep, *[-1] * (b.dim() - 1)))


# (row groups of 32 that sources fill in part: 1, 31 and 8 rows of the last one are no source's)
@pytest.mark.parametrize("P,S,m,H", [(4200, 63, 8, 64), (4200, 33, 20, 64), (8191, 88, 4, 16)])
def test_filter_pass_with_mostly_zero_keys(P, S, m, H):
    """Edges to zero keys and of zero sources are 0, whichever route forms them, and ties go to the lowest index: heads
    with little more than m keys that are not 0, with half of them 0, and beside a head with an infinite key (whose
    lists have no agreed order, but stay its own)."""
    say(f"mostly zero keys P={P} S={S} m={m} H={H}")
    d, few, N = 128, 4, P + 2
    assert H * S * P >= 1 << 23 > few * S * P
    g = torch.Generator("cuda").manual_seed(P + S)
    K = torch.randn(few, N, d, generator=g, device="cuda")
    s = torch.rand(few, P, generator=g, device="cuda") + 0.1
    K[0, : P - m - 20] = 0.0                     # the others lie behind the zero keys, which win the ties
    s[0, P - m - 20:] += 1.0
    K[1, torch.rand(N, generator=g, device="cuda") < 0.5] = 0.0
    K[3, 1000] = torch.inf
    K = K.to(torch.bfloat16)
    rep = H // few
    kw = dict(head_dim=d, n_tokens=N, window=2, n_sources=S, n_neighbors=m, rounds=1)

    def run(heads, K, s):
        p = gk.Params(n_kv_heads=heads, n_q_heads=heads, **kw)
        dbg = [torch.full((heads, S, n) if n else (heads, S), -1, dtype=t, device="cuda")
               for n, t in ((0, torch.int32), (m, torch.int32), (m, torch.float32))]
        out = gk.graphkv_propagate(p, K, s.clone(), *dbg)
        return (out, *dbg)

    dense = run(few, K, s)
    many = run(H, K.repeat(rep, 1, 1), s.repeat(rep, 1))
    for a, b in zip(many, dense):
        a = a.view(rep, *b.shape)[:, :3]
        assert torch.equal(a, b[None, :3].expand_as(a))
    assert 0 <= int(many[2].min()) and int(many[2].max()) < P


# (9, 17, 18 and 25 parts, whose maxima can't be 128 altogether; ranks 62 and 64 of them; one source group and two)
@pytest.mark.parametrize("P,S,m,H", [(65000, 64, 240, 28), (65000, 64, 240, 15), (131008, 64, 490, 14), (65000, 100, 240, 5)])
def test_bounds_from_uneven_parts_of_the_sample(P, S, m, H):
    """Bounds taken from as many maxima as so many parts of the sample leave are as tight as a list needs, even of the
    largest ranks: no head is redone.  Lists and scores are those of many heads, whose bounds come from the whole sample."""
    say(f"uneven parts P={P} S={S} m={m} H={H}")
    d, rep = 128, -(-130 // H)
    g = torch.Generator("cuda").manual_seed(P + H)
    K = torch.randn(H, P + 8, d, generator=g, device="cuda").to(torch.bfloat16)
    s = torch.rand(H, P, generator=g, device="cuda") + 0.1
    kw = dict(head_dim=d, n_tokens=P + 8, window=8, n_sources=S, n_neighbors=m, rounds=1)

    def run(heads, K, s):
        p = gk.Params(n_kv_heads=heads, n_q_heads=heads, **kw)
        nbr = torch.full((heads, S, m), -1, dtype=torch.int32, device="cuda")
        ws = gk.alloc_workspace(p, "cuda")
        redo = np.inf
        for _ in range(3):
            gk.graphkv_profile_begin()
            out = gk.graphkv_propagate(p, K, s.clone(), None, nbr, None, ws)
            torch.cuda.synchronize()
            redo = min(redo, 1e3 * gk.graphkv_profile_end()["redo_rows"][0])
        return out, nbr, redo

    out, nbr, redo = run(H, K, s)
    say(f"  redo launch {redo:.1f} us")
    assert redo < 50     # (6 where no head is flagged; a head takes 180 and more)
    want, lists, _ = run(rep * H, K.repeat(rep, 1, 1), s.repeat(rep, 1))
    assert torch.equal(lists.view(rep, H, S, m), nbr.expand(rep, -1, -1, -1))
    assert torch.equal(want.view(rep, H, P), out.expand(rep, -1, -1))


# (ranks 64 and 65 of the sample: the last taken from maxima and the first counted; the largest of a long prompt; two source groups)
@pytest.mark.parametrize("P,S,m,H,signal", [(16001, 40, 249, 8, 1), (16001, 40, 256, 8, 1), (16001, 70, 256, 4, 1), (131008, 33, 600, 2, 1)])
def test_later_rounds_of_few_heads_take_bound_and_filter_in_one_launch(P, S, m, H, signal):
    """Whatever the rank; with new sources in every round (an enhanced signal), each round against a one-round call of many
    heads on the scores of the round before."""
    say(f"later rounds P={P} S={S} m={m} H={H}")
    d, T, rep = 128, 3, -(-130 // H)
    g = torch.Generator("cuda").manual_seed(P + m)
    cent = torch.randn(H, 64, d, generator=g, device="cuda")
    kind = torch.randint(0, 64, (H, P + 8, 1), generator=g, device="cuda").expand(-1, -1, d)
    K = (cent.gather(1, kind) + 0.5 * torch.randn(H, P + 8, d, generator=g, device="cuda")).to(torch.bfloat16)
    s = torch.rand(H, P, generator=g, device="cuda") + 0.1

    def run(heads, K, s, rounds):
        p = gk.Params(n_kv_heads=heads, n_q_heads=heads, head_dim=d, n_tokens=P + 8, window=8, n_sources=S, n_neighbors=m,
                      rounds=rounds, signal=signal)
        dbg = [torch.full((rounds, heads, S, n) if n else (rounds, heads, S), -1, dtype=t, device="cuda")
               for n, t in ((0, torch.int32), (m, torch.int32), (m, torch.float32))]
        gk.graphkv_profile_begin()
        out = gk.graphkv_propagate(p, K, s.clone(), *dbg)
        torch.cuda.synchronize()
        return gk.graphkv_profile_end(), out, *dbg

    took, _, *few = run(H, K, s, T)
    assert took["cosine_bound_new"][1] == T - 1 and "cosine_filter_new" not in took
    many = K.repeat(rep, 1, 1)
    for t in range(T):
        _, out, *one = run(rep * H, many, s.repeat(rep, 1), 1)
        for a, b in zip(one, few):
            a = a.view(rep, *b[t].shape)
            assert torch.equal(a, b[t][None].expand_as(a)), t
        s = out[:H]


@pytest.mark.parametrize("w,pool_mode,scorer", [(20, 0, 0), (32, 1, 0), (64, 0, 0), (8, 0, 1)])
def test_calls_with_more_keys_than_the_caches_hold(w, pool_mode, scorer):
    """Batches beyond 256 MiB of keys read and write past the caches; their layers alone (8 MiB each) don't.  Scores that are cut
    as a layer's are the same bits; others (whole blocks of 32 query rows) agree to the rounding of 32-bit sums."""
    say(f"past the caches w={w} pool_mode={pool_mode} scorer={scorer}")
    L, H, G, N, d, B = 34, 4, 4 if w == 64 else 1, 8192 + w, 128, w + 100
    g = torch.Generator("cuda").manual_seed(w)
    K, V = (torch.randn(L, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    Q = (torch.randn(L, H * G, w, d, generator=g, device="cuda") + K[:, :, :w].repeat_interleave(G, dim=1)).to(torch.bfloat16)
    p = gk.Params(n_kv_heads=H, n_q_heads=H * G, head_dim=d, n_tokens=N, window=w, budget=B, pool_kernel=7, pool_mode=pool_mode,
                  rounds=0, scorer=scorer, dtype=gk.BF16)
    assert L * H * N * d * 2 > 256 << 20
    sc = torch.empty(L, H, N - w, device="cuda")
    Ks, Vs, idx = gk.graphkv_compress_batched(p, L, None, K, V, Q, scores_out=sc)
    idx = idx.view(L, H, B)
    at = idx.long()[..., None].expand(-1, -1, -1, d)
    assert torch.equal(Ks.view(L, H, B, d), K.gather(2, at)) and torch.equal(Vs.view(L, H, B, d), V.gather(2, at))
    for l in (0, 16, L - 1):
        s1 = torch.empty(H, N - w, device="cuda")
        _, _, i1 = gk.graphkv_compress(p, K[l], V[l], Q[l], scores_out=s1)
        if scorer or (G * w) % 32:
            assert torch.equal(s1, sc[l]) and torch.equal(i1, idx[l])
        else:   # (sums of 8192 terms in another order, 2^-24 each)
            assert (s1 - sc[l]).abs().max() <= 1e-5 * s1.abs().max()
