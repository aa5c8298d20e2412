"""The attention kernels that let four waves share a query block (few work items) beside the ones
that give every block one wave (many), on the same heads, against the oracle.

The number of query heads of the layer decides, not the list: 66 heads of 1024 tokens are 1056
items, 3 heads are 48.
"""
import numpy as np
import pytest
import torch

from oracle import minference_oracle as O
from tests.helpers import assert_close_rows, random_qkv, to_f64
from tests.test_gpu_attention import VS_CASES, random_bs_index, run_heads, token_major

pytestmark = pytest.mark.gpu

FEW = [0, 65]           # heads of the large layer that the small one holds too, as its heads 0 and 2


@pytest.fixture(scope="module")
def B():
    from paper_2407_02490_amd import binding
    binding.lib()
    return binding


def inputs(kind, N):
    q, k, v = random_qkv(91, 66, 2, N)
    if kind == "overflow":              # late keys outgrow every reference taken before them
        k = k.clone()
        k[:, 700:] *= 60.0
    if kind == "underflow":             # every logit about -228 in the base-2 domain
        g = torch.Generator().manual_seed(78)
        u = torch.randn(128, generator=g)
        u = u / u.norm() * 128 ** 0.5
        q = (u + 0.3 * torch.randn(66, N, 128, generator=g)).to(torch.bfloat16).cuda()
        k = (-14.0 * u + 0.3 * torch.randn(2, N, 128, generator=g)).to(torch.bfloat16).cuda()
    return q, k, v


@pytest.mark.parametrize("layout", ["head", "token"])
@pytest.mark.parametrize("kind", ["normal", "overflow", "underflow"])
def test_few_and_many_items(B, rng, kind, layout):
    N = 1024
    q, k, v = inputs(kind, N)
    Vl, Sl = sorted(rng.choice(N, 200, replace=False).tolist()), list(range(0, 96)) + [300, 301, 700]
    idx, cnt = random_bs_index(rng, N // 64, 7)
    calls = {
        "dense": (lambda heads, *a: B.minf_dense_attn(*a, heads), lambda Q, K, V: O.dense_attention(Q, K, V)),
        "ashape": (lambda heads, *a: B.minf_ashape_attn(*a, heads, 100, 200),
                   lambda Q, K, V: O.ashape_attention(Q, K, V, 100, 200)),
        "window": (lambda heads, *a: B.minf_ashape_attn(*a, heads, 0, 65),
                   lambda Q, K, V: O.ashape_attention(Q, K, V, 0, 65)),
        "vs": (lambda heads, *a: B.minf_vs_attn(*a, heads, B.vs_index_from_host([Vl] * len(heads), [Sl] * len(heads), N)),
               lambda Q, K, V: O.vs_attention(Q, K, V, Vl, Sl, Bm=64)),
        "bs": (lambda heads, *a: B.minf_bs_attn(*a, heads, B.bs_index_from_host(np.stack([idx] * len(heads)),
                                                                               np.stack([cnt] * len(heads)))),
               lambda Q, K, V: O.bs_attention(Q, K, V, idx, cnt)),
    }
    many = (q, k, v, list(range(66)), FEW)
    few = (q[[0, 30, 65]], k[[0, 0, 1]], v[[0, 0, 1]], [0, 2], [0, 2])
    for name, (call, oracle) in calls.items():
        want = [oracle(to_f64(q[h]), to_f64(k[h // 33]), to_f64(v[h // 33])) for h in FEW]
        for cq, ck, cv, heads, checked in (many, few):
            o = torch.full_like(cq, float("nan"))
            tq, tk, tv, o = (token_major(t) if layout == "token" else t for t in (cq, ck, cv, o))
            call(heads, tq, tk, tv, o)
            torch.cuda.synchronize()
            for h, w in zip(checked, want):
                assert_close_rows(o[h], w, f"{name} {kind} {layout} {len(heads)} heads, head {h}")
            assert len(heads) == 66 or bool(torch.isnan(o[1].float()).all())


@pytest.mark.parametrize("n_init,n_local", [(0, 1), (0, 64), (1, 31), (63, 33), (64, 65), (65, 127), (100, 129),
                                            (130, 1), (200, 300), (704, 1)])
def test_window_edges(B, n_init, n_local):
    """Tiles that hold the end of the sink, the start of the window, the diagonal or several of them,
    with four blocks per workgroup (52 heads of 11 blocks) and with four waves per block (3 heads)."""
    N = 704
    q, k, v = random_qkv(97, 52, 2, N)
    want = {h: O.ashape_attention(to_f64(q[h]), to_f64(k[h // 26]), to_f64(v[h // 26]), n_init, n_local) for h in (0, 51)}
    for cq, ck, cv, heads, at in ((q, k, v, [0, 51], (0, 51)), (q[[0, 7, 51]], k[[0, 0, 1]], v[[0, 0, 1]], [0, 2], (0, 2))):
        o = torch.full_like(cq, float("nan"))
        B.minf_ashape_attn(cq, ck, cv, o, heads, n_init, n_local)
        torch.cuda.synchronize()
        for h, w in zip(at, want.values()):
            assert_close_rows(o[h], w, f"({n_init}, {n_local}) {len(cq)} heads, head {h}")


@pytest.mark.parametrize("nq,N", [(66, 1024), (66, 512), (5, 1024), (40, 4096)])
def test_bits_of_a_head_do_not_depend_on_the_listed_heads(B, rng, nq, N):
    """A head alone, in a short list and with all heads of the layer: the same bits from every call."""
    q, k, v = random_qkv(95, nq, 1, N)
    Vl, Sl = sorted(rng.choice(N, 60, replace=False).tolist()), list(range(0, 130)) + [300, 301]
    idx, cnt = random_bs_index(rng, N // 64, 20)
    calls = {
        "dense": lambda hs, o: B.minf_dense_attn(q, k, v, o, hs),
        "ashape": lambda hs, o: B.minf_ashape_attn(q, k, v, o, hs, 100, 200),
        "vs": lambda hs, o: B.minf_vs_attn(q, k, v, o, hs, B.vs_index_from_host([Vl] * len(hs), [Sl] * len(hs), N)),
        "bs": lambda hs, o: B.minf_bs_attn(q, k, v, o, hs, B.bs_index_from_host(np.stack([idx] * len(hs)),
                                                                               np.stack([cnt] * len(hs)))),
    }
    for name, call in calls.items():
        got = []
        for hs in ([3], [4, 3, 1], list(range(nq))):
            o = torch.full_like(q, float("nan"))
            call(hs, o)
            torch.cuda.synchronize()
            got.append(o[3])
        assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2]), name


# items of a layer beyond which no kernel splits its blocks (and rows too short for four blocks per workgroup)
def many_heads(N):
    return 1025 // (N // 64) + 1


@pytest.mark.parametrize("layout", ["head", "token"])
@pytest.mark.parametrize("N,Vl,Sl", VS_CASES)
def test_degenerate_masks_with_one_wave_per_block(B, N, Vl, Sl, layout):
    nq = many_heads(N)
    q0, k0, v0 = random_qkv(96, nq, 1, N)
    q, k, v, o = (token_major(t) if layout == "token" else t for t in (q0, k0, v0, torch.full_like(q0, float("nan"))))
    B.minf_vs_attn(q, k, v, o, [0, nq - 1], B.vs_index_from_host([Vl] * 2, [Sl] * 2, N))
    torch.cuda.synchronize()
    for h in (0, nq - 1):
        want = O.vs_attention(to_f64(q0[h]), to_f64(k0[0]), to_f64(v0[0]), Vl, Sl, Bm=64)
        assert_close_rows(o[h], want, f"{layout} head {h}")


@pytest.mark.parametrize("layout", ["head", "token"])
@pytest.mark.parametrize("kind", ["normal", "overflow"])
def test_more_than_one_round_of_columns_with_one_wave_per_block(B, rng, kind, layout):
    """1500 kept verticals: two rounds of the column list, also in the exact passes."""
    N = 2048
    nq = many_heads(N)
    q0, k0, v0 = random_qkv(97, nq, 1, N)
    if kind == "overflow":
        k0[:, 1400:] *= 60.0
    Vl, Sl = sorted(rng.choice(N, 1500, replace=False).tolist()), [0, 777]
    q, k, v, o = (token_major(t) if layout == "token" else t for t in (q0, k0, v0, torch.full_like(q0, float("nan"))))
    B.minf_vs_attn(q, k, v, o, [nq - 1], B.vs_index_from_host([Vl], [Sl], N))
    torch.cuda.synchronize()
    want = O.vs_attention(to_f64(q0[nq - 1]), to_f64(k0[0]), to_f64(v0[0]), Vl, Sl, Bm=64)
    assert_close_rows(o[nq - 1], want, f"{kind} {layout}")


@pytest.mark.parametrize("nq", [1, 70])
@pytest.mark.parametrize("kind", ["normal", "overflow"])
def test_bad_block_ids(B, rng, nq, kind):
    """Ids outside [0, NB) anywhere in a list, with four waves per block and with one."""
    N, topk = 1024, 12
    NB = N // 64
    q, k, v = random_qkv(98, nq, 1, N)
    if kind == "overflow":
        k[:, 700:] *= 60.0
    idx = -np.ones((NB, topk), np.int64)
    clean = -np.ones((NB, topk), np.int64)
    cnt = np.zeros(NB, np.int64)
    for b in range(NB):
        good = np.sort(rng.choice(b + 1, min(topk // 2, b + 1), replace=False))
        mixed = [int(x) for x in good]
        for bad in (-1, NB, 99, -5):
            mixed.insert(int(rng.integers(0, len(mixed) + 1)), bad)
        idx[b, :len(mixed)] = mixed
        clean[b, :len(good)], cnt[b] = good, len(good)
    dev = B.bs_index_from_host(idx[None], np.full((1, NB), topk))
    o = run_heads(B.minf_bs_attn, q, k, v, [nq - 1], dev)
    want = O.bs_attention(to_f64(q[nq - 1]), to_f64(k[0]), to_f64(v[0]), clean, cnt)
    assert_close_rows(o[nq - 1], want, f"bs bad ids {nq} heads {kind}")


@pytest.mark.parametrize("kind", ["normal", "overflow"])
@pytest.mark.parametrize("Sl", [[0], [0, 70], list(range(0, 8000, 70)), [5000] + list(range(6000, 6300))])
def test_shares_of_short_and_many_runs(B, rng, Sl, kind):
    """Runs of fewer steps than waves, more than one chunk of 64 runs, blocks without a run key."""
    N = 8192
    q, k, v = random_qkv(92, 1, 1, N)
    if kind == "overflow":
        k[:, 4000:] *= 60.0
    Vl = sorted(rng.choice(N, 700, replace=False).tolist())
    dev = B.vs_index_from_host([Vl], [Sl], N)
    o = run_heads(B.minf_vs_attn, q, k, v, [0], dev)
    Qh, Kh, Vh = to_f64(q[0]), to_f64(k[0]), to_f64(v[0])
    for b in (0, 1, 2, 63, 77, 78, 93, 94, 126, 127):
        want = O.vs_attention(Qh, Kh, Vh, Vl, Sl, 64 * b, 64 * b + 64, Bm=64)
        assert_close_rows(o[0, 64 * b:64 * b + 64], want, f"block {b}")


# (query heads, tokens, verticals, slashes, blocks): how each kind takes its blocks
ONE_LAUNCH = {
    "one wave, one wave": (6, 33024, 200, 203, 9),
    "four waves, four waves": (4, 1024, 100, 300, 9),
    "four waves, one wave": (4, 4096, 100, 300, 2),
    "one wave, four waves": (8, 4096, 48, 100, 24),
    "four blocks, one wave": (17, 4160, 60, 1400, 9),
    "four blocks, one wave, a launch each": (9, 8256, 60, 4200, 9),
}


@pytest.mark.parametrize("layout", ["head", "token"])
@pytest.mark.parametrize("take", ONE_LAUNCH)
def test_one_launch_of_both_kinds(B, rng, take, layout):
    """minf_vs_bs_attn, for every way the two kinds take their blocks: the same bits as the two calls,
    and the oracle's values on some blocks."""
    nq, N, nv, ns, topk = ONE_LAUNCH[take]
    NB, nb = N // 64, nq // 3
    q, k, v = random_qkv(93, nq, 1, N)
    vs_heads, bs_heads = list(range(nq - nb - 1)), list(range(nq - nb, nq))       # one head in neither list
    Vl = sorted(rng.choice(N, nv, replace=False).tolist())
    Sl = sorted(set(range(0, ns - 40)) | set(rng.choice(N, 40, replace=False).tolist()))
    vidx = B.vs_index_from_host([Vl] * len(vs_heads), [Sl] * len(vs_heads), N)
    idx, cnt = random_bs_index(rng, NB, topk)
    bidx = B.bs_index_from_host(np.stack([idx] * nb), np.stack([cnt] * nb))
    o1, o2 = torch.full_like(q, 7.0), torch.full_like(q, 7.0)
    tq, tk, tv, o1, o2 = (token_major(t) if layout == "token" else t for t in (q, k, v, o1, o2))
    B.minf_vs_attn(tq, tk, tv, o1, vs_heads, vidx)
    B.minf_bs_attn(tq, tk, tv, o1, bs_heads, bidx)
    B.minf_vs_bs_attn(tq, tk, tv, o2, vs_heads, vidx, bs_heads, bidx)
    torch.cuda.synchronize()
    assert torch.equal(o1, o2) and bool((o2[nq - nb - 1] == 7.0).all())
    Kh, Vh = to_f64(k[0]), to_f64(v[0])
    for b in (0, NB // 2, NB - 1):
        rows = slice(64 * b, 64 * b + 64)
        for h in (vs_heads[0], vs_heads[-1]):
            want = O.vs_attention(to_f64(q[h]), Kh, Vh, Vl, Sl, 64 * b, 64 * b + 64, Bm=64)
            assert_close_rows(o2[h, rows], want, f"{take} {layout} vs head {h} block {b}")
        cols = (64 * idx[b, :cnt[b]][:, None] + np.arange(64)).ravel()
        mask = np.where(cols[None, :] <= 64 * b + np.arange(64)[:, None], 0.0, -np.inf)
        s = to_f64(q[bs_heads[0], rows]) @ Kh[cols].T / 128 ** 0.5 + mask
        p = np.exp(s - np.max(s, axis=1, keepdims=True, initial=-1e30))
        den = p.sum(1, keepdims=True)
        want = np.divide(p @ Vh[cols], den, out=np.zeros((64, 128)), where=den > 0)
        assert_close_rows(o2[bs_heads[0], rows], want, f"{take} {layout} bs block {b}")


# common part of a run for four blocks = width - 192 keys in whole 64-key tiles, at least 8 of them
@pytest.mark.parametrize("Sl", [list(range(0, 642, 60)), list(range(0, 640)), list(range(0, 641)), list(range(0, 705)),
                                list(range(0, 2100)), list(range(90, 1500)), list(range(0, 700)) + list(range(1000, 2700))])
@pytest.mark.parametrize("layout,kind", [("head", "normal"), ("token", "normal"), ("head", "overflow")])
def test_common_part_of_long_runs(B, rng, Sl, layout, kind):
    """Four blocks per workgroup: runs just short of and just at the width from which their common
    part is shared, a run that starts past the diagonal, two long runs, blocks that reach key 0, an
    odd number of blocks (4160 tokens: a workgroup with one block)."""
    N = 4160
    q0, k0, v0 = random_qkv(94, 17, 1, N)
    if kind == "overflow":
        k0 = k0.clone()
        k0[:, 2500:] *= 60.0
    Vl = sorted(rng.choice(N, 150, replace=False).tolist())
    q, k, v = (token_major(t) if layout == "token" else t for t in (q0, k0, v0))
    o = torch.full_like(q0, float("nan"))
    o = token_major(o) if layout == "token" else o
    # the slashes an index has room for choose the kernel: head 0's list makes it 1400 of 4160
    B.minf_vs_attn(q, k, v, o, list(range(17)), B.vs_index_from_host([Vl] * 17, [list(range(1400))] + [Sl] * 16, N))
    torch.cuda.synchronize()
    for h in (1, 16):
        want = O.vs_attention(to_f64(q0[h]), to_f64(k0[0]), to_f64(v0[0]), Vl, Sl, Bm=64)
        for b in range(0, 65):
            assert_close_rows(o[h, 64 * b:64 * b + 64], want[64 * b:64 * b + 64], f"head {h} block {b}")


@pytest.mark.parametrize("layout", ["head", "token"])
@pytest.mark.parametrize("nq,nkv,N", [(2, 1, 704), (4, 1, 6208), (3, 3, 8256), (12, 2, 12352)])
def test_batch_elements_are_the_calls_alone(B, nq, nkv, N, layout):
    """Three prompts in one call: indices and outputs have the bits of three calls, with workspaces of
    the reported size (which hold one, two or three elements at a time) and larger ones."""
    nb, heads = 3, list(range(nq))[::-1]
    x = [random_qkv(300 + b, nq, nkv, N) for b in range(nb)]
    q, k, v = (torch.stack([e[t] for e in x]) for t in range(3))
    if layout == "token":
        q, k, v = (t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v))
    nv, ns, topk = min(300, N), min(2000, N), 20

    def layer(q, k, v, n, extra):
        o = [torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(4)]
        vi, bi = B.alloc_vs_index(n * nq, nv, ns, N), B.alloc_bs_index(n * nq, N, topk)
        for t in (vi.v_idx, vi.s_idx, vi.cover, vi.cover_bits, bi.blk_idx, bi.blk_cnt, bi.order):
            t.fill_(-7)
        B.minf_build_vs_index(q, k, heads, 64, nv, ns, vi, torch.empty(
            extra * B.minf_vs_index_workspace_bytes(q, k, nq, 64), dtype=torch.uint8, device="cuda"))
        B.minf_build_bs_index(q, k, heads, topk, bi, torch.empty(
            extra * B.minf_bs_index_workspace_bytes(q, k, nq, topk), dtype=torch.uint8, device="cuda"))
        B.minf_vs_attn(q, k, v, o[0], heads, vi)
        B.minf_bs_attn(q, k, v, o[1], heads, bi)
        B.minf_ashape_attn(q, k, v, o[2], heads, 100, 500)
        B.minf_dense_attn(q, k, v, o[3], heads)
        torch.cuda.synchronize()
        runs = vi.counts[:, 2].tolist()
        return ([vi.v_idx, vi.s_idx, vi.cover_bits, vi.counts, bi.blk_idx, bi.blk_cnt, bi.order] +
                [vi.cover[r, :c] for r, c in enumerate(runs)], o)

    alone = [layer(q[b], k[b], v[b], 1, 1) for b in range(nb)]
    for extra in (1, 4):
        idx, out = layer(q, k, v, nb, extra)
        for b in range(nb):
            for t, (got, want) in enumerate(zip(idx[:7], alone[b][0][:7])):
                assert torch.equal(got[b * nq:(b + 1) * nq], want), f"index array {t} of element {b}"
            for r in range(nq):
                assert torch.equal(idx[7 + b * nq + r], alone[b][0][7 + r]), f"runs of element {b}, head {r}"
            for t, (got, want) in enumerate(zip(out, alone[b][1])):
                assert torch.equal(got[b].view(torch.int16), want.view(torch.int16)), f"output {t} of element {b}"


@pytest.mark.parametrize("step", [0, 1])
def test_outputs_laid_over_each_other_come_out_in_batch_order(B, step):
    """Outputs of a batch with stride 0, or one head apart: what a later element writes stays."""
    nb, nq, N = 3, 2, 320
    x = [random_qkv(500 + b, nq, 1, N) for b in range(nb)]
    q, k, v = (torch.stack([e[t] for e in x]) for t in range(3))
    vi, bi = B.alloc_vs_index(nb * nq, 60, 100, N), B.alloc_bs_index(nb * nq, N, 2)
    B.minf_build_vs_index(q, k, [0, 1], 64, 60, 100, vi, torch.empty(
        B.minf_vs_index_workspace_bytes(q, k, nq, 64), dtype=torch.uint8, device="cuda"))
    B.minf_build_bs_index(q, k, [0, 1], 2, bi, torch.empty(
        B.minf_bs_index_workspace_bytes(q, k, nq, 2), dtype=torch.uint8, device="cuda"))
    v1, b1 = B.alloc_vs_index(nb, 60, 100, N), B.alloc_bs_index(nb, N, 2)          # head 0 of each element, head 1 of each
    for t in ("v_idx", "s_idx", "cover", "cover_bits", "counts"):
        getattr(v1, t).copy_(getattr(vi, t)[0::nq])
    for t in ("blk_idx", "blk_cnt", "order"):
        getattr(b1, t).copy_(getattr(bi, t)[1::nq])
    calls = [lambda o: B.minf_vs_attn(q, k, v, o, [0, 1], vi), lambda o: B.minf_bs_attn(q, k, v, o, [0, 1], bi),
             lambda o: B.minf_ashape_attn(q, k, v, o, [0, 1], 70, 100), lambda o: B.minf_dense_attn(q, k, v, o, [0, 1]),
             lambda o: B.minf_vs_bs_attn(q, k, v, o, [0], v1, [1], b1)]
    for i, call in enumerate(calls):
        want = torch.empty_like(q)
        call(want)
        out = torch.full((step * (nb - 1) + nq, N, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        call(out.as_strided(q.shape, (step * N * 128, N * 128, 128, 1)))
        torch.cuda.synchronize()
        for b in range(nb):
            for h in range(nq):
                if (b, h) == max((c, g) for c in range(nb) for g in range(nq) if step * c + g == step * b + h):
                    assert torch.equal(out[step * b + h], want[b, h]), f"call {i}, element {b}, head {h}"


@pytest.mark.parametrize("nq,row", [(2, (1 << 23) - 8), (2, 1 << 23), (2, (1 << 23) + 136), (600, (1 << 23) + 136)])
def test_gathered_rows_far_apart(B, nq, row):
    """Token distances at and beyond 2^24 bytes (128 tokens in 2 GiB): four waves per block, one wave per
    block (600 heads), and both kinds in one launch."""
    N, heads = 128, [0, nq - 1]
    q, k0, v0 = random_qkv(77, nq, 1, N)
    store = torch.empty((N - 1) * row + 256, dtype=torch.bfloat16, device="cuda")
    k, v = (store.as_strided((1, N, 128), (0, row, 1), at) for at in (0, 128))
    k.copy_(k0), v.copy_(v0)
    V, S = np.array([1, 2, 5, 17, 40, 63, 64, 65, 90, 126]), np.array([0, 70])
    idx = B.vs_index_from_host([V] * 2, [S] * 2, N)
    blocks = B.bs_index_from_host(np.zeros((1, 2, 1)), np.ones((1, 2)))
    o, both = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    B.minf_vs_attn(q, k, v, o, heads, idx)
    if nq > 2:
        B.minf_vs_bs_attn(q, k, v, both, heads, idx, [1], blocks)
    else:                                                        # one kind's list would take the other's head
        both.copy_(o)
    torch.cuda.synchronize()
    for h in heads:
        want = O.vs_attention(to_f64(q[h]), to_f64(k0[0]), to_f64(v0[0]), V, S, Bm=64)
        assert_close_rows(o[h], want, f"head {h}")
        assert torch.equal(both[h], o[h])


def index_rows(idx):
    """Arrays of an index with their valid runs, per row."""
    runs = idx.counts[:, 2].tolist()
    return [[t[r] for t in (idx.v_idx, idx.s_idx, idx.cover_bits, idx.counts)] + [idx.cover[r, :c]]
            for r, c in enumerate(runs)]


def build(B, q, k, heads, nv, ns, extra):
    rows = len(heads) * (q.shape[0] if q.dim() == 4 else 1)
    idx = B.alloc_vs_index(rows, nv, ns, q.shape[-2])
    ws = torch.empty(extra * B.minf_vs_index_workspace_bytes(q, k, len(heads), 64), dtype=torch.uint8, device="cuda")
    B.minf_build_vs_index(q, k, heads, 64, nv, ns, idx, ws)
    return idx


@pytest.mark.parametrize("engine", ["wave", "ring"])
def test_batch_elements_with_four_blocks_per_workgroup(B, monkeypatch, engine):
    """17 heads of 65 blocks are too many to split, 1400 slashes enough for vs_share_kernel: its batch
    elements, those of the one launch with a Block-Sparse head, and of the ring engine, against calls alone."""
    monkeypatch.setenv("MINF_VS_ENGINE", engine)
    nb, nq, N, nv, ns, topk = 3, 17, 4160, 40, 1400, 5
    x = [random_qkv(700 + b, nq, 1, N) for b in range(nb)]
    q, k, v = (torch.stack([e[t] for e in x]) for t in range(3))
    vs_heads, bs_heads = list(range(1, nq)), [0]

    def run(q, k, v, n):
        vi, bi = build(B, q, k, vs_heads, nv, ns, 4), B.alloc_bs_index(n, N, topk)
        B.minf_build_bs_index(q, k, bs_heads, topk, bi, torch.empty(
            4 * B.minf_bs_index_workspace_bytes(q, k, 1, topk), dtype=torch.uint8, device="cuda"))
        o, both = torch.zeros_like(q), torch.zeros_like(q)
        B.minf_vs_attn(q, k, v, o, vs_heads, vi)
        B.minf_bs_attn(q, k, v, o, bs_heads, bi)
        B.minf_vs_bs_attn(q, k, v, both, vs_heads, vi, bs_heads, bi)
        torch.cuda.synchronize()
        return o, both

    o, both = run(q, k, v, nb)
    if engine == "wave":
        assert torch.equal(o, both)
    for b in range(nb):
        o1, both1 = run(q[b], k[b], v[b], 1)
        assert torch.equal(o[b], o1) and torch.equal(both[b], both1), f"element {b}"


@pytest.mark.parametrize("N,nv,ns", [(41024, 500, 1500), (41024, 1000, 6096), (131072, 1000, 9000), (131072, 30, 2048)])
def test_batch_elements_of_rows_beyond_the_register_selection(B, N, nv, ns):
    """Three elements that share a larger workspace, with the prefilter on both lists, on none and on one of
    them: the index of calls alone."""
    nb, heads = 3, [1, 0]
    x = [random_qkv(800 + b, 2, 1, N) for b in range(nb)]
    q, k = (torch.stack([e[t] for e in x]) for t in range(2))
    got = index_rows(build(B, q, k, heads, nv, ns, 4))
    for b in range(nb):
        for r, want in enumerate(index_rows(build(B, q[b], k[b], heads, nv, ns, 1))):
            assert all(torch.equal(a, w) for a, w in zip(got[b * len(heads) + r], want)), f"element {b}, row {r}"


@pytest.mark.parametrize("N,nq,topk", [(32768, 22, 100), (135168, 2, 37)])
def test_batch_elements_of_the_candidate_lists(B, N, nq, topk):
    """Rows of logits for an element alone and candidate lists for three together (2112 workgroups of 16
    rows), and lists of rows beyond 2048 blocks: the same index."""
    nb, heads = 3, list(range(nq))
    x = [random_qkv(900 + b, nq, 1, N) for b in range(nb)]
    q, k = (torch.stack([e[t] for e in x]) for t in range(2))

    def run(q, k, n):
        idx = B.alloc_bs_index(n * nq, N, topk)
        B.minf_build_bs_index(q, k, heads, topk, idx, torch.empty(
            4 * B.minf_bs_index_workspace_bytes(q, k, nq, topk), dtype=torch.uint8, device="cuda"))
        torch.cuda.synchronize()
        return idx.blk_idx, idx.blk_cnt, idx.order

    got = run(q, k, nb)
    for b in range(nb):
        for a, w in zip(got, run(q[b], k[b], 1)):
            assert torch.equal(a[b * nq:(b + 1) * nq], w), f"element {b}"
