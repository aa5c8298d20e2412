"""Selection kernels of the index builds at the sizes where their dispatch changes."""
import numpy as np
import pytest
import torch

from oracle import minference_oracle as O
from tests.helpers import check_topk, random_qkv, to_f64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2407_02490_amd import binding
    binding.lib()
    return binding


def build_vs(B, q, k, heads, nv, ns):
    N = q.shape[1]
    idx = B.alloc_vs_index(len(heads), nv, ns, N)
    ws = torch.empty(B.minf_vs_index_workspace_bytes(q, k, len(heads), 64), dtype=torch.uint8, device="cuda")
    B.minf_build_vs_index(q, k, heads, 64, nv, ns, idx, ws)
    torch.cuda.synchronize()
    return idx


# 8192 | 32768 | 40960 scores: the steps of what a thread holds; behind the last, the candidates of the
# prefilter if it serves both lists, from 131072 on also if it serves one, else from memory; the run bits come
# from LDS up to 262144
@pytest.mark.parametrize("N,nv,ns", [(64, 64, 64), (128, 1, 1), (4096, 256, 512), (8192, 1000, 6096), (8256, 1000, 6096),
                                     (32768, 100, 1800), (32832, 3000, 200), (40960, 500, 1500), (41024, 500, 1500),
                                     (131072, 1000, 6096), (262144, 30, 2048), (262208, 30, 2048)])
def test_vs_selection_and_runs(B, N, nv, ns):
    q, k, _ = random_qkv(61, 2, 1, N)
    idx = build_vs(B, q, k, [0, 1], nv, ns)
    # runs and bitmap against the builder that takes the same lines as a list
    n_runs = idx.counts[:, 2].tolist()
    again = B.VSIndex(2, nv, ns, N, "cuda")
    again.v_idx.copy_(idx.v_idx), again.s_idx.copy_(idx.s_idx), again.counts.copy_(idx.counts)
    B.minf_vs_index_from_lines(again)
    torch.cuda.synchronize()
    assert torch.equal(idx.counts, again.counts) and torch.equal(idx.cover_bits, again.cover_bits)
    for r in range(2):
        assert torch.equal(idx.cover[r, :n_runs[r]], again.cover[r, :n_runs[r]])
    if N <= 65536:
        col, diag = O.vs_line_scores(O.vs_estimate(to_f64(q[1]), to_f64(k[0]), 64))
        check_topk(idx.v_idx[1].cpu().numpy(), col, nv)
        check_topk(idx.s_idx[1].cpu().numpy(), diag, ns)


@pytest.mark.parametrize("N,nv,ns", [(41024, 1000, 6096), (41024, 500, 1500), (65536, 1000, 6096), (97472, 1000, 6096),
                                     (97536, 1000, 6096), (131072, 1000, 9000), (131072, 9000, 30), (131072, 40000, 40000)])
def test_vs_selection_of_long_rows(B, N, nv, ns):
    """Rows beyond what a thread holds, with the prefilter for both lists (97536: 4 x 6096 groups of 4), for one
    of them (from 131072 on) and for none: exactly the largest line scores, which lie at the start of the
    workspace, equal ones to the lower position."""
    q, k, _ = random_qkv(67, 2, 1, N)
    idx = B.alloc_vs_index(2, nv, ns, N)
    ws = torch.empty(B.minf_vs_index_workspace_bytes(q, k, 2, 64), dtype=torch.uint8, device="cuda")
    B.minf_build_vs_index(q, k, [0, 1], 64, nv, ns, idx, ws)
    torch.cuda.synchronize()
    scores = ws[:4 * N * 4].view(torch.float32).view(2, 2, N).cpu()
    for which, (lines, n) in enumerate(((idx.v_idx, nv), (idx.s_idx, ns))):
        for r in range(2):
            best = torch.sort(scores[which, r], descending=True, stable=True).indices[:n]
            assert torch.equal(lines[r].cpu(), torch.sort(best).values.int()), f"list {which}, row {r}"


@pytest.mark.parametrize("N", [1024, 4160, 12352, 33024, 65600, 131072])
def test_vs_scores_do_not_depend_on_the_listed_heads(B, N):
    """A head listed alone and with all others (four K/V heads): the same line scores, bit for bit
    (they lie at the start of the workspace, [heads][N] of the columns, then of the diagonals), and
    the same lines."""
    heads = list(range(8))
    q, k, _ = random_qkv(64, 8, 4, N)
    got = []
    for hs in (heads, [5]):
        idx = B.alloc_vs_index(len(hs), 50, 200, N)
        ws = torch.empty(B.minf_vs_index_workspace_bytes(q, k, len(hs), 64), dtype=torch.uint8, device="cuda")
        B.minf_build_vs_index(q, k, hs, 64, 50, 200, idx, ws)
        torch.cuda.synchronize()
        scores = ws[:2 * len(hs) * N * 4].view(torch.int32).view(2, len(hs), N)
        r = hs.index(5)
        got.append((scores[0, r].cpu(), scores[1, r].cpu(), idx.v_idx[r].cpu(), idx.s_idx[r].cpu(), idx.counts[r].cpu()))
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("N", [4096, 8256, 41024])
def test_vs_ties_go_to_the_lower_position(B, N):
    """All logits equal: every key before the last 64 has the same column sum."""
    q, k, _ = random_qkv(62, 1, 1, N)
    idx = build_vs(B, q, torch.zeros_like(k), [0], 700, 10)
    assert torch.equal(idx.v_idx[0].cpu(), torch.arange(700, dtype=torch.int32))


@pytest.mark.parametrize("N,heads,topk", [(8256, 66, 100), (8256, 66, 7), (32768, 40, 100), (65600, 9, 100)])
def test_bs_few_and_many_rows_and_order(B, N, heads, topk):
    """Listed alone, a head's blocks are pooled and selected 32 per workgroup; the full lists of 66 and
    40 heads fill the chip with workgroups of 128 blocks (9 heads of 65600 tokens do not: there only
    the longer order is new).  512 blocks overflow the candidate lists, whose running cut depends on
    which waves select.  The same index either way, and the oracle's."""
    NB = N // 64
    q, k, _ = random_qkv(63, heads, 1, N)
    got = []
    for hs in ([heads - 1], list(range(heads))):
        idx = B.alloc_bs_index(len(hs), N, topk)
        ws = torch.empty(B.minf_bs_index_workspace_bytes(q, k, len(hs), topk), dtype=torch.uint8, device="cuda")
        B.minf_build_bs_index(q, k, hs, topk, idx, ws)
        torch.cuda.synchronize()
        got.append((idx.blk_idx[-1].cpu(), idx.blk_cnt[-1].cpu(), idx.order[-1].cpu()))
    assert all(torch.equal(a, b) for a, b in zip(*got))
    first = got[0][0][:, 0].numpy()
    assert np.array_equal(got[0][2].numpy(), np.lexsort((np.arange(NB), first)))
    qp, kp = (to_f64(t).reshape(NB, 64, 128).mean(1) for t in (q[heads - 1], k[0]))
    for b in (0, 31, 32, 63, NB // 2, NB - 1):
        score = kp[:b + 1] @ qp[b] / 128 ** 0.5
        n = min(topk, b + 1)
        assert got[0][1][b] == n and bool((got[0][0][b, n:] == -1).all())
        # pooled values are sums of 64 bf16 numbers in float32: the logits agree to about 1e-6
        check_topk(got[0][0][b, :n].numpy(), score, n, tol=1e-5, relative=False)


@pytest.mark.parametrize("kind", ["random", "special"])
@pytest.mark.parametrize("N,heads,topk", [(32768, 66, 100), (32704, 66, 37), (65536, 33, 112), (131072, 17, 1)])
def test_bs_rows_in_lds_and_candidate_lists_agree(B, N, heads, topk, kind):
    """A head alone is selected from rows of logits in LDS (up to 512, 1024, 2048 blocks), in a list of
    more than 2048 groups of 16 blocks by candidate lists: the same bits, ties (repeated keys), infinite and
    NaN logits included."""
    NB = N // 64
    q, k, _ = random_qkv(64, heads, 1, N)
    if kind == "special":
        k = k.clone().view(1, NB, 64, 128)
        k[:, 3::7] = k[:, 2:3]                                # equal logits
        k[:, 11::13, 0, 5] = float("inf")                     # +inf or -inf by the sign of the pooled query
        k[:, 17::29, 1, 7] = float("nan")
        k = k.view(1, N, 128)
    got = []
    for hs in ([heads - 1], list(range(heads))):
        idx = B.alloc_bs_index(len(hs), N, topk)
        idx.blk_idx.fill_(-5)
        ws = torch.empty(B.minf_bs_index_workspace_bytes(q, k, len(hs), topk), dtype=torch.uint8, device="cuda")
        B.minf_build_bs_index(q, k, hs, topk, idx, ws)
        torch.cuda.synchronize()
        got.append((idx.blk_idx[-1].cpu(), idx.blk_cnt[-1].cpu()))
    assert all(torch.equal(a, b) for a, b in zip(*got))
    live = torch.arange(topk)[None] < got[0][1][:, None]
    assert bool((got[0][0][~live] == -1).all()) and bool((got[0][0][live] >= 0).all())


@pytest.mark.parametrize("N", [64, 128, 192, 1984, 2048, 4032, 4096])
def test_vs_scores_of_short_rows_in_every_grid(B, N):
    """Chunks of 64 or 128 keys in pass 2, partial sums combined there or by a launch of their own: the
    line scores of a head have the same bits alone and in a list over eight K/V heads; indices as the oracle's."""
    q, k, _ = random_qkv(66, 16, 8, N)
    nv, ns, got = min(40, N), min(100, N), []
    for hs in (list(range(16)), [13], [13, 2, 5]):
        idx = B.alloc_vs_index(len(hs), nv, ns, N)
        ws = torch.empty(B.minf_vs_index_workspace_bytes(q, k, len(hs), 64), dtype=torch.uint8, device="cuda")
        B.minf_build_vs_index(q, k, hs, 64, nv, ns, idx, ws)
        torch.cuda.synchronize()
        scores = ws[:2 * len(hs) * N * 4].view(torch.int32)
        r, pad = hs.index(13), (-len(hs) * N * 4) % 256 // 4            # the arrays start 256-byte aligned
        col = scores[r * N:(r + 1) * N].cpu()
        diag = ws[(len(hs) * N + pad) * 4:].view(torch.int32)[r * N:(r + 1) * N].cpu()
        got.append((col, diag, idx.v_idx[r].cpu(), idx.s_idx[r].cpu(), idx.counts[r].cpu(), idx.cover_bits[r].cpu()))
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
    col, diag = O.vs_line_scores(O.vs_estimate(to_f64(q[13]), to_f64(k[6]), 64))
    check_topk(got[0][2].numpy(), col, nv)
    check_topk(got[0][3].numpy(), diag, ns)
