"""Trees of up to 256 nodes at batches of one to six requests per compute unit: the LDS of a launch depends on both,
and the waves of a workgroup with it."""
import numpy as np
import pytest

import oracle
from tests import parity

pytestmark = pytest.mark.gpu


def _text(rng, n, pool, vocab):
    parts, have = [], 0
    while have < n:
        a = int(rng.integers(0, len(pool) - 20))
        parts.append(pool[a:a + int(rng.integers(20, 160))])
        have += len(parts[-1])
    t = np.concatenate(parts)[:n].copy()
    mut = rng.random(n) < 0.02
    t[mut] = rng.integers(0, vocab, int(mut.sum()))
    return t.astype(np.int32)


# One request to a compute unit: around the sizes at which a wave less fits (16 waves end at 132 nodes, 15 at 142, ...
# 10 at 229); more of them: where the workgroups of a compute unit just fit together, and just do not.
@pytest.mark.parametrize("nodes,batch", [
    (n, 6) for n in (132, 133, 138, 142, 143, 149, 162, 177, 194, 215, 229, 230, 239, 240, 255, 256)] + [
    (72, 300), (73, 300), (128, 300), (136, 500), (236, 500), (66, 700), (128, 700), (256, 700), (64, 1000),
    (78, 1000), (132, 1000), (186, 1000), (256, 1000), (106, 1300), (122, 1300), (256, 1300)])
def test_trees_of_all_sizes(nodes, batch):
    rng = np.random.default_rng(1000 * nodes + batch)
    vocab, P, D, ms = 300, 64, 200, 0.002
    alpha = (nodes + 0.5) / P
    pool = rng.integers(0, vocab, 900)
    docs = [_text(rng, 400, pool, vocab) for _ in range(30)]
    ctxs = [_text(rng, int(rng.integers(1, 500)), pool, vocab) for _ in range(min(batch, 12))]
    NV = len(ctxs)
    of = np.arange(batch) % NV
    g = parity.GpuPath(vocab, D, P, alpha, ms, batch, 500 + nodes + 1, sum(len(d) + 1 for d in docs))
    try:
        assert g.max_nodes == nodes
        g.build_global(docs)
        g.build_requests(range(batch), [ctxs[v] for v in of])
        tg = oracle.Trie(D)
        for d in docs:
            tg.add_doc(d)
        want = parity.oracle_speculate_batch(tg, ctxs, D, P, alpha, ms, nodes)
        bad = parity.compare_trees(g.speculate(range(batch)), {k: v[of] for k, v in want.items()}, "drafts")
        assert not bad, "\n".join(bad)
        # a step on: the target model follows the drafts' first children for some nodes
        tgt = np.full((NV, nodes + 1), vocab - 1, np.int32)
        longer, exp = [], []
        for v in range(NV):
            n, at = int(want["n_nodes"][v]), -1
            for _ in range(7 * v):
                kids = np.flatnonzero(want["parents"][v, :n] == at)
                if not len(kids):
                    break
                tgt[v, at + 1] = want["tokens"][v, kids[0]]
                at = int(kids[0])
            L, path, bonus = oracle.accept(want["tokens"][v, :n], want["parents"][v, :n], tgt[v])
            exp.append((L, list(path), bonus))
            longer.append(np.concatenate([ctxs[v], want["tokens"][v, list(path)], [bonus]]).astype(np.int32))
        al, ap, bo, got = g.accept_append_speculate(range(batch), tgt[of])
        for b in range(batch):
            L, path, bonus = exp[of[b]]
            assert al[b] == L and bo[b] == bonus and list(ap[b, :L]) == path, b
        want = parity.oracle_speculate_batch(tg, longer, D, P, alpha, ms, nodes)
        bad = parity.compare_trees(got, {k: v[of] for k, v in want.items()}, "drafts a step on")
        assert not bad, "\n".join(bad)
    finally:
        g.close()


@pytest.mark.parametrize("den_mode,linear", [(0, 0), (1, 0), (0, 1)])
@pytest.mark.parametrize("nodes", [1, 2, 5, 16, 63, 64])
def test_more_candidates_than_a_tree_has_room_for(nodes, den_mode, linear):
    """Nodes with 1 to 300 children, of which most score alike: what does not fit the frontier is left out by score and
    token, the lowest of the equals staying, at the root and below it, among up to 64 suffixes and among more."""
    rng = np.random.default_rng(1000 * nodes + 10 * den_mode + linear)
    vocab, D, P = 700, 12, 2
    docs, contexts = [], []
    for head, (children, most) in enumerate([(1, 1), (nodes, 1), (nodes + 1, 1), (nodes + 2, 2), (64, 1), (65, 1), (150, 2), (300, 3)]):
        for x in rng.permutation(np.arange(20, 320))[:children]:
            for _ in range(int(rng.integers(1, most + 1))):
                docs.append(np.array([head, x] + list(rng.integers(320, 324, 3)), np.int32))
        contexts += [np.array([400 + head, head], np.int32), np.array([head], np.int32)]
    docs = [docs[i] for i in rng.permutation(len(docs))]
    alpha = nodes / 2.0
    g = parity.GpuPath(vocab, D, P, alpha, 0.0, len(contexts), 8, sum(len(d) + 1 for d in docs), den_mode=den_mode, linear=linear)
    try:
        g.build_global(docs)
        g.build_requests(range(len(contexts)), contexts)
        got = g.speculate(range(len(contexts)))
        tg = parity.oracle_global_trie(docs, D, vocab)
        want = parity.oracle_speculate_batch(tg, contexts, D, P, alpha, 0.0, int(np.floor(alpha * P)), den_mode=den_mode, linear=linear)
        bad = parity.compare_trees(got, want, "%d nodes" % nodes)
        assert not bad, "\n".join(bad)
    finally:
        g.close()


@pytest.mark.parametrize("nodes", [2, 16, 31, 33, 40, 56, 61])
def test_one_candidate_too_many(nodes):
    """A root whose first 64 suffixes have one child more than the tree has nodes, or three, against one with as many as it has:
    what does not fit is left out, of the equals the last ones, and costs no more than a look at it (put in one by one:
    1.2 times as long with 16 nodes, 1.4 with 56)."""
    import torch
    import paper_2411_04975_amd as sd
    vocab, D, B, head = 400, 6, 64, 1
    us = {}
    for extra in (0, 1, 3) if nodes + 4 <= 64 else (0, 1):
        kids = nodes + extra + 1  # (the last one goes on behind the 64 and enters by itself)
        counts = np.full(kids, 64 // kids)
        counts[:64 - counts.sum()] += 1
        docs = [[head, 10 + i, 300 + j % 3] for i, n in enumerate(counts) for j in range(n)] + [[head, 9 + kids, 303]] * 20
        docs = [np.array(docs[i], np.int32) for i in np.random.default_rng(kids).permutation(len(docs))]
        contexts = [np.array([350, head], np.int32)] * B
        g = parity.GpuPath(vocab, D, 1, float(nodes), 0.0, B, 8, sum(len(d) + 1 for d in docs))
        try:
            g.build_global(docs)
            g.build_requests(range(B), contexts)
            got = g.speculate(range(B))
            want = parity.oracle_speculate_batch(parity.oracle_global_trie(docs, D, vocab), contexts[:1], D, 1, float(nodes), 0.0, nodes)
            bad = parity.compare_trees(got, {k: np.repeat(v, B, 0) for k, v in want.items()})
            assert not bad, "\n".join(bad)
            out = sd.Trees(B, nodes, g.dev)
            times = []
            for _ in range(8):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                for _ in range(50):
                    sd.sd_speculate(g.ctx, None, out)
                b.record()
                torch.cuda.synchronize()
                times.append(a.elapsed_time(b) * 20)
            us[extra] = min(times)
        finally:
            g.close()
    print("%d nodes:" % nodes, us)
    if nodes >= 16:
        assert max(us.values()) < 1.12 * us[0]
