"""Reverse Cuthill-McKee where breadth-first levels are wide: runs of wide levels, frontier nodes with
as many next-level nodes as a wavefront orders (64) and more, levels that are narrow again in between,
components that end in a wide level.  Positions are integers: equal to the serial oracle's."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _layered(widths, leaves, rng, sym):
    """Every node of a layer hangs on a node of the layer before and has a few more edges there;
    `leaves` extra next-layer nodes hang on one node of each layer."""
    src, dst, first, n = [], [], 0, widths[0]
    for w in widths[1:]:
        prev = np.arange(first, n)
        new = np.arange(n, n + w + leaves)
        up = rng.choice(prev, size=(3, w))
        src += [up[0], up[1], up[2], np.full(leaves, prev[len(prev) // 2])]
        dst += [new[:w], new[:w], new[:w], new[w:]]
        if not sym:  # some edges back to what is placed already
            src.append(new[: w // 2])
            dst.append(rng.choice(prev, size=w // 2))
        first, n = n, n + w + leaves
    return np.concatenate(src), np.concatenate(dst), n


@pytest.mark.parametrize("sym", [True, False])
@pytest.mark.parametrize("leaves", [0, 63, 64, 65, 4000])
def test_wide_levels(leaves, sym):
    import paper_2501_01951_amd as mg

    rng = np.random.default_rng(100 + leaves)
    parts, n = [], 0
    for widths in ([1, 40, 1500] + [2100] * 21 + [1024, 1025, 300, 2000], [1, 20000, 20000, 5], [1, 1200]):
        s, d, m = _layered(widths, leaves, rng, sym)
        parts.append((s + n, d + n))
        n += m
    n += 7  # nodes without edges
    perm = rng.permutation(n).astype(np.uint32)
    src = perm[np.concatenate([p[0] for p in parts])]
    dst = perm[np.concatenate([p[1] for p in parts])]
    print(f"rcm wide levels: leaves {leaves} symmetric {sym} n {n}", flush=True)
    want = oracle.rcm(oracle.build_csr(src, dst, n, sym, True))
    flags = mg.ADD_SELF_LOOPS | (mg.SYMMETRIZE if sym else 0)
    g = mg.build_csr(torch.from_numpy(src.view(np.int32)).cuda(),
                     torch.from_numpy(dst.view(np.int32)).cuda(), n, flags)
    got = mg.reorder_rcm(g).cpu().numpy().view(np.uint32)
    g.free()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("wide", [262_144, 262_145, 300_000])
def test_levels_of_more_nodes_than_a_block_takes_at_once(wide):
    """A grid of 1024 blocks has 256 frontier nodes each up to 262,144: a hub's leaves, most of them with a node or two
    of their own, one with 70 in the second level after them."""
    import paper_2501_01951_amd as mg

    rng = np.random.default_rng(wide)
    leaf = np.arange(1, wide + 1)
    second = wide + 1 + np.arange(wide // 2 * 3)
    up = np.concatenate([leaf[: len(second) - wide // 2], leaf[: wide // 2]])
    third = second[-1] + 1 + np.arange(70)
    src = np.concatenate([np.zeros(wide, np.int64), up, np.full(70, second[wide // 3])])
    dst = np.concatenate([leaf, second, third])
    n = int(third[-1]) + 1
    perm = rng.permutation(n).astype(np.uint32)
    src, dst = perm[src], perm[dst]
    want = oracle.rcm(oracle.build_csr(src, dst, n, True, True))
    g = mg.build_csr(torch.from_numpy(src.view(np.int32)).cuda(), torch.from_numpy(dst.view(np.int32)).cuda(), n)
    got = mg.reorder_rcm(g).cpu().numpy().view(np.uint32)
    g.free()
    assert np.array_equal(got, want)
