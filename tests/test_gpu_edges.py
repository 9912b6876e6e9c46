"""Edges of single kernels (tile remainders, smallest and largest of a range,
special values) through the public entry points."""
import numpy as np
import pytest
import torch

from gpu_common import compare, make_pair, step_pair
from oracle import mlp as M
from paper_1904_08553_amd import dc
from paper_1904_08553_amd import workloads as W

pytestmark = pytest.mark.gpu


def dev_bits(bits):
    return torch.from_numpy(bits.astype(np.uint16).view(np.int16)).cuda().contiguous()


@pytest.mark.parametrize("n", [15, 17, 65_536 + 3])
def test_forward_tiles_and_nan_rows(n):
    """The logit of a sample depends on that sample alone, wherever its tile
    lies in a wave's walk, and a NaN feature makes every first-layer unit's
    activation 0: exactly the logit of a network without its first layer."""
    print(f"case: mlp forward tiles n={n}", flush=True)
    rng = np.random.default_rng(n)
    w = M.init_weights(n)
    w[M.OFF_B2:M.OFF_W3] = 0.05
    bits = M.bf16_bits(rng.uniform(-1, 1, (n, 8))).reshape(n, 8)
    nan = rng.random(n) < 0.1
    bits[nan, rng.integers(0, 8)] = 0x7FC0
    net = dc.MLP(w)
    z = net.forward(dev_bits(bits)).cpu().numpy()
    off = 16 * (n // 32) + 3  # other tiles, other lanes
    z_off = net.forward(dev_bits(bits[off:])).cpu().numpy()
    assert np.array_equal(z[off:], z_off)
    w0 = w.copy()
    w0[:M.OFF_W2] = 0.0  # W1 and b1
    net0 = dc.MLP(w0)
    z0 = net0.forward(dev_bits(np.zeros((1, 8), np.uint16))).cpu().numpy()[0]
    assert np.all(z[nan] == z0)
    assert np.all(np.isfinite(z))
    net.close()
    net0.close()


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4097])
def test_steps_at_scan_tile_edges(n):
    """Vertex counts around the scan tile (2,048) with weighted changes: the
    restricted compaction's ranks, movers and run sums over one tile, a full
    one and a remainder of one element."""
    print(f"case: steps n={n}", flush=True)
    (u, v, w), batches = W.DCSBM(n=n, m=6 * n, blocks=20, dmax=200, seed=n).stream(3, frac=0.05)
    o, g = make_pair(n, u, v, w)
    compare(o, g, "init")
    for t, b in enumerate(batches):
        step_pair(o, g, b)
        compare(o, g, f"n={n} step {t}")


@pytest.mark.parametrize("copies", [1, 8, 9, 8 + 256, 8 + 257, 1500])
def test_runs_of_one_pair(copies):
    """A pair inserted `copies` times in one batch (around the records its own
    thread sums, and the wave's rounds over the rest), beside a hub whose
    changes fill several waves of a row tile, in both screening kinds."""
    print(f"case: runs of {copies}", flush=True)
    n = 3000
    rng = np.random.default_rng(copies)
    u, v, w = W.DCSBM(n=n, m=5 * n, blocks=12, dmax=100, seed=7).graph()
    hub = 2049
    present = np.concatenate([v[u == hub], u[v == hub]])
    fresh = np.setdiff1d(np.arange(n), np.concatenate([present, [hub]]))
    add_u = np.concatenate([np.full(copies, u[0]), np.full(len(fresh), hub)]).astype(np.int32)
    add_v = np.concatenate([np.full(copies, v[0]), fresh]).astype(np.int32)
    add_w = rng.integers(1, 4, len(add_u)).astype(np.int32)
    order = rng.permutation(len(add_u))
    gone = np.setdiff1d(np.arange(1, len(u)), np.flatnonzero((u == hub) | (v == hub)))[:700]
    first = W.Batch(add_u[order], add_v[order], add_w[order], u[gone], v[gone])
    # the hub's row leaves again, the repeated pair is replaced
    second = W.Batch(u[:1], v[:1], np.array([2], np.int32),
                     np.concatenate([u[:1], np.full(len(fresh), hub)]).astype(np.int32),
                     np.concatenate([v[:1], fresh]).astype(np.int32))
    for mode in ("delta", "all"):
        o, g = make_pair(n, u, v, w, mode=mode)
        for t, b in enumerate((first, second)):
            step_pair(o, g, b)
            compare(o, g, f"copies={copies} {mode} step {t}")


@pytest.mark.parametrize("records", [2, 2046, 2048, 2050, 4096, 4098, 16 * 2048, 16 * 2048 + 2, 64 * 2048, 64 * 2048 + 2, (1 << 20) - 2, 1 << 20, (1 << 20) + 2, 8192 * 131 + 2])
def test_initial_csr_at_sort_sizes(records):
    """The initial CSR (both directed records of every edge, sorted, equal
    pairs summed) against numpy at the sizes where the radix sort changes its
    tile, with ragged last tiles and a repeated pair."""
    print(f"case: initial csr of {records} records", flush=True)
    rng = np.random.default_rng(records)
    n, m = 50_021, records // 2
    u = rng.integers(0, n, m)
    v = (u + rng.integers(1, n, m)) % n
    w = rng.integers(1, 9, m)
    if m > 1:
        u[-1], v[-1] = v[0], u[0]
    g = dc.DynamicCommunities(n, u.astype(np.int32), v.astype(np.int32), w.astype(np.int32),
                              max_levels=1, max_sweeps=1)
    off, col, cw = g.csr()
    key = np.concatenate([u, v]) * n + np.concatenate([v, u])
    uk, inv = np.unique(key, return_inverse=True)
    assert np.array_equal(np.repeat(np.arange(n), np.diff(off)) * n + col, uk)
    assert np.array_equal(cw, np.bincount(inv, weights=np.concatenate([w, w])).astype(np.int64))
    g.close()


@pytest.mark.parametrize("slm", [False, True])
@pytest.mark.parametrize("cliques", [1, 65, 2047, 2048, 2049])
def test_level_one_sizes(cliques, slm):
    """A chain of heavy triangles: level 0 ends with one community each, so
    level 1 has as many vertices, on both sides of the size up to which a
    level is swept without bins; then changes that merge and split some."""
    print(f"case: level 1 of {cliques} vertices slm={slm}", flush=True)
    t = np.arange(cliques) * 3
    u = np.concatenate([t, t, t + 1, t[:-1] + 2]).astype(np.int32)
    v = np.concatenate([t + 1, t + 2, t + 2, t[1:]]).astype(np.int32)
    w = np.concatenate([np.full(3 * cliques, 9), np.full(cliques - 1, 1)]).astype(np.int32)
    n = 3 * cliques
    o, g = make_pair(n, u, v, w, slm=slm)
    compare(o, g, "init")
    k = t[: cliques // 2]
    near = np.column_stack([k, k + 4]) if len(k) else np.empty((0, 2), int)
    first = W.Batch(near[:, 0].astype(np.int32), near[:, 1].astype(np.int32),
                    np.full(len(near), 7, np.int32), t[: 1 + cliques // 5].astype(np.int32),
                    (t[: 1 + cliques // 5] + 1).astype(np.int32))
    second = W.Batch(first.del_u, first.del_v, np.full(len(first.del_u), 3, np.int32),
                     first.add_u, first.add_v)
    for i, b in enumerate((first, second)):
        step_pair(o, g, b)
        compare(o, g, f"cliques={cliques} step {i}")


@pytest.mark.parametrize("del_rule", [0, 1])
@pytest.mark.parametrize("entries", [7, 8, 9, 16, 17, 32, 33, 64, 65])
def test_rows_at_bin_edges(entries, del_rule):
    """Circulant graphs whose rows all have `entries` entries of random weight,
    beside rows of one and two entries: full and nearly full groups of lanes,
    all labels distinct in the first sweep; then batches in which new sources
    have as many sinks, in both deletion rules' screening passes."""
    print(f"case: rows of {entries} entries del_rule={del_rule}", flush=True)
    rng = np.random.default_rng(entries)
    n, half = 300, 150
    i = np.arange(n)
    u = [i for k in range(entries // 2)] + ([i[:half]] if entries % 2 else [])
    v = [(i + 1 + k) % n for k in range(entries // 2)] + ([i[:half] + half] if entries % 2 else [])
    u += [np.arange(n, n + 40), np.arange(n, n + 20)]  # a pendant path beside it
    v += [np.arange(n + 1, n + 41), rng.integers(0, n, 20)]
    u, v = np.concatenate(u).astype(np.int32), np.concatenate(v).astype(np.int32)
    w = rng.integers(1, 6, len(u)).astype(np.int32)
    total = n + 41 + 8
    o, g = make_pair(total, u, v, w, del_rule=del_rule)
    compare(o, g, "init")
    for t in range(3):
        src = total - 1 - t  # an isolated vertex so far
        add_v = rng.choice(n, entries, replace=False).astype(np.int32)
        cut = rng.choice(len(u), 30, replace=False)
        b = W.Batch(np.full(entries, src, np.int32), add_v,
                    rng.integers(1, 6, entries).astype(np.int32), u[cut], v[cut])
        keep = np.setdiff1d(np.arange(len(u)), cut)
        u = np.concatenate([u[keep], b.add_u])
        v = np.concatenate([v[keep], b.add_v])
        step_pair(o, g, b)
        compare(o, g, f"entries={entries} step {t}")


@pytest.mark.parametrize("labels", [128, 256, 257, 320, 321, 512, 513])
def test_rows_of_distinct_labels(labels):
    """A vertex joined to one end of each of `labels` heavy pairs, which stay
    communities: a row that brings as many labels, around what the wave's table
    lists and holds, alone and in the server's merged sweeps."""
    print(f"case: a row of {labels} labels", flush=True)
    i = np.arange(labels)
    u, v, w = (2 * i).astype(np.int32), (2 * i + 1).astype(np.int32), np.full(labels, 9, np.int32)
    n, hub = 2 * labels + 1, 2 * labels
    none = np.empty(0, np.int32)
    to = lambda k: W.Batch(np.full(len(k), hub, np.int32), (2 * k).astype(np.int32),
                           (1 + k % 3).astype(np.int32), none, none)
    cut = W.Batch(none, none, none, np.full(labels // 2, hub, np.int32), u[::2][: labels // 2])
    batches = [to(i), cut, to(i[::2][: labels // 2])]
    o, g = make_pair(n, u, v, w)
    compare(o, g, "init")
    want = []
    for t, b in enumerate(batches):
        step_pair(o, g, b)
        compare(o, g, f"labels={labels} step {t}")
        want.append(o.C.copy())
    srv = dc.Server(max_inflight=2)
    gids = [srv.add_graph(n, u, v, w) for _ in range(2)]
    tickets = [(t, gid, srv.submit(gid, b.add_u, b.add_v, b.add_w, b.del_u, b.del_v))
               for t, b in enumerate(batches) for gid in gids]
    for t, gid, tk in tickets:
        assert np.array_equal(srv.poll(tk, gid)[0], want[t]), f"graph {gid} batch {t}"
    assert srv.stats()["merged_rounds"] > 0
    srv.close()


@pytest.mark.parametrize("hubs", [1, 1024, 1025])
def test_hub_tables_past_one_round(hubs):
    """Rows of 4,100 distinct labels (more than the LDS table takes, so each is
    evaluated in its own part of the global tables), as many as one round of the
    offsets' scan covers and one more."""
    print(f"case: {hubs} hub rows", flush=True)
    leaves = 4100
    u = np.repeat(np.arange(hubs, dtype=np.int32), leaves)
    v = np.tile(np.arange(hubs, hubs + leaves, dtype=np.int32), hubs)
    w = ((u.astype(np.int64) * 7 + v * 13) % 5 + 1).astype(np.int32)
    o, g = make_pair(hubs + leaves, u, v, w, max_levels=1, max_sweeps=1)
    compare(o, g, f"hubs={hubs}")


@pytest.mark.parametrize("n", [1 << 19, (1 << 19) + 1, (1 << 20) + 1, (1 << 21) + 1])
def test_movers_at_block_rounds(n):
    """Triangles with random edges between them, from singletons: most vertices
    of a block move, to more labels than its table holds; then a batch that moves
    few.  Vertex counts around those at which a block takes more of the list."""
    print(f"case: movers of {n} vertices", flush=True)
    rng = np.random.default_rng(n)
    i = np.arange(n // 3) * 3
    u = np.concatenate([i, i, i + 1, rng.integers(0, n, n // 8)])
    v = np.concatenate([i + 1, i + 2, i + 2, rng.integers(0, n, n // 8)])
    u, v = u[u != v].astype(np.int32), v[u != v].astype(np.int32)
    w = (1 + u % 3).astype(np.int32)
    o, g = make_pair(n, u, v, w)
    compare(o, g, "init")
    add_u = rng.integers(0, n, 500).astype(np.int32)
    add_v = ((add_u + 1 + rng.integers(0, n - 1, 500)) % n).astype(np.int32)
    step_pair(o, g, W.Batch(add_u, add_v, np.full(500, 9, np.int32), u[:200], v[:200]))
    compare(o, g, "step")


@pytest.mark.parametrize("n,edges,changes", [(100, 3_000, 1_500), (700, 60_000, 30_000),
                                             (2_048, 30_000, 2_100), (4_097, 60_000, 20_000)])
def test_long_change_slices(n, edges, changes):
    """Batches with more than two rounds of changes a tile of rows: hundreds of
    changes a row and a few, a last tile of one row; insertions, additions to
    pairs that are there, replacements and deletions, in both screening forms."""
    print(f"case: {changes} changes of {n} vertices", flush=True)
    rng = np.random.default_rng(n)
    key = rng.choice(n * (n - 1) // 2, edges, replace=False)
    hi = ((1 + np.sqrt(1 + 8 * key.astype(np.float64))) / 2).astype(np.int64)
    hi -= key < hi * (hi - 1) // 2
    hi += key >= hi * (hi + 1) // 2
    u, v = (key - hi * (hi - 1) // 2).astype(np.int32), hi.astype(np.int32)
    w = rng.integers(1, 5, edges).astype(np.int32)
    kept = edges - changes // 2  # the rest come in as new pairs
    for mode in ("delta", "all"):
        o, g = make_pair(n, u[:kept], v[:kept], w[:kept], mode=mode)
        gone = rng.choice(kept, changes // 2, replace=False)
        again = gone[: changes // 4]  # replaced, and others added to
        more = rng.choice(kept, changes // 4, replace=False)
        more = np.setdiff1d(more, gone)
        add = np.concatenate([np.arange(kept, edges), again, more])
        rng.shuffle(add)
        first = W.Batch(u[add], v[add], w[add], u[gone], v[gone])
        back = gone[changes // 4:]
        second = W.Batch(u[back], v[back], w[back], u[kept:], v[kept:])
        for t, b in enumerate((first, second)):
            step_pair(o, g, b)
            compare(o, g, f"n={n} {mode} step {t}")
