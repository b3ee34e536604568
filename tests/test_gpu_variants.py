"""Kernel variants at the sizes where they change over, against the CPU
oracle: one test per rule that picks a variant."""

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

gnn = pytest.importorskip("paper_2303_00158_amd.gnn")

DEV = torch.device("cuda:0")


def csr(rows):
    rowptr = np.zeros(len(rows) + 1, dtype=np.int64)
    rowptr[1:] = np.cumsum([len(r) for r in rows])
    return rowptr, np.concatenate([np.sort(r) for r in rows]).astype(np.int64)


def build(rowptr, col, dst, fanout, norm=False):
    """gnn.build_block's block and the oracle's, both on the host."""
    g = gnn.DeviceGraph(torch.from_numpy(rowptr).to(DEV), torch.from_numpy(col).to(DEV))
    n = rowptr.size - 1
    blk = gnn.DeviceBlock(n, dst.size, fanout, True, norm, DEV)
    ws = gnn.sampler_workspace(n, dst.size, fanout, DEV)
    gnn.build_block(g, torch.from_numpy(dst).to(DEV), fanout, 11, 2, 1, blk, ws,
                    gcn_norm_t=gnn.gcn_norm(g) if norm else None)
    torch.cuda.synchronize()
    assert int(blk.counts[3].item()) == 0
    return blk.host(), oracle.build_block(rowptr, col, dst, fanout, 11, 2, 1)


# Columns sorted by a thread (up to 16 entries), a wavefront in registers (64)
# or through LDS (128 with up to 2,048 rows of capacity, else 512), the
# workgroup through LDS (2,048) or by counting rows (longer, or up to 8,192
# rows in the block); rows spread over the block and crowded into a part of it.
@pytest.mark.parametrize("n_dst", [700, 2048, 2049, 8192, 8193, 20_000])
def test_transpose_sort_tiers(n_dst):
    lens = [l for l in (1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 511, 512, 513, 1024, 2047, 2048, 2049, 4097, 8193,
                        12_000, 20_000) if l <= n_dst]
    rng = np.random.default_rng(n_dst)
    dst = rng.permutation(n_dst).astype(np.int64)
    rows = [[] for _ in range(n_dst + len(lens) + 3)]
    for i, l in enumerate(lens):
        for v in rng.choice(n_dst, size=l, replace=False):
            rows[v].append(n_dst + i)
    for i, l in enumerate((60, 500, 2000)):
        for v in dst[100:100 + l]:
            rows[v].append(n_dst + len(lens) + i)
    # repeated edges: their row stands in the column as often
    for v in rng.choice(n_dst, size=n_dst // 8, replace=False):
        rows[v] += rows[v][:1]
    rowptr, col = csr(rows)
    got, ref = build(rowptr, col, dst, 32)
    for key in ("src_ids", "rowptr", "col", "cscptr", "cscrow"):
        assert np.array_equal(got[key], getattr(ref, key)), key


# Fanouts of up to 16 and 32 take 16 and 32 lanes per row, larger ones a
# wavefront; degrees just above the fanout make most draws meet a value that
# an earlier draw took, those that gave way among them.
@pytest.mark.parametrize("fanout", [1, 2, 5, 15, 16, 17, 25, 31, 32, 33, 64, 65])
def test_sampler_lanes_per_row(fanout):
    rng = np.random.default_rng(fanout)
    n = 1500
    degrees = [0, 1, fanout - 1, fanout, fanout + 1, fanout + 2, fanout + 3, 2 * fanout + 1, 900]
    rows = [rng.choice(n, size=degrees[v % len(degrees)], replace=False) for v in range(n)]
    rowptr, col = csr(rows)
    for n_dst in (1, 2, 3, 4, 5, 63, 1021):
        dst = rng.permutation(n)[:n_dst].astype(np.int64)
        got, ref = build(rowptr, col, dst, fanout, norm=True)
        for key in ("src_ids", "rowptr", "col", "cscptr", "cscrow"):
            assert np.array_equal(got[key], getattr(ref, key)), (n_dst, key)
        assert np.array_equal(got["src_norm"], oracle.gcn_norm(rowptr)[ref.src_ids]), n_dst


# A hop that may mark an eighth of the vertices marks them in bytes, else in
# bits; the last vertices sit at the end of the padded maps.
@pytest.mark.parametrize("n", [31, 32, 33, 8191, 8192, 8193, 70_000, 300_000])
def test_sampler_vertex_marks(n):
    rng = np.random.default_rng(n)
    ids = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, size=min(n, 3000))]))
    deg = np.zeros(n, dtype=np.int64)
    deg[ids] = rng.integers(0, 12, size=ids.size)
    rowptr = np.zeros(n + 1, dtype=np.int64)
    rowptr[1:] = np.cumsum(deg)
    col = rng.integers(max(0, n - 20_000), n, size=int(rowptr[-1])).astype(np.int64)
    for v in ids:
        col[rowptr[v]:rowptr[v + 1]].sort()
    dst = rng.permutation(ids).astype(np.int64)
    g = gnn.DeviceGraph(torch.from_numpy(rowptr).to(DEV), torch.from_numpy(col).to(DEV))
    ws = gnn.sampler_workspace(n, dst.size, 7, DEV)
    # hops of both kinds share the maps, each meeting what the last one cleared
    for step, m in enumerate([dst.size, min(dst.size, n // 60 + 1), dst.size]):
        blk = gnn.DeviceBlock(n, m, 7, True, False, DEV)
        gnn.build_block(g, torch.from_numpy(dst[:m]).to(DEV), 7, 1, step, 1, blk, ws)
        torch.cuda.synchronize()
        got, ref = blk.host(), oracle.build_block(rowptr, col, dst[:m], 7, 1, step, 1)
        for key in ("src_ids", "rowptr", "col", "cscptr", "cscrow"):
            assert np.array_equal(got[key], getattr(ref, key)), (step, key)
