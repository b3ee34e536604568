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
# or through LDS (128 with up to 2,048 rows of capacity, 256 up to 65,536, else
# 512), the workgroup through LDS (1,024 and 2,048) or by counting rows (longer,
# or as many rows as LDS counts in one pass: 2,048, 4,096 and 8,192); rows
# spread over the block and crowded into a part of it.
@pytest.mark.parametrize("n_dst", [700, 2048, 2049, 4096, 4097, 8192, 8193, 20_000, 65_536, 65_537])
def test_transpose_sort_tiers(n_dst):
    lens = [l for l in (1, 2, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025,
                        2047, 2048, 2049, 4097, 8193, 12_000, 20_000) if l <= n_dst]
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


# Layers with K of more than 256 and n_out of 192 and more take the 256 x 256
# matrix-core tiles once the capacity has 128 of them (32,513 rows at one tile column),
# else the 64 x 64 and 128 x 128 ones; K % 128 and n_out % 8 keep some out.  The
# forward's tiles are 192, 224 or 256 rows high.
@pytest.mark.parametrize("k_each,cat,n_out,cap,rows", [
    (256, True, 256, 32_513, 32_513), (256, True, 256, 32_512, 32_512), (256, True, 192, 40_000, 33_333),
    (384, False, 200, 32_600, 32_600), (264, False, 256, 33_000, 33_000), (192, True, 256, 33_000, 32_999),
    (256, True, 188, 33_000, 33_000), (512, False, 264, 17_000, 16_500), (256, True, 256, 57_000, 57_000)])
def test_update_tall_layers(k_each, cat, n_out, cap, rows):
    g = torch.Generator(device=DEV).manual_seed(k_each + n_out + cap)
    a = [torch.randn((cap, k_each), generator=g, device=DEV).bfloat16() for _ in range(2 if cat else 1)]
    grad = torch.randn((cap, n_out), generator=g, device=DEV)
    K = k_each * len(a)
    w = torch.randn((K, n_out), generator=g, device=DEV) / K ** 0.5
    bias = torch.randn(n_out, generator=g, device=DEV)
    for t in (*a, grad):
        t[rows:] = float("nan")  # never part of a result
    m_dev = torch.tensor([rows], dtype=torch.int64, device=DEV) if rows < cap else None
    wt = w.t().contiguous().bfloat16()
    out = torch.zeros((cap, n_out), dtype=torch.bfloat16, device=DEV)
    dw, db = torch.empty((K, n_out), device=DEV), torch.empty(n_out, device=DEV)
    da = torch.zeros((cap, K), device=DEV)
    nbr = a[1] if cat else None
    gnn.update_fwd(a[0], nbr, w, bias, out, True, gnn.GNN_BF16, m_dev=m_dev, wt=wt)
    ws = torch.full_like(gnn.update_bwd_workspace(K, n_out, cap, gnn.GNN_BF16, DEV), 255)  # NaN patterns
    gnn.update_bwd(a[0], nbr, w, grad, dw, db, da, gnn.GNN_BF16, m_dev=m_dev, ws=ws)
    da_only, dw2, db2 = da.clone(), torch.empty_like(dw), torch.empty_like(db)
    gnn.update_bwd(a[0], nbr, w, grad, dw2, db2, None, gnn.GNN_BF16, m_dev=m_dev, ws=ws)
    torch.cuda.synchronize()
    A = torch.cat([x[:rows] for x in a], 1).double()
    W, G = w.bfloat16().double(), grad[:rows].bfloat16().double()
    # 2-norm, relative: fp32 sums of n terms walk off by about 2^-24 sqrt(n)
    # (4 x for the spread); the bf16 result adds its rounding, at most 2^-9
    u = 2.0 ** -24
    for got, want, tol in ((out[:rows], (A @ W + bias.double()).clamp(min=0), 2.0 ** -9 + 4 * u * K ** 0.5),
                           (dw, A.t() @ G, 4 * u * rows ** 0.5), (dw2, A.t() @ G, 4 * u * rows ** 0.5),
                           (db, grad[:rows].double().sum(0), 4 * u * rows ** 0.5),
                           (da_only[:rows], G @ W.t(), 4 * u * n_out ** 0.5)):
        assert float((got.double() - want).norm() / want.norm()) <= tol
    # (with and without dA the rows may be split differently: db2 has its own sums)
    assert float((db2.double() - db.double()).norm() / db.double().norm()) <= 8 * u * rows ** 0.5
    # the entry that brings its own scratch gives the same bits for every size it took
    if ws.numel() <= 32 << 20:
        dw3, db3, da3 = torch.empty_like(dw), torch.empty_like(db), torch.zeros_like(da)
        gnn.update_bwd_noalloc(a[0], nbr, w, grad, dw3, db3, da3, gnn.GNN_BF16, m_dev=m_dev)
        assert torch.equal(dw3, dw) and torch.equal(db3, db) and torch.equal(da3[:rows], da[:rows])
    else:
        assert K >= 512 and n_out >= 512


# Transpose columns of more than 16 entries are summed by the workgroup, the
# first 64 of them per workgroup; repeated entries, several 64-entry windows,
# widths from one lane to more than a workgroup.
@pytest.mark.parametrize("f", [1, 32, 63, 100, 130, 256, 260, 300])
@pytest.mark.parametrize("kind", ["mean", "gcn", "max"])
def test_aggregate_bwd_long_columns(kind, f):
    from tests.test_gpu_parity import relerr, upload_block
    rng = np.random.default_rng(f)
    n_dst, n_src = 700, 900
    lens = np.concatenate([[0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 699, 700], rng.integers(1, 30, size=n_src - 13)])
    rows = [[] for _ in range(n_dst)]
    for c, l in enumerate(lens):
        for v in rng.choice(n_dst, size=l, replace=False):
            rows[v].append(c)
    for v in range(0, n_dst, 3):
        rows[v] += rows[v][:2]
    rowptr = np.zeros(n_dst + 1, dtype=np.int64)
    rowptr[1:] = np.cumsum([len(r) for r in rows])
    col = np.concatenate([np.array(r, dtype=np.int32) for r in rows])
    row_of = np.repeat(np.arange(n_dst, dtype=np.int32), np.diff(rowptr))
    order = np.argsort(col, kind="stable")
    cscptr = np.zeros(n_src + 1, dtype=np.int64)
    cscptr[1:] = np.cumsum(np.bincount(col, minlength=n_src))
    blk = oracle.Block(src_ids=np.arange(n_src, dtype=np.int64), rowptr=rowptr, col=col, cscptr=cscptr,
                       cscrow=row_of[order].astype(np.int32), n_dst=n_dst)
    norm = rng.uniform(0.1, 1, size=n_src).astype(np.float32) if kind == "gcn" else None
    b = upload_block(blk, norm)
    d_a = rng.standard_normal((n_dst, f if kind == "gcn" else 2 * f)).astype(np.float32)
    h = rng.standard_normal((n_src, f)).astype(np.float32)
    d_src = torch.empty((n_src, f), device=DEV)
    d_a_d, h_d = torch.from_numpy(d_a).to(DEV), torch.from_numpy(h).to(DEV)
    if kind == "max":
        _, arg = oracle.aggregate_fwd_max(blk, h, oracle.F32)
        want = oracle.aggregate_bwd_max(blk, arg, d_a, f, h, oracle.F64)
        gnn.aggregate_bwd_max(b, torch.from_numpy(arg).to(DEV), d_a_d, f, d_src, h_d)
    else:
        ok, gk = (oracle.GCN, gnn.GNN_AGG_GCN_SYM) if kind == "gcn" else (oracle.SAGE, gnn.GNN_AGG_SAGE_MEAN)
        want = oracle.aggregate_bwd(ok, blk, norm, d_a, f, h, oracle.F64)
        gnn.aggregate_bwd(b, gk, d_a_d, f, d_src, h_d)
    # fp32 sums of up to 900 terms: within 900 2^-24 of the terms' magnitude sum
    assert relerr(d_src.cpu().numpy(), want) <= 1e-5


# Forward sums: bf16 rows of an even number of elements, at least eight, on a
# 4-byte boundary take eight elements per lane and up to two rows per
# wavefront; others four. The slots' order is that of the tile-deduplicated
# aggregation for all of them.
@pytest.mark.parametrize("f", [1, 2, 6, 7, 8, 10, 12, 16, 50, 98, 100, 101, 102, 128, 130, 256, 258, 514, 600])
@pytest.mark.parametrize("shift", [0, 1, 2])
def test_aggregate_fwd_lanes(f, shift):
    from tests.test_gpu_parity import from_np_act, to_np_act, relerr, upload_block
    rng = np.random.default_rng(f)
    n = 300
    rows = [rng.choice(n, size=int(d), replace=True) for d in rng.choice([0, 1, 2, 3, 8, 9, 17, 64, 65, 130], size=n)]
    rowptr, col = csr(rows)
    blk = oracle.build_block(rowptr, col, rng.permutation(n)[:211].astype(np.int64), 200, 1, 1, 1)
    norm = rng.uniform(0.1, 1, size=blk.n_src).astype(np.float32)
    b = upload_block(blk, norm)
    for dt in (torch.bfloat16, torch.float32):
        base = torch.zeros(blk.n_src * f + 8, dtype=dt, device=DEV)
        h = base[shift:shift + blk.n_src * f].view(blk.n_src, f)  # rows on any element boundary
        h.copy_(torch.from_numpy(rng.standard_normal((blk.n_src, f)).astype(np.float32)))
        for okind, kind in ((oracle.SAGE, gnn.GNN_AGG_SAGE_MEAN), (oracle.GCN, gnn.GNN_AGG_GCN_SYM)):
            for odt in (torch.bfloat16, torch.float32):
                obase = torch.full((blk.n_dst * f + 8,), 7.0, dtype=odt, device=DEV)
                out = obase[shift:shift + blk.n_dst * f].view(blk.n_dst, f)
                gnn.aggregate_fwd(b, kind, h, out)
                dedup = torch.empty((blk.n_dst, f), dtype=odt, device=DEV)
                gnn.aggregate_fwd_dedup(b, kind, h.contiguous(), dedup)
                want = oracle.aggregate_fwd(okind, blk, norm, to_np_act(h), oracle.F64)
                # fp32 sums of up to 200 terms; a bf16 result rounds by at most 2^-8 relative
                assert relerr(out.float().cpu().numpy(), want) <= (2.0 ** -8 if odt == torch.bfloat16 else 1e-5)
                assert torch.equal(out, dedup)
                rest = torch.cat([obase[:shift], obase[shift + blk.n_dst * f:]])
                assert bool((rest == 7.0).all())  # nothing beside the rows is written


# Outputs above 32 MiB bypass the caches; a count known to the host gets a
# workgroup for every few rows.
@pytest.mark.parametrize("rows,dim,tdt,odt", [
    (83_886, 100, torch.float32, torch.float32), (83_887, 100, torch.float32, torch.float32),
    (167_773, 100, torch.float32, torch.bfloat16), (90_001, 256, torch.float16, torch.float32),
    (70_001, 256, torch.float16, torch.bfloat16), (66_000, 260, torch.bfloat16, torch.bfloat16)])
def test_gather_large_outputs(rows, dim, tdt, odt):
    g = torch.Generator(device=DEV).manual_seed(rows)
    table = torch.randn((50_000, dim), generator=g, device=DEV).to(tdt)
    table[7, :4] = torch.tensor([float("nan"), float("inf"), -0.0, 1e-30], device=DEV).to(tdt)
    ids = torch.randint(0, 50_000, (rows,), generator=g, device=DEV)
    ids[-1] = 7
    out = torch.full((rows + 1, dim), 3.0, dtype=odt, device=DEV)
    gnn.gather_features(table, ids, out[:rows])
    want = table[ids].to(odt)
    bits = torch.int32 if odt == torch.float32 else torch.int16
    same = (out[:rows].view(bits) == want.view(bits)) | (torch.isnan(out[:rows]) & torch.isnan(want))
    assert bool(same.all()) and bool((out[rows] == 3.0).all())


# Gradients above 32 MiB bypass the caches.
@pytest.mark.parametrize("n_src", [8192, 8193])
@pytest.mark.parametrize("kind", ["mean", "max"])
def test_aggregate_bwd_large_gradient(kind, n_src):
    from tests.test_gpu_parity import relerr, upload_block
    f, n_dst = 1024, 50
    rng = np.random.default_rng(n_src)
    rows = [rng.choice(n_src, size=40, replace=False) for _ in range(n_dst)] + [[] for _ in range(n_src - n_dst)]
    rowptr, col = csr(rows)
    blk = oracle.build_block(rowptr, col, np.arange(n_dst, dtype=np.int64), 40, 1, 1, 1)
    # every vertex a source, so that the gradient is n_src rows
    blk.src_ids = np.arange(n_src, dtype=np.int64)
    blk.cscptr = np.concatenate([blk.cscptr, np.full(n_src + 1 - blk.cscptr.size, blk.cscptr[-1])])
    b = upload_block(blk)
    d_a = rng.standard_normal((n_dst, 2 * f)).astype(np.float32)
    h = rng.standard_normal((n_src, f)).astype(np.float32)
    d_src = torch.full((n_src + 1, f), 5.0, device=DEV)
    h_d, d_a_d = torch.from_numpy(h).to(DEV), torch.from_numpy(d_a).to(DEV)
    if kind == "max":
        _, arg = oracle.aggregate_fwd_max(blk, h, oracle.F32)
        want = oracle.aggregate_bwd_max(blk, arg, d_a, f, h, oracle.F64)
        gnn.aggregate_bwd_max(b, torch.from_numpy(arg).to(DEV), d_a_d, f, d_src, h_d)
    else:
        want = oracle.aggregate_bwd(oracle.SAGE, blk, None, d_a, f, h, oracle.F64)
        gnn.aggregate_bwd(b, gnn.GNN_AGG_SAGE_MEAN, d_a_d, f, d_src, h_d)
    assert relerr(d_src[:n_src].cpu().numpy(), want) <= 1e-6  # fp32 sums of a few terms
    assert bool((d_src[n_src] == 5.0).all())


# A last layer tall and wide enough that gnn_update_bwd gives it to the 256 x 256
# tiles: the folded two-layer backward keeps the engine's splits for it.
@pytest.mark.parametrize("kind,f1,n_out,n_dst", [("mean", 256, 256, 32_513), ("max", 256, 200, 32_700),
                                                 ("gcn", 264, 256, 33_000)])
def test_two_layer_bwd_tall_last_layer(kind, f1, n_out, n_dst):
    rng = np.random.default_rng(n_dst)
    n, f0, fanout = 36_000, 64, 3
    g = torch.Generator(device=DEV).manual_seed(n_dst)
    rowptr = np.arange(n + 1, dtype=np.int64) * 4
    col = np.sort(rng.integers(0, n, size=(n, 4)), axis=1).reshape(-1).astype(np.int64)
    graph = gnn.DeviceGraph(torch.from_numpy(rowptr).to(DEV), torch.from_numpy(col).to(DEV))
    b = gnn.DeviceBlock(n, n_dst, fanout, True, True, DEV)
    gnn.build_block(graph, torch.from_numpy(rng.permutation(n)[:n_dst].astype(np.int64)).to(DEV), fanout, 1, 0, 1, b,
                    gnn.sampler_workspace(n, n_dst, fanout, DEV), gcn_norm_t=gnn.gcn_norm(graph))
    n_src = int(b.counts[1])
    mk = lambda *s: torch.randn(s, generator=g, device=DEV)  # noqa
    cat = kind != "gcn"
    x, m1 = mk(n, f0).bfloat16(), mk(n, f0).bfloat16()
    h1, agg = mk(b.src_ids.numel(), f1).clamp_(min=0).bfloat16(), mk(n_dst, f1).bfloat16()
    d_a, g2 = mk(n_dst, 2 * f1 if cat else f1), mk(n_dst, n_out)
    arg = torch.zeros((n_dst, f1), dtype=torch.int32, device=DEV)
    K1, K2 = (2 * f0, 2 * f1) if cat else (f0, f1)
    out = [torch.empty((K1, f1), device=DEV), torch.empty(f1, device=DEV), torch.empty((K2, n_out), device=DEV),
           torch.empty(n_out, device=DEV)]
    rows = torch.tensor([n_src], dtype=torch.int64, device=DEV)
    cap1 = b.src_ids.numel()
    gk = {"mean": gnn.GNN_AGG_SAGE_MEAN, "gcn": gnn.GNN_AGG_GCN_SYM, "max": gnn.GNN_AGG_SAGE_MAX}[kind]
    ws = gnn.two_layer_bwd_workspace(gk, f0, f1, n_out, cap1, n_dst, DEV)
    ws.fill_(255)  # NaN patterns
    print(f"[two_layer_bwd tall] {kind} f1={f1} n_out={n_out} n_dst={n_dst}", flush=True)
    g1 = torch.empty((b.src_ids.numel(), f1), device=DEV)
    if kind == "max":
        gnn.aggregate_fwd_max(b, h1, torch.empty_like(agg), arg)
        gnn.two_layer_bwd_max(b, x, m1, rows, cap1, h1, agg, arg, d_a, g2, *out, ws=ws)
        gnn.aggregate_bwd_max(b, arg, d_a, f1, g1, h1)
    else:
        gnn.two_layer_bwd(b, gk, x if cat else None, m1, rows, cap1, h1, agg, d_a, g2, *out, ws=ws)
        gnn.aggregate_bwd(b, gk, d_a, f1, g1, h1)
    dw1, db1 = torch.empty_like(out[0]), torch.empty_like(out[1])
    gnn.update_bwd(x if cat else m1, m1 if cat else None, torch.zeros((K1, f1), device=DEV), g1, dw1, db1, None,
                   gnn.GNN_BF16, m_dev=rows)
    torch.cuda.synchronize()
    assert torch.equal(out[0], dw1) and torch.equal(out[1], db1)
    A = torch.cat([h1[:n_dst], agg], 1).double() if cat else agg.double()
    tol = 4 * 2.0 ** -24 * n_dst ** 0.5  # fp32 sums of n_dst terms, 4 x for the spread
    for got, want in ((out[2], A.t() @ g2.bfloat16().double()), (out[3], g2.double().sum(0))):
        assert float((got.double() - want).norm() / want.norm()) <= tol


# Tall capacities with few live rows (a row count on the device): the tiles that
# hold rows and their height follow the count.  A tile's sums do not depend on
# either, so the rows are those of the full capacity's call bit for bit; the
# weight gradient has splits of its own.
@pytest.mark.parametrize("k_each,cat,n_out,cap,rows", [
    (256, True, 256, 45_056, 1), (256, True, 192, 60_000, 500), (384, False, 200, 100_000, 10_000),
    (256, True, 384, 26_624, 193), (256, True, 256, 180_000, 18_000), (256, True, 256, 57_000, 49_152)])
def test_update_tall_capacity_few_rows(k_each, cat, n_out, cap, rows):
    g = torch.Generator(device=DEV).manual_seed(cap + rows)
    a = [torch.randn((cap, k_each), generator=g, device=DEV).bfloat16() for _ in range(2 if cat else 1)]
    nbr = a[1] if cat else None
    grad = torch.randn((cap, n_out), generator=g, device=DEV)
    K = k_each * len(a)
    w = torch.randn((K, n_out), generator=g, device=DEV) / K ** 0.5
    bias = torch.randn(n_out, generator=g, device=DEV)
    wt = w.t().contiguous().bfloat16()
    res = []
    for m_dev in (None, torch.tensor([rows], dtype=torch.int64, device=DEV)):
        out = torch.full((cap, n_out), 7.0, dtype=torch.bfloat16, device=DEV)
        da = torch.full((cap, K), 7.0, device=DEV)
        dw, db = torch.empty((K, n_out), device=DEV), torch.empty(n_out, device=DEV)
        gnn.update_fwd(a[0], nbr, w, bias, out, True, gnn.GNN_BF16, m_dev=m_dev, wt=wt)
        ws = torch.full_like(gnn.update_bwd_workspace(K, n_out, cap, gnn.GNN_BF16, DEV), 255)  # NaN patterns
        gnn.update_bwd(a[0], nbr, w, grad, dw, db, da, gnn.GNN_BF16, m_dev=m_dev, ws=ws)
        res.append((out, da, dw, db))
    torch.cuda.synchronize()
    (out, da, _, _), (out_m, da_m, dw, db) = res
    assert torch.equal(out_m[:rows], out[:rows]) and torch.equal(da_m[:rows], da[:rows])
    assert bool((out_m[rows:] == 7.0).all()) and bool((da_m[rows:] == 7.0).all())
    A = torch.cat([x[:rows] for x in a], 1).double()
    tol = 4 * 2.0 ** -24 * max(rows, 16) ** 0.5  # (as test_update_tall_layers)
    for got, want in ((dw, A.t() @ grad[:rows].bfloat16().double()), (db, grad[:rows].double().sum(0))):
        assert float((got.double() - want).norm()) <= tol * float(want.norm())


def transpose_block(member, norm=None):
    """A block of which aggregation backward reads the transpose: member[j, i]
    says whether column j holds row i (bool, on the device)."""
    n_src, n_dst = member.shape
    nnz = int(member.sum())
    cap = max(n_dst, -(-nnz // 1024))
    b = gnn.DeviceBlock(max(n_src, cap), cap, 1024, True, norm is not None, DEV)
    b.counts[0], b.counts[1], b.counts[2] = n_dst, n_src, nnz
    b.cscptr[1:n_src + 1] = member.sum(1).cumsum(0)
    b.cscrow[:nnz] = member.nonzero()[:, 1].int()
    b.rowptr[1:n_dst + 1] = member.sum(0).cumsum(0)
    if norm is not None:
        b.src_norm[:n_src] = norm
    return b


def bwd_in_64_bits(kind, member, d_a, f, norm, argmax):
    """gnn_aggregate_bwd's or its max form's formula, without a mask."""
    n_src, n_dst = member.shape
    x, M = d_a.double(), member.double()
    own = torch.zeros((n_src, f), dtype=torch.float64, device=DEV)
    if kind == "gcn":
        own[:n_dst] = x * norm[:n_dst, None].double() ** 2
        return own + norm[:, None].double() * (M @ (x * norm[:n_dst, None].double()))
    own[:n_dst] = x[:, :f]
    if kind == "mean":
        return own + M @ (x[:, f:] / member.sum(0).clamp(min=1)[:, None])
    won = member[argmax.long(), torch.arange(n_dst, device=DEV)[:, None]]
    return own.scatter_add_(0, argmax.long(), x[:, f:] * won)


def run_bwd(kind, b, d_a, f, argmax):
    d = torch.full((b.src_ids.numel(), f), 5.0, device=DEV)
    if kind == "max":
        gnn.aggregate_bwd_max(b, argmax, d_a, f, d)
    else:
        gnn.aggregate_bwd(b, gnn.GNN_AGG_GCN_SYM if kind == "gcn" else gnn.GNN_AGG_SAGE_MEAN, d_a, f, d)
    return d


# Rows of up to 128 elements: columns summed by the row's own lanes (up to 8
# entries), by a wavefront (up to 16 S, S = 64 / ceil(f / 4)) and by the
# workgroup, and the entries at which a lane's groups of four begin.
@pytest.mark.parametrize("f", [1, 3, 4, 16, 32, 50, 64, 100, 128])
@pytest.mark.parametrize("kind", ["mean", "gcn", "max"])
def test_aggregate_bwd_narrow_columns(kind, f):
    S = 64 // (-(-f // 4))
    lens = [0, 1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17]
    lens += [x + d for x in (S, 3 * S, 4 * S, 8 * S, 16 * S, 48 * S, 64 * S) for d in (-1, 0, 1)] + [1500]
    lens = [min(x, 1500) for x in lens]
    rng = np.random.default_rng(f)
    n_dst, n_src = 1500, 1500 + 64
    member = np.zeros((n_src, n_dst), dtype=bool)
    at = rng.permutation(n_src)[:len(lens)]
    for j, l in zip(at, lens):
        member[j, rng.choice(n_dst, size=l, replace=False)] = True
    member[-1] |= ~member.any(0)  # (every row has an edge)
    member = torch.from_numpy(member).to(DEV)
    g = torch.Generator(device=DEV).manual_seed(f)
    norm = torch.rand(n_src, generator=g, device=DEV) + 0.1
    d_a = torch.randn((n_dst, f if kind == "gcn" else 2 * f), generator=g, device=DEV)
    argmax = torch.randint(0, n_src, (n_dst, f), generator=g, device=DEV).int()
    longest = torch.from_numpy(at[-8:]).to(DEV)  # (winners enough in the long columns)
    argmax[::2] = longest[torch.randint(0, 8, (n_dst, f), generator=g, device=DEV)].int()[::2]
    b = transpose_block(member, norm if kind == "gcn" else None)
    print(f"[narrow columns] {kind} f={f}", flush=True)
    got = run_bwd(kind, b, d_a, f, argmax)
    want = bwd_in_64_bits(kind, member, d_a, f, norm, argmax)
    size = bwd_in_64_bits(kind, member, d_a.abs(), f, norm, argmax)  # (of the terms)
    # at most 1,500 / 4 additions follow one another (with f = 128 some 50): they
    # walk off by 2^-24 sqrt(50); 2 x for the weights' own rounding
    assert bool(((got[:n_src].double() - want).norm(dim=1) <= 16 * 2.0 ** -24 * size.norm(dim=1)).all())
    assert bool((got[n_src:] == 5.0).all())


# The error of a hub's sum at narrow widths: not above that of S slots that
# take an edge each in turn, whose partial sums are added in order.
@pytest.mark.parametrize("f", [4, 16, 32, 128])
def test_aggregate_bwd_hub_precision(f):
    n_dst, hubs = 4000, 24
    member = torch.zeros((n_dst + hubs, n_dst), dtype=torch.bool, device=DEV)
    member[n_dst:] = True
    b = transpose_block(member)
    w = np.float32(1.0) / np.float32(hubs)
    S = 64 // (-(-f // 4))
    errors = np.zeros(2)
    for seed in range(8):
        g = torch.Generator(device=DEV).manual_seed(seed)
        d_a = torch.rand((n_dst, 2 * f), generator=g, device=DEV)  # (terms of one sign: the sums grow)
        got = run_bwd("mean", b, d_a, f, None)[n_dst:n_dst + hubs]
        assert torch.equal(got, got[:1].expand(hubs, f))
        x = d_a[:, f:].cpu().numpy().astype(np.float64)
        acc = np.zeros((S, f), dtype=np.float32)
        for t in range(0, n_dst, 64):
            for k in range(t, min(t + 64, n_dst)):
                acc[(k - t) % S] = (x[k] * w + acc[(k - t) % S]).astype(np.float32)
        ref = acc[0]
        for s in range(1, S):
            ref = ref + acc[s]
        want = (x * np.float64(w)).sum(0)
        errors += [((got[0].cpu().numpy() - want) ** 2).sum(), ((ref - want) ** 2).sum()]
    # (1.2 x: the ratio of two random errors of 8 f sums)
    assert errors[0] ** 0.5 <= 1.2 * errors[1] ** 0.5


# More long columns than a wavefront's list holds: those past it are summed by
# the wavefront that met them, in the same parts, so a run repeats bit for bit.
@pytest.mark.parametrize("f,kind", [(128, "mean"), (128, "max"), (130, "mean"), (130, "max")])
def test_aggregate_bwd_more_long_columns_than_listed(f, kind):
    n_dst, n_src = 64, 8192 * 18
    g = torch.Generator(device=DEV).manual_seed(f)
    order = torch.rand((n_src, n_dst), generator=g, device=DEV).argsort(1)
    member = torch.zeros((n_src, n_dst), dtype=torch.bool, device=DEV).scatter_(1, order[:, :40], True)
    d_a = torch.randn((n_dst, 2 * f), generator=g, device=DEV)
    argmax = torch.randint(0, n_src, (n_dst, f), generator=g, device=DEV).int()
    b = transpose_block(member)
    print(f"[long columns] {kind} f={f}", flush=True)
    got = run_bwd(kind, b, d_a, f, argmax)
    want = bwd_in_64_bits(kind, member, d_a, f, None, argmax)
    assert float((got[:n_src].double() - want).norm() / want.norm()) <= 1e-6  # fp32 sums of 40 terms
    assert torch.equal(run_bwd(kind, b, d_a, f, argmax), got)


# The bf16 conversion of the kernels against the integer rule, by the gather's
# vector and element-wise forms: every sign and exponent with mantissas at and
# beside the ties (to even and to odd), carries into the exponent, subnormals,
# infinities, and quiet and signalling NaNs.
@pytest.mark.parametrize("dim", [8, 5])
def test_bf16_conversion_bits(dim):
    mantissas = np.array([0, 1, 2, 0x7fff, 0x8000, 0x8001, 0xffff, 0x10000, 0x17fff, 0x18000, 0x18001, 0x3f8000,
                          0x3fffff, 0x400000, 0x408000, 0x7f7fff, 0x7f8000, 0x7f8001, 0x7fffff], dtype=np.uint32)
    head = np.arange(512, dtype=np.uint32) << 23  # sign and exponent
    bits = (head[:, None] | mantissas).reshape(-1)
    bits = np.concatenate([bits, np.zeros(-bits.size % 40, dtype=np.uint32)]).reshape(-1, dim)
    table = torch.from_numpy(bits.view(np.float32)).to(DEV)
    out = torch.empty(bits.shape, dtype=torch.bfloat16, device=DEV)
    gnn.gather_features(table, torch.arange(bits.shape[0], device=DEV), out)
    got = out.view(torch.int16).cpu().numpy().view(np.uint16)
    assert np.array_equal(got, oracle.f32_to_bf16_bits(bits.view(np.float32)).reshape(bits.shape))
