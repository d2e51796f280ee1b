"""GPU parity of ntp_edge_softmax (GAT-style attention weights, Section 2.1) and of
ntp_aggregate_weighted (aggregation with caller-supplied edge weights) against the oracle."""
import sys

import numpy as np
import pytest

import oracle
import ntp_inputs as gen
import paper_2412_20379_amd as ntp
from helpers import assert_close, TOL_F32

pytestmark = pytest.mark.gpu
TOL_ALPHA = 1e-5          # relative, per weight


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def _scores(n, seed, scale=1.5):
    rng = gen.stream_rng(seed, 31)
    return (rng.normal(size=n) * scale).astype(np.float32), (rng.normal(size=n) * scale).astype(np.float32)


def _device_alpha(g, nnz, p, q, slope, want_out=True):
    import torch
    from gpu_util import dev_f32
    a_in = torch.full((nnz,), float("nan"), device="cuda:0")
    a_out = torch.full((nnz,), float("nan"), device="cuda:0") if want_out else None
    ntp.ntp_edge_softmax(g, dev_f32(p), dev_f32(q), slope, a_in, a_out)
    torch.cuda.synchronize()
    return a_in, a_out


def _check_alpha(og, a_in, a_out, p, q, slope, what):
    r_in, r_out = oracle.edge_softmax(og, p, q, slope)
    got_in = a_in.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got_in)), what
    err = np.abs(got_in - r_in) / r_in
    say("   %s: alpha_in max rel err %.2e" % (what, err.max()))
    assert err.max() <= TOL_ALPHA, what
    deg = np.diff(og.csr.rowptr)
    sums = np.bincount(np.repeat(np.arange(og.n), deg), weights=got_in, minlength=og.n)
    assert np.abs(sums[deg > 0] - 1.0).max() <= 1e-5          # rows without entries have no weights
    if a_out is not None:
        got_out = a_out.cpu().numpy()
        assert (np.abs(got_out.astype(np.float64) - r_out) / r_out).max() <= TOL_ALPHA, what
        # the same edge carries the same bits in both orders
        import scipy.sparse as sp
        n = og.n
        # entry ids of the by-destination order, transposed to the by-source order
        ids = sp.csr_matrix((np.arange(1, og.csr.nnz + 1, dtype=np.float64), og.csr.colidx, og.csr.rowptr), shape=(n, n))
        t = ids.transpose().tocsr()
        t.sort_indices()
        perm = t.data.astype(np.int64) - 1
        assert np.array_equal(a_in.cpu().numpy()[perm].view(np.uint32), got_out.view(np.uint32)), what + ": orders differ in bits"


@pytest.fixture(scope="module")
def hub():
    """directed, every degree bin populated, the hub's row beyond the split threshold"""
    n = 3000
    src, dst = gen.directed_random_edges(n, 40000, 21, hub=5, hub_in=2600, hub_out=900)
    og = oracle.build_graph(n, src, dst, oracle.DIRECTED_GCN_FLAGS)
    g = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS)
    yield n, src, dst, g, og
    g.close()


@pytest.mark.parametrize("slope", [0.2, 0.0, 1.0])
def test_attention_weights_directed(hub, slope):
    n, src, dst, g, og = hub
    p, q = _scores(n, 3)
    a_in, a_out = _device_alpha(g, og.csr.nnz, p, q, slope)
    _check_alpha(og, a_in, a_out, p, q, slope, "hub graph slope %g" % slope)


def test_attention_weights_extreme_scores(hub):
    """scores far apart: the shift by the row maximum keeps everything finite"""
    n, src, dst, g, og = hub
    p, q = _scores(n, 4, scale=25.0)
    a_in, a_out = _device_alpha(g, og.csr.nnz, p, q, 0.2)
    got = a_in.cpu().numpy().astype(np.float64)
    ref, _ = oracle.edge_softmax(og, p, q, 0.2)
    assert np.all(np.isfinite(got))
    big = ref > 1e-30                     # weights that are not denormal in fp32
    assert (np.abs(got[big] - ref[big]) / ref[big]).max() <= 5e-5      # exp(x) carries the rounding of x ~ 50
    assert np.abs(np.add.reduceat(got, og.csr.rowptr[:-1]) - 1.0).max() <= 1e-5


def test_attention_weights_symmetric_and_configs():
    for cfg, scale in ((1, 1), (2, 1), (4, 64)):
        n, src, dst = gen.make_graph(cfg, seed=0, scale_down=scale)
        og = oracle.build_graph(n, src, dst, oracle.GCN_FLAGS)
        g = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_GCN_FLAGS)
        assert ntp.ntp_graph_info(g)["is_symmetric"]
        p, q = _scores(n, cfg)
        a_in, a_out = _device_alpha(g, og.csr.nnz, p, q, 0.2)
        _check_alpha(og, a_in, a_out, p, q, 0.2, "config %d" % cfg)
        g.close()


def test_attention_degree_edge_cases():
    degs = [1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257,
            511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 5000]
    n = 6000
    rng = gen.stream_rng(5, 1)
    src, dst = [], []
    for v, d in enumerate(degs):
        others = rng.choice(np.setdiff1d(np.arange(n), [v]), size=d - 1, replace=False)
        src.append(others)
        dst.append(np.full(d - 1, v))
    src = np.concatenate(src).astype(np.int32)
    dst = np.concatenate(dst).astype(np.int32)
    og = oracle.build_graph(n, src, dst, oracle.DIRECTED_GCN_FLAGS)
    g = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS)
    p, q = _scores(n, 9)
    a_in, a_out = _device_alpha(g, og.csr.nnz, p, q, 0.2)
    _check_alpha(og, a_in, a_out, p, q, 0.2, "degree edge cases")
    g.close()


@pytest.mark.parametrize("f,dtype", [(16, "f32"), (76, "f32"), (256, "f32"), (64, "bf16")])
def test_weighted_aggregation(hub, f, dtype):
    """forward and backward aggregation with the attention weights as edge weights"""
    import torch
    from gpu_util import dev_f32, dev_bf16_bits, host_bf16
    from helpers import TOL_BF16
    n, src, dst, g, og = hub
    p, q = _scores(n, 6)
    a_in, a_out = _device_alpha(g, og.csr.nnz, p, q, 0.2)
    # the oracle aggregates with the very weights the device holds (isolates the aggregation) ...
    wg = oracle.weighted(og, a_in.cpu().numpy(), a_out.cpu().numpy())
    x = gen.normal_features(n, f, seed=f)
    for direction, m, w in ((ntp.NTP_FWD, wg.csr, a_in), (ntp.NTP_BWD, wg.csc, a_out)):
        if dtype == "f32":
            y = torch.full((n, f), float("nan"), device="cuda:0")
            ntp.ntp_aggregate_weighted(g, direction, w, dev_f32(x), y, f, f, f)
            torch.cuda.synchronize()
            ref, ref_abs = oracle.aggregate(m, x, with_abs=True)
            assert_close(y.cpu().numpy(), ref, ref_abs, TOL_F32, "weighted %d f=%d" % (direction, f))
        else:
            bits, xv = dev_bf16_bits(x)
            y = torch.zeros((n, f), dtype=torch.int16, device="cuda:0")
            ntp.ntp_aggregate_weighted(g, direction, w, bits, y, f, f, f, ntp.NTP_BF16)
            torch.cuda.synchronize()
            ref, ref_abs = oracle.aggregate(m, xv, with_abs=True)
            assert_close(host_bf16(y), oracle.round_bf16(ref).astype(np.float64), ref_abs, TOL_BF16, "weighted bf16")
    # ... and end to end: oracle weights, oracle aggregation
    if dtype == "f32":
        r_in, r_out = oracle.edge_softmax(og, p, q, 0.2)
        ref, ref_abs = oracle.aggregate(oracle.weighted(og, r_in, r_out).csr, x, with_abs=True)
        y = torch.full((n, f), float("nan"), device="cuda:0")
        ntp.ntp_aggregate_weighted(g, ntp.NTP_FWD, a_in, dev_f32(x), y, f, f, f)
        torch.cuda.synchronize()
        assert_close(y.cpu().numpy(), ref, ref_abs, TOL_F32, "attention + aggregation f=%d" % f)
    # the stored (GCN) weights are untouched
    from gpu_util import check_agg
    check_agg(g, og, x, "fwd", dtype, "stored weights after a weighted call")


def test_weighted_backward_on_a_one_form_graph(hub):
    """a graph without the by-source form scatters along its rows with by-destination weights"""
    import torch
    from gpu_util import dev_f32
    n, src, dst, _, og = hub
    g = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS | ntp.NTP_SCATTER_BWD)
    p, q = _scores(n, 8)
    a_in, _ = _device_alpha(g, og.csr.nnz, p, q, 0.2, want_out=False)
    with pytest.raises(ntp.NtpError):
        ntp.ntp_edge_softmax(g, dev_f32(p), dev_f32(q), 0.2, a_in, torch.empty_like(a_in))
    r_in, r_out = oracle.edge_softmax(og, p, q, 0.2)
    f = 48
    x = gen.normal_features(n, f, seed=2)
    y = torch.full((n, f), float("nan"), device="cuda:0")
    ntp.ntp_aggregate_weighted(g, ntp.NTP_BWD, a_in, dev_f32(x), y, f, f, f)
    torch.cuda.synchronize()
    ref, ref_abs = oracle.aggregate(oracle.weighted(og, r_in, r_out).csc, x, with_abs=True)
    assert_close(y.cpu().numpy(), ref, ref_abs, TOL_F32, "scatter with attention weights")
    g.close()


def test_attention_argument_errors(hub):
    import torch
    from gpu_util import dev_f32
    n, src, dst, g, og = hub
    p, q = _scores(n, 1)
    a = torch.empty(og.csr.nnz, device="cuda:0")
    with pytest.raises(ntp.NtpError):
        ntp.ntp_edge_softmax(g, dev_f32(p), dev_f32(q), -0.5, a)
    with pytest.raises(ntp.NtpError):
        ntp.ntp_edge_softmax(g, None, dev_f32(q), 0.2, a)
    streamed = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS | ntp.NTP_FORCE_STREAM, chunk_edges=5000)
    with pytest.raises(ntp.NtpError) as e:
        ntp.ntp_edge_softmax(streamed, dev_f32(p), dev_f32(q), 0.2, a)
    assert e.value.code == ntp.NTP_EBUDGET
    streamed.close()
    with pytest.raises(ntp.NtpError):
        ntp.ntp_aggregate_weighted(g, 7, a, a, a, 4, 4, 4)


@pytest.mark.parametrize("chunk_edges", [101, 700, 5003])
def test_attention_weights_on_a_chunked_resident_graph(hub, chunk_edges):
    """several resident chunks, among them pieces of the hub's row: the bits of the one-chunk graph"""
    import torch
    n, src, dst, g, og = hub
    p, q = _scores(n, 12)
    a_in, a_out = _device_alpha(g, og.csr.nnz, p, q, 0.2)
    gc = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS, chunk_edges=chunk_edges)
    assert ntp.ntp_graph_info(gc)["n_chunks"] > 1
    c_in, c_out = _device_alpha(gc, og.csr.nnz, p, q, 0.2)
    _check_alpha(og, c_in, c_out, p, q, 0.2, "chunked %d" % chunk_edges)
    if chunk_edges >= 5003:          # same segments as the one-chunk plan: identical reduction trees
        assert torch.equal(a_in, c_in) and torch.equal(a_out, c_out)
    gc.close()


# ---- gradient of the scores through the attention weights (ntp_edge_softmax_bwd) ---------------
TOL_SCORE_GRAD = 1e-5     # relative to the sum of the magnitudes that enter each gradient


def _grad_scales(og, p, q, Z, dY, slope):
    """per vertex: sum over its edges of alpha (A + sum alpha A), A = |dY[v]| . |Z[u]| -- the
    magnitude of everything that is added up to form dq[v] (by destination) and dp[u] (by source)"""
    a_in, _ = oracle.edge_softmax(og, p, q, slope)
    n = og.n
    rp, ci = og.csr.rowptr, og.csr.colidx
    rows = np.repeat(np.arange(n), np.diff(rp))
    A = np.einsum("ej,ej->e", np.abs(dY.astype(np.float64))[rows], np.abs(Z.astype(np.float64))[ci])
    tA = np.zeros(n)
    np.add.at(tA, rows, a_in * A)
    mag = a_in * (A + tA[rows])
    sq = np.zeros(n)
    sp = np.zeros(n)
    np.add.at(sq, rows, mag)
    np.add.at(sp, ci, mag)
    return sp, sq


def _score_grad_case(g, og, m, slope, seed, what, ldz=None, lddy=None, scale=1.0):
    import torch
    from gpu_util import dev_f32
    n, nnz = og.n, og.csr.nnz
    ldz = ldz or m
    lddy = lddy or m
    p, q = _scores(n, seed)
    rng = gen.stream_rng(seed, 77)
    Z = (rng.normal(size=(n, m)) * scale).astype(np.float32)
    dY = (rng.normal(size=(n, m)) * scale).astype(np.float32)
    say("   score gradient: %s n=%d nnz=%d m=%d ldz=%d lddy=%d slope=%g" % (what, n, nnz, m, ldz, lddy, slope))
    a_in, a_out = _device_alpha(g, nnz, p, q, slope)
    Zd = torch.full((n, ldz), float("nan"), device="cuda:0")
    Zd[:, :m] = dev_f32(Z)
    dYd = torch.full((n, lddy), float("nan"), device="cuda:0")
    dYd[:, :m] = dev_f32(dY)
    dp = torch.full((n,), float("nan"), device="cuda:0")
    dq = torch.full((n,), float("nan"), device="cuda:0")
    ntp.ntp_edge_softmax_bwd(g, dev_f32(p), dev_f32(q), slope, a_in, a_out, Zd, dYd, m, ldz, lddy, dp, dq)
    torch.cuda.synchronize()
    r_dp, r_dq, _, _ = oracle.edge_softmax_bwd(og, p, q, Z, dY, slope)
    sp, sq = _grad_scales(og, p, q, Z, dY, slope)
    got_p = dp.cpu().numpy().astype(np.float64)
    got_q = dq.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got_p)) and np.all(np.isfinite(got_q)), what
    tiny = np.finfo(np.float32).tiny
    ep = np.abs(got_p - r_dp) / np.maximum(sp, tiny)
    eq = np.abs(got_q - r_dq) / np.maximum(sq, tiny)
    say("      max |err| / scale: dp %.2e dq %.2e" % (ep.max(), eq.max()))
    assert ep.max() <= TOL_SCORE_GRAD and eq.max() <= TOL_SCORE_GRAD, what
    # normwise as well: the gradients as vectors
    assert np.abs(got_p - r_dp).max() <= TOL_SCORE_GRAD * sp.max()
    assert np.abs(got_q - r_dq).max() <= TOL_SCORE_GRAD * sq.max()
    return dp, dq


@pytest.mark.parametrize("m", [1, 8, 40, 50, 64, 128, 256, 1024])
def test_score_gradient_widths(hub, m):
    n, src, dst, g, og = hub
    _score_grad_case(g, og, m, 0.2, 40 + m, "hub graph")


@pytest.mark.parametrize("segments", [700, 730, 1100])
@pytest.mark.parametrize("flags", [0, ntp.NTP_EDGE_PERM])
def test_a_row_of_many_segments(segments, flags):
    """a star: up to 724 segments combine their row's partial sums themselves, more leave it to a launch in between"""
    n = 256 * segments + 1
    src, dst = np.arange(1, n, dtype=np.int32), np.zeros(n - 1, np.int32)
    og = oracle.build_graph(n, src, dst, 0)
    g = ntp.ntp_graph_build(n, src, dst, flags=flags)
    p, q = _scores(n, segments)
    _check_alpha(og, *_device_alpha(g, og.csr.nnz, p, q, 0.2), p, q, 0.2, "star of %d segments" % segments)
    _score_grad_case(g, og, 8, 0.2, segments, "star")
    g.close()


@pytest.mark.parametrize("slope", [0.0, 1.0])
def test_score_gradient_slopes(hub, slope):
    n, src, dst, g, og = hub
    _score_grad_case(g, og, 64, slope, 5, "hub graph")


def test_score_gradient_strided_and_unaligned(hub):
    n, src, dst, g, og = hub
    _score_grad_case(g, og, 64, 0.2, 8, "padded rows", ldz=80, lddy=96)
    _score_grad_case(g, og, 64, 0.2, 9, "odd strides (scalar loads)", ldz=67, lddy=65)
    _score_grad_case(g, og, 24, 0.2, 10, "large values", scale=50.0)


def test_score_gradient_degree_edge_cases():
    degs = [1, 2, 3, 4, 5, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257,
            511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 5000]
    n = 6000
    rng = gen.stream_rng(6, 1)
    src, dst = [], []
    for v, d in enumerate(degs):
        others = rng.choice(np.setdiff1d(np.arange(n), [v]), size=d - 1, replace=False)
        src.append(others)
        dst.append(np.full(d - 1, v))
    # and sources with many out-edges: vertex 100 + i points at i * 37 vertices
    for i in range(1, 40):
        u = 100 + i
        src.append(np.full(i * 37, u))
        dst.append(rng.choice(np.setdiff1d(np.arange(n), [u]), size=i * 37, replace=False))
    src = np.concatenate(src).astype(np.int32)
    dst = np.concatenate(dst).astype(np.int32)
    og = oracle.build_graph(n, src, dst, oracle.DIRECTED_GCN_FLAGS)
    g = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS)
    _score_grad_case(g, og, 32, 0.2, 11, "degree edge cases")
    _score_grad_case(g, og, 20, 0.2, 12, "degree edge cases")
    g.close()


def test_score_gradient_symmetric_and_configs():
    for cfg, scale, m in ((1, 1, 16), (2, 1, 64), (4, 64, 76)):
        n, src, dst = gen.make_graph(cfg, seed=0, scale_down=scale)
        og = oracle.build_graph(n, src, dst, oracle.GCN_FLAGS)
        g = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_GCN_FLAGS)
        _score_grad_case(g, og, m, 0.2, 20 + cfg, "config %d" % cfg)
        g.close()


def test_score_gradient_on_a_chunked_resident_graph(hub):
    """several resident chunks: same plan of whole rows and segments -> the bits of the one-chunk
    graph; smaller chunks cut the hub's rows into pieces that lie in several chunks"""
    import torch
    n, src, dst, g, og = hub
    d1 = _score_grad_case(g, og, 64, 0.2, 13, "one chunk")
    for chunk_edges in (5003, 700, 101):
        gc = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS, chunk_edges=chunk_edges)
        assert ntp.ntp_graph_info(gc)["n_chunks"] > 1
        d2 = _score_grad_case(gc, og, 64, 0.2, 13, "chunks of %d edges" % chunk_edges)
        if chunk_edges == 5003:
            assert torch.equal(d1[0], d2[0]) and torch.equal(d1[1], d2[1])
        gc.close()


def test_score_gradient_argument_errors(hub):
    import torch
    n, src, dst, g, og = hub
    a = torch.zeros(og.csr.nnz, device="cuda:0")
    s = torch.zeros(n, device="cuda:0")
    v = torch.zeros(n, 1100, device="cuda:0")
    out = torch.empty(n, device="cuda:0")
    for m, ldz, lddy in ((0, 8, 8), (1025, 1100, 1100), (64, 32, 64), (64, 64, 32)):
        with pytest.raises(ntp.NtpError) as e:
            ntp.ntp_edge_softmax_bwd(g, s, s, 0.2, a, a, v, v, m, ldz, lddy, out, out.clone())
        assert e.value.code == ntp.NTP_EINVAL
    with pytest.raises(ntp.NtpError):
        ntp.ntp_edge_softmax_bwd(g, s, s, 0.2, a, None, v, v, 8, 1100, 1100, out, out.clone())
    with pytest.raises(ntp.NtpError) as e:      # wider than the scalar-load path takes
        ntp.ntp_edge_softmax_bwd(g, s, s, 0.2, a, a, v, v, 301, 1100, 1100, out, out.clone())
    assert e.value.code == ntp.NTP_EUNSUPPORTED
    one_form = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS | ntp.NTP_SCATTER_BWD)
    with pytest.raises(ntp.NtpError) as e:
        ntp.ntp_edge_softmax_bwd(one_form, s, s, 0.2, a, a, v, v, 8, 1100, 1100, out, out.clone())
    assert e.value.code == ntp.NTP_EUNSUPPORTED
    one_form.close()


# ---- the same gradient on graphs built with NTP_EDGE_PERM (one dot product per edge) -----------
PERM = ntp.NTP_EDGE_PERM


@pytest.fixture(scope="module")
def hub_perm():
    n = 3000
    src, dst = gen.directed_random_edges(n, 40000, 21, hub=5, hub_in=2600, hub_out=900)
    og = oracle.build_graph(n, src, dst, oracle.DIRECTED_GCN_FLAGS)
    g = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS | PERM)
    assert np.array_equal(ntp.ntp_graph_export_perm(g), oracle.edge_permutation(og))
    yield n, src, dst, g, og
    g.close()


@pytest.mark.parametrize("m", [1, 8, 50, 64, 256, 1024])
def test_score_gradient_by_permutation_widths(hub_perm, m):
    n, src, dst, g, og = hub_perm
    _score_grad_case(g, og, m, 0.2, 140 + m, "hub graph with edge permutation")


def test_score_gradient_by_permutation_slopes_and_strides(hub_perm):
    n, src, dst, g, og = hub_perm
    _score_grad_case(g, og, 64, 0.0, 15, "slope 0")
    _score_grad_case(g, og, 64, 1.0, 16, "slope 1")
    _score_grad_case(g, og, 64, 0.2, 17, "odd strides", ldz=67, lddy=65)


def test_score_gradient_by_permutation_symmetric_chunked_and_sparse():
    import torch
    for cfg, scale, m in ((1, 1, 16), (2, 1, 64), (4, 64, 76)):
        n, src, dst = gen.make_graph(cfg, seed=0, scale_down=scale)
        og = oracle.build_graph(n, src, dst, oracle.GCN_FLAGS)
        g = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_GCN_FLAGS | PERM)
        _score_grad_case(g, og, m, 0.2, 30 + cfg, "config %d with edge permutation" % cfg)
        g.close()
    n = 3000
    src, dst = gen.directed_random_edges(n, 40000, 21, hub=5, hub_in=2600, hub_out=900)
    og = oracle.build_graph(n, src, dst, oracle.DIRECTED_GCN_FLAGS)
    for chunk_edges in (5003, 700, 101):
        gc = ntp.ntp_graph_build(n, src, dst, flags=ntp.NTP_DIRECTED_GCN_FLAGS | PERM, chunk_edges=chunk_edges)
        _score_grad_case(gc, og, 32, 0.2, 19, "chunks of %d edges with edge permutation" % chunk_edges)
        gc.close()
    # fewer stored entries than vertices (no self loops, most vertices without edges)
    n = 5000
    src, dst = gen.directed_random_edges(n, 900, 5)
    flags = oracle.DEDUP
    og = oracle.build_graph(n, src, dst, flags)
    assert og.csr.nnz < n
    for extra in (0, PERM):
        g = ntp.ntp_graph_build(n, src, dst, flags=flags | extra)
        _score_grad_case(g, og, 16, 0.2, 23, "sparse graph without self loops, flags +%d" % extra)
        g.close()


def test_score_gradient_accumulates_over_calls(hub, hub_perm):
    """accumulate = 1 adds the call's gradient to what dp, dq hold, with and without the permutation"""
    import torch
    from gpu_util import dev_f32
    for n, src, dst, g, og in (hub, hub_perm):
        nnz, m = og.csr.nnz, 24
        p, q = _scores(n, 31)
        rng = gen.stream_rng(31, 78)
        Z1, dY1, Z2, dY2 = (rng.normal(size=(n, m)).astype(np.float32) for _ in range(4))
        a_in, a_out = _device_alpha(g, nnz, p, q, 0.2)
        dp = torch.full((n,), float("nan"), device="cuda:0")
        dq = torch.full((n,), float("nan"), device="cuda:0")
        pd, qd = dev_f32(p), dev_f32(q)
        ntp.ntp_edge_softmax_bwd(g, pd, qd, 0.2, a_in, a_out, dev_f32(Z1), dev_f32(dY1), m, m, m, dp, dq, False)
        first = (dp.clone(), dq.clone())
        ntp.ntp_edge_softmax_bwd(g, pd, qd, 0.2, a_in, a_out, dev_f32(Z2), dev_f32(dY2), m, m, m, dp, dq, True)
        torch.cuda.synchronize()
        r1 = oracle.edge_softmax_bwd(og, p, q, Z1, dY1, 0.2)
        r2 = oracle.edge_softmax_bwd(og, p, q, Z2, dY2, 0.2)
        s1 = _grad_scales(og, p, q, Z1, dY1, 0.2)
        s2 = _grad_scales(og, p, q, Z2, dY2, 0.2)
        tiny = np.finfo(np.float32).tiny
        for got, a, b, sa, sb in ((dp, r1[0], r2[0], s1[0], s2[0]), (dq, r1[1], r2[1], s1[1], s2[1])):
            err = np.abs(got.cpu().numpy().astype(np.float64) - (a + b)) / np.maximum(sa + sb, tiny)
            assert err.max() <= TOL_SCORE_GRAD
        # and the second call alone, subtracted back, is what a fresh call gives (to rounding)
        dp2 = torch.empty_like(dp)
        dq2 = torch.empty_like(dq)
        ntp.ntp_edge_softmax_bwd(g, pd, qd, 0.2, a_in, a_out, dev_f32(Z2), dev_f32(dY2), m, m, m, dp2, dq2, False)
        torch.cuda.synchronize()
        assert torch.equal(first[0] + dp2, dp) and torch.equal(first[1] + dq2, dq)



def test_score_gradients_summed_in_one_buffer(hub, hub_perm):
    """dp and dq may be the same accumulated buffer: it gains dq, then dp (the sums of split rows come last otherwise)"""
    import torch
    from gpu_util import dev_f32
    for n, src, dst, g, og in (hub, hub_perm):
        nnz, m = og.csr.nnz, 24
        p, q = _scores(n, 33)
        rng = gen.stream_rng(33, 79)
        Z, dY = (dev_f32(rng.normal(size=(n, m)).astype(np.float32)) for _ in range(2))
        a_in, a_out = _device_alpha(g, nnz, p, q, 0.2)
        pd, qd = dev_f32(p), dev_f32(q)
        dp, dq = torch.empty(n, device="cuda:0"), torch.empty(n, device="cuda:0")
        ntp.ntp_edge_softmax_bwd(g, pd, qd, 0.2, a_in, a_out, Z, dY, m, m, m, dp, dq, False)
        both = dev_f32(rng.normal(size=n).astype(np.float32))
        want = (both + dq) + dp
        ntp.ntp_edge_softmax_bwd(g, pd, qd, 0.2, a_in, a_out, Z, dY, m, m, m, both, both, True)
        assert torch.equal(both, want)


def test_two_heads_on_column_blocks(hub):
    """several attention heads = one call per head on its block of columns of a wider matrix
    (row strides, offset base pointers): each head's results equal those of a separate compact run"""
    import torch
    from gpu_util import dev_f32
    n, src, dst, g, og = hub
    nnz, c = og.csr.nnz, 12                 # two heads of 12 columns in rows of 24 (+ 8 padding)
    ld = 32
    rng = gen.stream_rng(55, 3)
    Z = rng.normal(size=(n, 2 * c)).astype(np.float32)
    dY = rng.normal(size=(n, 2 * c)).astype(np.float32)
    Zd = torch.full((n, ld), float("nan"), device="cuda:0")
    dYd = torch.full((n, ld), float("nan"), device="cuda:0")
    Zd[:, :2 * c] = dev_f32(Z)
    dYd[:, :2 * c] = dev_f32(dY)
    Yd = torch.full((n, ld), float("nan"), device="cuda:0")
    for h in range(2):
        p, q = _scores(n, 60 + h)
        a_in, a_out = _device_alpha(g, nnz, p, q, 0.2)
        cols = slice(h * c, (h + 1) * c)
        # forward aggregation of the head's columns with its weights, in place in the wide buffers
        ntp.ntp_aggregate_weighted(g, ntp.NTP_FWD, a_in, Zd[:, cols], Yd[:, cols], c, ld, ld)
        dp = torch.empty(n, device="cuda:0")
        dq = torch.empty(n, device="cuda:0")
        ntp.ntp_edge_softmax_bwd(g, dev_f32(p), dev_f32(q), 0.2, a_in, a_out, Zd[:, cols], dYd[:, cols], c, ld, ld, dp, dq)
        torch.cuda.synchronize()
        r_in, r_out = oracle.edge_softmax(og, p, q, 0.2)
        ref, ref_abs = oracle.aggregate(oracle.weighted(og, r_in, r_out).csr, Z[:, cols], with_abs=True)
        got = Yd[:, cols].cpu().numpy().astype(np.float64)
        assert (np.abs(got - ref) / np.maximum(ref_abs, 1e-300)).max() <= 2e-5, "head %d forward" % h
        r_dp, r_dq, _, _ = oracle.edge_softmax_bwd(og, p, q, Z[:, cols], dY[:, cols], 0.2)
        sp, sq = _grad_scales(og, p, q, Z[:, cols], dY[:, cols], 0.2)
        tiny = np.finfo(np.float32).tiny
        assert (np.abs(dp.cpu().numpy() - r_dp) / np.maximum(sp, tiny)).max() <= TOL_SCORE_GRAD, "head %d dp" % h
        assert (np.abs(dq.cpu().numpy() - r_dq) / np.maximum(sq, tiny)).max() <= TOL_SCORE_GRAD, "head %d dq" % h
    assert torch.isnan(Yd[:, 2 * c:]).all()          # padding columns untouched
