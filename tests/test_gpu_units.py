"""The unit a workgroup chooses for its own sketch terms, and what it does where that unit does not hold:
one workgroup out of range among many, drifts that no sample of the chunk sees, chunks without any drift,
and the kernels that redo a sketch in several windows (one worker slot), skewed, placed and plain layouts
and several row groups.  Always against the oracle."""
import numpy as np
import pytest
import torch

import fda_synth as S
from fda_tolerance import check_cells
from oracle import fda_oracle as O

pytestmark = pytest.mark.gpu
RTOL = 1e-5
DEV = "cuda:0"


def drifts(kind, K, d, g):
    u = torch.randn((K, d), generator=g, device=DEV) * 1e-4
    if kind == "outlier":                 # one worker of one chunk, off the sampled runs of 8
        u[K - 1, d // 2 + 13] = 0.9
    elif kind == "sparse":                # nothing but a few coordinates move
        keep = torch.zeros(d, dtype=torch.bool, device=DEV)
        keep[torch.randint(0, d, (9,), generator=g, device=DEV)] = True
        u *= keep
    elif kind == "frozen":                # most chunks do not move at all, one coordinate among them does
        u[:, : 3 * d // 4] = 0.0
        u[0, d // 3] = 2e-4
    elif kind == "uneven":                # a layer whose drifts are 10^4 times the others'
        u[:, d // 4: d // 4 + d // 50 + 1] *= 1e4
    return u


@pytest.mark.parametrize("kind", ["outlier", "sparse", "frozen", "uneven"])
@pytest.mark.parametrize("K,d,l,m,dtype", [
    (1, 90_001, 3, 500, "f32"),           # one slot, plain rows: redone in two windows
    (2, 60_003, 2, 5000, "f32"),          # two slots, plain rows
    (3, 70_001, 5, 251, "bf16"),          # four slots with a spare one, skewed and placed
    (8, 120_007, 9, 250, "bf16"),         # nine rows (the widest workgroup), four slots
    (20, 50_001, 5, 33, "f32"),           # six slots, placed; more workers than the mean-state pass samples
])
def test_units_and_redo(kind, K, d, l, m, dtype):
    import paper_2405_20988_amd as F
    g = torch.Generator(device=DEV)
    g.manual_seed(40 + K)
    w_t0 = (torch.randn(d, generator=g, device=DEV) * 0.05).to(torch.bfloat16).float()
    xi = torch.randn(d, generator=g, device=DEV) / d ** 0.5
    w = (w_t0 + drifts(kind, K, d, g)).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    coef = S.hash_coefficients(40 + K, l)
    mon = F.FdaMonitor(K, d, dtype, 3, l, m, 0.06, coef, device=DEV)
    w_host, w0_host, xi_host = S.slab_to_numpy(w), w_t0.cpu().numpy(), xi.cpu().numpy()
    ref = O.local_state(w_host, dtype, w0_host, xi_host, coef, m)
    mref = O.mean_state(w_host, dtype, w0_host, xi_host, coef, m)
    for _ in range(2):                    # the second call starts from what the first one left
        mon.local_state(w, w_t0, xi)
        n, p, sk = mon.state_numpy()
        assert np.allclose(n, ref["n"], rtol=RTOL, atol=0)
        assert (np.abs(p - ref["p"]) <= RTOL * ref["p_abs"] + 1e-30).all()
        check_cells(sk, ref["sk"], ref["sk_abs"], ref["sk_cnt"], ref["u_mean_abs"])
        path = mon.last_state_path()
        assert mon.estimate_variance(1e30).state_path == path
        if kind == "outlier" and dtype == "f32":
            assert path >= 1
        mon.mean_state(w, w_t0, xi)
        nb, pb, skb = mon.mean_numpy()
        assert nb == pytest.approx(mref["n"], rel=RTOL)
        assert abs(pb - mref["p"]) <= RTOL * mref["p_abs"] + 1e-30
        check_cells(skb, mref["sk"], mref["sk_abs"], mref["sk_cnt"], mref["u_mean_abs"])
    mon.close()


@pytest.mark.parametrize("K,d,l,m,dtype,groups,mean_groups", [
    (1, 5_003, 9, 33, "f32", 1, 1),         # one slot, plain rows of 16-bit or 11-bit fields
    (1, 5_003, 9, 1025, "bf16", 1, 1),
    (2, 2_047, 9, 1100, "bf16", 1, 1),      # two slots, nine fields of 13 bits, placement groups of three rows
    (4, 2_049, 9, 250, "f32", 1, 1),        # four slots: all registers of a wave
    (3, 70_001, 9, 1, "bf16", 1, 1),
    (5, 20_001, 9, 2200, "f32", 3, 1),      # the state pass splits the rows, the mean-state pass does not
    (3, 9_001, 10, 64, "f32", 2, 2),         # the first sketch of two row groups
])
def test_nine_rows_in_one_workgroup(K, d, l, m, dtype, groups, mean_groups):
    """Integer-valued drifts: states and average state bit for bit, so every field of every record is checked."""
    import paper_2405_20988_amd as F
    g = torch.Generator(device=DEV)
    g.manual_seed(K + l)
    w_t0 = torch.zeros(d, device=DEV)
    xi = torch.zeros(d, device=DEV)
    w = torch.randint(-4, 5, (K, d), generator=g, device=DEV).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    coef = S.hash_coefficients(7, l)
    mon = F.FdaMonitor(K, d, dtype, 3, l, m, 0.06, coef, device=DEV)
    assert mon.plan["row_groups"] == groups and mon.plan["mean_row_groups"] == mean_groups
    ref = O.local_state(S.slab_to_numpy(w), dtype, w_t0.cpu().numpy(), xi.cpu().numpy(), coef, m)
    mon.local_state(w, w_t0, xi)
    n, _, sk = mon.state_numpy()
    assert np.array_equal(n, ref["n"].astype(np.float32)) and np.array_equal(sk, ref["sk"].astype(np.float32))
    mon.mean_state(w, w_t0, xi)
    _, _, skb = mon.mean_numpy()
    assert np.array_equal(skb, (ref["sk"].sum(axis=0) / K).astype(np.float32))
    mon.close()


@pytest.mark.parametrize("K,d,l,m", [(1, 5, 1, 1), (2, 70_001, 1, 31), (17, 30_001, 2, 33), (33, 9_001, 3, 257),
                                     (5, 400_001, 16, 64), (40, 2_049, 8, 1000)])
def test_step_estimate_equals_estimate_of_its_states(K, d, l, m):
    """fda_step takes the estimate in the launch that merges the partials, fda_estimate_variance from the
    states: the same bits, whatever the number of workers, cells and partitions."""
    import paper_2405_20988_amd as F
    g = torch.Generator(device=DEV)
    g.manual_seed(K)
    w_t0 = torch.randn(d, generator=g, device=DEV) * 0.05
    xi = torch.randn(d, generator=g, device=DEV) / d ** 0.5
    w = w_t0 + torch.randn((K, d), generator=g, device=DEV) * 1e-3
    mon = F.FdaMonitor(K, d, "f32", 3, l, m, 0.06, S.hash_coefficients(K, l), device=DEV)
    w_prev = w_t0.clone()
    for mean in (False, True, False):
        a = mon.step(w, w_t0, w_prev, xi, 1e30, mean=mean, want_host=True).as_dict()
        b = (mon.estimate_variance_mean(1e30) if mean else mon.estimate_variance(1e30)).as_dict()
        assert a == b
    mon.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [1, 63, 1023, 1024, 1025, 70_003, 1_572_863, 1_572_864, 1_577_059])
def test_sync_stores_rows_at_every_alignment(dtype, d):
    """Rows are stored in vectors counted from their own first line boundary: row lengths and row starts off
    every boundary, block remainders on both sides of the small blocks' limit; nothing outside the rows moves."""
    import paper_2405_20988_amd as F
    from paper_2405_20988_amd import binding as B
    K, pad = 4, 37                                   # (a division by 4 is exact: torch may multiply by 1 / K)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    for first in (0, 1, 6, 63):                      # element offset of the slab in its allocation
        buf = torch.full((first + K * (d + pad) + 64,), 7.0, device=DEV, dtype=tdt)
        w = buf[first:first + K * (d + pad)].view(K, d + pad)[:, :d]
        w.copy_((torch.randn((K, d), generator=g, device=DEV) * 0.05).to(tdt))
        rows = w.clone()
        w_t0 = torch.randn(d, generator=g, device=DEV) * 0.05
        old = w_t0.clone()
        w_prev, xi, w_bar = torch.zeros_like(w_t0), torch.zeros_like(w_t0), torch.zeros_like(w_t0)
        mon = F.FdaMonitor(K, d, dtype, 3, 1, 7, 0.06, S.hash_coefficients(1, 1), row_stride=d + pad, device=DEV)
        st = torch.cuda.current_stream().cuda_stream
        mean = torch.zeros_like(w_t0)
        for k in range(K):
            mean += rows[k].float()
        mean /= K
        for from_mean in (False, True):
            w.copy_(rows)
            w_t0.copy_(old)
            if from_mean:
                B.fda_mean_state(mon.ctx, w.data_ptr(), w_t0.data_ptr(), xi.data_ptr(), mon.mean.data_ptr(),
                                 w_bar.data_ptr(), st)
                B.fda_sync_from_mean(mon.ctx, w.data_ptr(), w_t0.data_ptr(), w_prev.data_ptr(), xi.data_ptr(),
                                     w_bar.data_ptr(), None, st)
                want = w_bar
                assert torch.allclose(want, mean, rtol=1e-5, atol=1e-7)
            else:
                B.fda_sync_xi(mon.ctx, w.data_ptr(), w_t0.data_ptr(), w_prev.data_ptr(), xi.data_ptr(), None, st)
                want = mean
            assert torch.equal(w_t0, want) and torch.equal(w_prev, old)
            assert torch.equal(w, want.to(tdt).expand(K, d))
            assert float(xi.double().norm()) == pytest.approx(1.0, rel=1e-5)
            out = buf.clone()
            out[first:first + K * (d + pad)].view(K, d + pad)[:, :d] = 7.0
            assert (out == 7.0).all()
        mon.close()


def test_results_read_back_by_more_contexts_than_there_are_places():
    """Results reach the host through 64 pinned places of the process; contexts beyond those get copies, and
    places come back when contexts are destroyed.  From several threads, each on a stream of its own."""
    import threading

    import paper_2405_20988_amd as F
    d, K, errors = 4097, 3, []

    def work(t):
        try:
            g = torch.Generator(device=DEV)
            g.manual_seed(t)
            with torch.cuda.stream(torch.cuda.Stream()):
                w_t0 = torch.randn(d, generator=g, device=DEV) * 0.05
                xi = torch.randn(d, generator=g, device=DEV) / d ** 0.5
                w = w_t0 + torch.randn((K, d), generator=g, device=DEV) * 1e-3
                w_prev = w_t0.clone()
                for _ in range(2):
                    mons = [F.FdaMonitor(K, d, "f32", 3, 3, 50, 0.06, S.hash_coefficients(q, 3), device=DEV)
                            for q in range(30)]
                    for mon in mons:
                        est = mon.step(w, w_t0, w_prev, xi, 1e30, want_host=True)
                        dev = F.FdaEstimate.from_buffer_copy(mon.est_dev.cpu().numpy().tobytes())
                        assert est.as_dict() == dev.as_dict() and est.mean_sqnorm > 0
                    mons[0].step(w, w_t0, w_prev, xi, 0.0, want_host=True)      # fires: waits for the rows too
                    assert torch.equal(w[0], w_t0) and torch.equal(w[2], w_t0)
                    w += torch.randn((K, d), generator=g, device=DEV) * 1e-3
                    for mon in mons:
                        mon.close()
        except Exception as exc:                     # noqa: BLE001 -- reported by the main thread
            errors.append(exc)
    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


@pytest.mark.parametrize("K,d,l,m,dtype,slots", [(3, 2_100_001, 2, 60, "f32", 4), (4, 2_600_003, 2, 60, "bf16", 4),
                                                 (6, 4_200_001, 2, 60, "f32", 6), (6, 4_200_001, 3, 31, "bf16", 6),
                                                 (8, 6_000_001, 1, 33, "f32", 8), (8, 6_000_001, 2, 31, "bf16", 8)])
def test_kernels_with_many_worker_slots(K, d, l, m, dtype, slots):
    """Short launches take more groups of two workers; these are long enough for four, six and eight."""
    import paper_2405_20988_amd as F
    g = torch.Generator(device=DEV)
    g.manual_seed(K + d)
    w_t0 = torch.randn(d, generator=g, device=DEV) * 0.05
    w = (w_t0 + torch.randn((K, d), generator=g, device=DEV) * 1e-3).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    xi = torch.randn(d, generator=g, device=DEV) / d ** 0.5
    coef = S.hash_coefficients(K, l)
    mon = F.FdaMonitor(K, d, dtype, 3, l, m, 0.06, coef, device=DEV)
    assert (mon.plan["worker_groups"], mon.plan["worker_slots"]) == (1, slots), mon.plan
    mon.local_state(w, w_t0, xi)
    n, p, sk = mon.state_numpy()
    ref = O.local_state(S.slab_to_numpy(w), dtype, w_t0.cpu().numpy(), xi.cpu().numpy(), coef, m)
    assert np.allclose(n, ref["n"], rtol=RTOL, atol=0)
    assert (np.abs(p - ref["p"]) <= RTOL * ref["p_abs"] + 1e-30).all()
    check_cells(sk, ref["sk"], ref["sk_abs"], ref["sk_cnt"], ref["u_mean_abs"])
    assert mon.last_state_path() == 0
    mon.close()


def test_step_refuses_a_misaligned_w_prev_whatever_it_decides():
    import paper_2405_20988_amd as F
    from paper_2405_20988_amd import binding as B
    K, d = 3, 5000
    w_t0 = torch.zeros(d, device=DEV)
    xi = torch.zeros(d, device=DEV)
    w = torch.ones((K, d), device=DEV)
    w_prev = torch.zeros(d + 1, device=DEV)
    mon = F.FdaMonitor(K, d, "f32", 3, 3, 50, 0.06, S.hash_coefficients(1, 3), device=DEV)
    for want_host in (False, True):
        with pytest.raises(F.FdaError):
            B.fda_step(mon.ctx, w.data_ptr(), w_t0.data_ptr(), w_prev.data_ptr() + 2, xi.data_ptr(),
                       mon.state.data_ptr(), None, 1e30, 1e-5, B.FDA_VARIANT_LINEAR, 0, mon.est_dev.data_ptr(),
                       want_host=want_host)
    mon.close()


@pytest.mark.parametrize("call", ["sync_xi", "linear_state"])
def test_eager_calls_between_the_capture_of_a_first_call_and_its_replay(call):
    """A context whose first call is only captured has no counters cleared yet; eager calls and, after them,
    several replays give what a context of its own gives."""
    import paper_2405_20988_amd as F
    K, d = 5, 200_003
    g = torch.Generator(device=DEV)
    g.manual_seed(9)
    w_t0 = torch.randn(d, generator=g, device=DEV) * 0.05
    w = w_t0 + torch.randn((K, d), generator=g, device=DEV) * 1e-3
    xi = torch.randn(d, generator=g, device=DEV) / d ** 0.5
    new = lambda: F.FdaMonitor(K, d, "f32", 1, 1, 1, 0.06, S.hash_coefficients(1, 1), device=DEV)
    mon, ref = new(), new()
    mon.workspace.fill_(0x5A)
    bufs = [[t.clone() for t in (w, w_t0, w_t0, xi)] for _ in range(2)]      # slab, w_t0, w_prev, xi

    def one(m, b):
        for dst, src in zip(b, (w, w_t0, w_t0, xi)):
            dst.copy_(src)
        if call == "sync_xi":
            m.sync_xi(*b)
        else:
            m.local_state(b[0], b[1], b[3])

    def check(m):
        torch.cuda.synchronize()
        assert torch.equal(m.state, ref.state) or call == "sync_xi"
        for x, y in zip(*bufs):
            assert torch.equal(x, y)
    one(ref, bufs[1])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        one(mon, bufs[0])
    one(mon, bufs[0])
    check(mon)
    for _ in range(3):
        bufs[0][3].zero_()
        mon.state.zero_()
        graph.replay()
        check(mon)
    mon.close()
    ref.close()


@pytest.mark.parametrize("first", ["local_state", "mean_state"])
@pytest.mark.parametrize("K,l,m", [(4, 5, 250), (1, 3, 64)])      # a table for each pass; one that both stream
def test_eager_sketches_between_the_capture_of_a_first_call_and_its_replay(first, K, l, m):
    """The hash tables that a captured first call records are not there yet when an eager call follows: it makes
    them itself.  States and average states are those of a context of its own, before and after the replays."""
    import paper_2405_20988_amd as F
    d = 30_011
    g = torch.Generator(device=DEV)
    g.manual_seed(K)
    w_t0 = torch.randn(d, generator=g, device=DEV) * 0.05
    w = w_t0 + torch.randn((K, d), generator=g, device=DEV) * 1e-3
    xi = torch.randn(d, generator=g, device=DEV) / d ** 0.5
    new = lambda: F.FdaMonitor(K, d, "f32", 3, l, m, 0.06, S.hash_coefficients(1, l), device=DEV)
    mon, ref = new(), new()
    ref.local_state(w, w_t0, xi)
    ref.mean_state(w, w_t0, xi)
    mon.workspace.fill_(0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        getattr(mon, first)(w, w_t0, xi)
    for replays in range(4):
        mon.state.zero_()
        mon.mean.zero_()
        mon.local_state(w, w_t0, xi)
        mon.mean_state(w, w_t0, xi)
        torch.cuda.synchronize()
        assert torch.equal(mon.state, ref.state) and torch.equal(mon.mean, ref.mean)
        out = mon.state if first == "local_state" else mon.mean
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(mon.state, ref.state) and torch.equal(mon.mean, ref.mean)
    mon.close()
    ref.close()


def test_contexts_are_destroyed_and_results_read_back_while_a_graph_is_captured():
    """The pinned page of the process is taken with the first result that is read back and goes with the last
    context: neither disturbs a capture on another stream."""
    import gc
    import threading

    import paper_2405_20988_amd as F
    gc.collect()
    K, d = 3, 5001
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    w_t0 = torch.randn(d, generator=g, device=DEV) * 0.05
    w = w_t0 + torch.randn((K, d), generator=g, device=DEV) * 1e-3
    xi = torch.randn(d, generator=g, device=DEV) / d ** 0.5
    other = torch.cuda.Stream()
    new = lambda: F.FdaMonitor(K, d, "f32", 3, 3, 50, 0.06, S.hash_coefficients(1, 3), device=DEV)
    mon, beside = new(), new()
    for m in (mon, beside):
        m.local_state(w, w_t0, xi)
    want = mon.state.clone()
    est, errors = [], []

    def read_back():
        try:
            with torch.cuda.stream(other):
                est.append(beside.estimate_variance(1e30))
            beside.close()                             # gives the page back
        except Exception as exc:                       # noqa: BLE001 -- reported below
            errors.append(exc)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mon.local_state(w, w_t0, xi)
        t = threading.Thread(target=read_back)
        t.start()
        t.join()
        mon.estimate_variance(1e30, want_host=False)
    assert not errors, errors
    for _ in range(3):
        mon.state.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(mon.state, want)
        dev = F.FdaEstimate.from_buffer_copy(mon.est_dev.cpu().numpy().tobytes())
        assert dev.as_dict() == est[0].as_dict()
    mon.close()


def test_kernel_times_are_read_while_a_graph_is_captured():
    """fda_profile_read waits for events of its own context: beside a capture on another stream that is allowed and
    leaves the capture whole."""
    import threading

    import paper_2405_20988_amd as F
    from paper_2405_20988_amd import binding as B
    K, d = 3, 5001
    g = torch.Generator(device=DEV)
    g.manual_seed(4)
    w_t0 = torch.randn(d, generator=g, device=DEV) * 0.05
    w = w_t0 + torch.randn((K, d), generator=g, device=DEV) * 1e-3
    xi = torch.randn(d, generator=g, device=DEV) / d ** 0.5
    mon, timed = (F.FdaMonitor(K, d, "f32", 3, 3, 50, 0.06, S.hash_coefficients(1, 3), device=DEV) for _ in range(2))
    mon.local_state(w, w_t0, xi)
    want = mon.state.clone()
    B.fda_profile_enable(timed.ctx, True)
    with torch.cuda.stream(torch.cuda.Stream()):
        timed.local_state(w, w_t0, xi)
    torch.cuda.synchronize()
    out = []

    def read():
        try:
            out.append(B.fda_profile_read(timed.ctx))
        except Exception as exc:                       # noqa: BLE001 -- compared below
            out.append(exc)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mon.local_state(w, w_t0, xi)
        t = threading.Thread(target=read)
        t.start()
        t.join()
    assert isinstance(out[0], tuple) and out[0][1] == 1, out
    for _ in range(3):
        mon.state.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(mon.state, want)
    mon.close()
    timed.close()


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("d", [1, 3, 1023, 1025, 4097, 1_572_863, 1_572_865, 44_739_242, 44_739_243, 100_663_297])
def test_update_xi_at_the_edges_of_its_blocks(d, shift):
    """Remainders of vectors and blocks, the sizes where the block size, the hints and the blocks per workgroup
    change, and vectors off 16 bytes.  Bound: the fp32 runs of four squares leave the norm within 2 * 2^-24, the
    rounded factor and the product add 2^-24 each."""
    import paper_2405_20988_amd as F
    g = torch.Generator(device=DEV)
    g.manual_seed(d)
    prev = torch.randn(d + shift, generator=g, device=DEV)[shift:]
    now = (torch.randn(d + shift, generator=g, device=DEV) * 1e-3)[shift:].add_(prev)
    buf = torch.full((d + shift + 8,), 7.0, device=DEV)
    mon = F.FdaMonitor(1, d, "bf16", 1, 1, 8, 0.06, S.hash_coefficients(1, 1), device=DEV)
    xi = buf[shift:shift + d]
    mon.update_xi(now, prev, xi)
    diff = (now - prev).double()
    want = diff / torch.linalg.vector_norm(diff)
    assert ((xi.double() - want).abs() <= 2.0 ** -22 * want.abs() + 1e-44).all()
    assert (buf[:shift] == 7.0).all() and (buf[shift + d:] == 7.0).all()
    mon.update_xi(now, now, xi)                          # no change: zeros
    assert not xi.any()
    mon.close()


@pytest.mark.parametrize("K,dtype", [(128, "f32"), (256, "bf16")])
def test_many_workers_of_a_small_model_are_synchronized(K, dtype):
    """Small blocks with streaming hints: a slab just beyond 512 MiB, rows off every line.  Whole numbers, whose mean
    over 2^k workers is exact."""
    import paper_2405_20988_amd as F
    d = 1_049_003
    g = torch.Generator(device=DEV)
    g.manual_seed(K)
    old = torch.randint(-8, 9, (d,), generator=g, device=DEV).float()
    storage = torch.float32 if dtype == "f32" else torch.bfloat16
    w = torch.empty((K, d), device=DEV, dtype=storage)
    mean = torch.zeros(d, device=DEV)
    for k in range(K):
        row = torch.randint(-8, 9, (d,), generator=g, device=DEV).float()
        mean += row
        w[k] = row
    mean /= K
    mon = F.FdaMonitor(K, d, dtype, 1, device=DEV)
    w_t0, w_prev, xi = old.clone(), torch.empty_like(old), torch.empty_like(old)
    want = (mean.double() - old.double()) / torch.linalg.vector_norm(mean.double() - old.double())
    mon.sync_xi(w, w_t0, w_prev, xi)
    assert torch.equal(w_t0, mean) and torch.equal(w_prev, old)
    assert bool((w == mean.to(storage)).all())
    assert torch.allclose(xi.double(), want, rtol=1e-6, atol=0)
    w_bar = torch.flip(mean, (0,)).contiguous()
    mon.sync_from_mean(w, w_t0, w_bar, w_prev)
    assert torch.equal(w_t0, w_bar) and torch.equal(w_prev, mean)
    assert bool((w == w_bar.to(storage)).all())
    mon.close()


@pytest.mark.parametrize("K,d", [(15, 5_001), (16, 5_001), (17, 1_023), (60, 30_001), (300, 5_003), (131, 70_001), (24, 262_147)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rows_split_over_workgroups(K, d, dtype):
    """fda_sync_from_mean stores the rows of a block from several workgroups: every row once, the models once."""
    import paper_2405_20988_amd as F
    g = torch.Generator(device=DEV)
    g.manual_seed(K)
    old, new = (torch.randn(d, generator=g, device=DEV) for _ in range(2))
    w = torch.randn((K, d), generator=g, device=DEV).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    mon = F.FdaMonitor(K, d, dtype, 1, device=DEV)
    w_t0, w_prev = old.clone(), torch.empty_like(old)
    mon.sync_from_mean(w, w_t0, new, w_prev)
    assert torch.equal(w_t0, new) and torch.equal(w_prev, old)
    assert bool((w == new.to(w.dtype)).all())
    mon.close()
