"""What a workgroup of a state pass does where its own fixed-point unit does not hold: the sums and the sketch that
it forms once more.  Always against the oracle."""
import numpy as np
import pytest
import torch

import fda_synth as S
from fda_tolerance import check_cells
from oracle import fda_oracle as O

pytestmark = pytest.mark.gpu
RTOL = 1e-5
DEV = "cuda:0"


def gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def check_both(w, w_t0, xi, dtype, l, m, seed, path=None, mean_path=None):
    """State and average state of the slab within the suite's tolerances; the passes' kinds of cell."""
    import paper_2405_20988_amd as F
    K, d = w.shape
    coef = S.hash_coefficients(seed, l)
    mon = F.FdaMonitor(K, d, dtype, 3, l, m, 0.06, coef, device=DEV)
    args = S.slab_to_numpy(w), dtype, w_t0.cpu().numpy(), xi.cpu().numpy(), coef, m
    ref, mref = O.local_state(*args), O.mean_state(*args)
    mon.local_state(w, w_t0, xi)
    n, p, sk = mon.state_numpy()
    assert np.isfinite(n).all() and np.allclose(n, ref["n"], rtol=RTOL, atol=0)
    assert (np.abs(p - ref["p"]) <= RTOL * ref["p_abs"] + 1e-30).all()
    check_cells(sk, ref["sk"], ref["sk_abs"], ref["sk_cnt"], ref["u_mean_abs"])
    got = mon.last_state_path()
    assert path is None or got in path, got
    assert mon.estimate_variance(1e30).nonfinite == 0
    mon.mean_state(w, w_t0, xi)
    nb, pb, skb = mon.mean_numpy()
    assert nb == pytest.approx(mref["n"], rel=RTOL)
    assert abs(pb - mref["p"]) <= RTOL * mref["p_abs"] + 1e-30
    check_cells(skb, mref["sk"], mref["sk_abs"], mref["sk_cnt"], mref["u_mean_abs"])
    assert mean_path is None or mon.last_mean_state_path() == mean_path
    mon.close()


@pytest.mark.parametrize("K,d,l,m,dtype", [(5, 100_001, 5, 250, "f32"), (2, 60_003, 9, 250, "f32"), (1, 70_001, 3, 500, "f32"),
                                           (8, 90_001, 7, 1000, "bf16"), (6, 50_001, 10, 64, "f32")])
def test_sums_where_most_of_a_chunk_hardly_moves(K, d, l, m, dtype):
    """Half of the model moves by 1e-3, the other half by 1e-20, except one coordinate of it that no workgroup
    samples (20 behind a multiple of 32; runs of 8 start at those): its square in units of the sampled drifts is
    2^150.  And a coordinate that rests at 1e14, which in those units is beyond fp32 itself."""
    g = gen(K)
    u = torch.randn((K, d), generator=g, device=DEV) * 1e-3
    half = d // 2
    u[:, half:] *= 1e-17
    w_t0 = torch.randn(d, generator=g, device=DEV) * 0.05
    w_t0[half:] = 0.0
    w_t0 = w_t0.to(torch.bfloat16).float()
    j = (half + 9_000) // 2048 * 2048 + 20 + 32 * 5
    u[:, j] = torch.randn(K, generator=g, device=DEV) * 1e-3
    w_t0[j + 2048] = 1e14
    w = (w_t0 + u).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    w_t0[j + 2048] = float(w[0, j + 2048])
    check_both(w, w_t0, torch.randn(d, generator=g, device=DEV) / d ** 0.5, dtype, l, m, K, path=(1, 2))


@pytest.mark.parametrize("size", [1e5, 1e6])
@pytest.mark.parametrize("together", [1, 2, 8])
@pytest.mark.parametrize("K,l,m", [(1, 1, 5000), (2, 1, 5000), (3, 1, 5000), (5, 2, 2000)])
def test_outliers_that_the_sample_sees(K, l, m, together, size):
    """The first coordinates of a chunk are a sampled run.  Drifts there, `size` times the others, do not coarsen the
    unit of the others: of the last worker, whose row spare worker slots repeat; one, two or a whole run of them."""
    import paper_2405_20988_amd as F
    d, g = 60_003, gen(K)
    plan = F.FdaMonitor(K, d, "f32", 3, l, m, 0.06, S.hash_coefficients(K, l), device=DEV).plan
    u = torch.randn((K, d), generator=g, device=DEV) * 1e-4
    for j in (plan["chunk"], 3 * plan["mean_chunk"]):
        u[K - 1, j:j + together] = 1e-4 * size
    w_t0 = torch.zeros(d, device=DEV)
    check_both(u, w_t0, torch.randn(d, generator=g, device=DEV) / d ** 0.5, "f32", l, m, K, path=(1, 2), mean_path=1)


@pytest.mark.parametrize("ratio", [2.0 ** 12, 2.0 ** 17, 2.0 ** 20, 2.0 ** 24])
@pytest.mark.parametrize("K,l,m,dtype", [(1, 3, 500, "f32"), (2, 1, 500, "bf16"), (3, 5, 250, "f32"), (8, 2, 500, "bf16")])
def test_a_redone_sketch_keeps_29_bits_of_the_other_drifts(K, l, m, dtype, ratio):
    """One workgroup's worth of coordinates, one drift `ratio` times the others'.  A cell is off by its own fp32
    rounding and by half a unit for each of its terms, with 2^29 units or more to a typical drift; the fp64 cells of the largest ratio are inside that too."""
    import paper_2405_20988_amd as F
    d, g = 2_000, gen(K)
    w = (torch.randn((K, d), generator=g, device=DEV) * 1e-3).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    w[K - 1, 700] = 1e-3 * ratio
    coef = S.hash_coefficients(K, l)
    mon = F.FdaMonitor(K, d, dtype, 3, l, m, 0.06, coef, device=DEV)
    zero = torch.zeros(d, device=DEV)
    ref = O.local_state(S.slab_to_numpy(w), dtype, zero.cpu().numpy(), zero.cpu().numpy(), coef, m)
    mon.local_state(w, zero, zero)
    n, _, sk = mon.state_numpy()
    assert mon.last_state_path() >= 1
    err = np.abs(sk.astype(np.float64) - ref["sk"])
    assert (err <= 2.0 ** -24 * np.abs(ref["sk"]) + ref["sk_cnt"][None] * 2.0 ** -30 * 0.8e-3 + 1e-45).all()
    assert np.allclose(n, ref["n"], rtol=2.0 ** -23, atol=0)
    mon.close()


@pytest.mark.parametrize("size", [2.0 ** 12, 2.0 ** 14, 2.0 ** 17])
@pytest.mark.parametrize("K,d,l,m,dtype", [(3, 2_049, 1, 16, "f32"), (2, 2_049, 3, 16, "bf16"), (6, 4_100, 2, 16, "f32"),
                                           (5, 10_245, 2, 32, "f32"), (8, 100_107, 1, 16, "f32"), (4, 300, 1, 16, "f32")])
def test_an_outlier_in_a_short_last_chunk(K, d, l, m, dtype, size):
    """The last workgroup has a few coordinates of its own, the last one of them `size` times the others: it leaves
    the other workers' drifts there their unit."""
    g = gen(d)
    w_t0 = torch.zeros(d, device=DEV)
    w = (torch.randn((K, d), generator=g, device=DEV) * 1e-3).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    w[K - 1, d - 1] = 1e-3 * size
    check_both(w, w_t0, torch.randn(d, generator=g, device=DEV) / d ** 0.5, dtype, l, m, K, path=(0, 1))


@pytest.mark.parametrize("K,l,m,dtype", [(3, 1, 500, "f32"), (4, 3, 500, "bf16"), (8, 2, 500, "f32")])
def test_what_is_typical_of_a_redone_chunk(K, l, m, dtype):
    """Two drifts 2^34 times the others, in sampled runs of their own (runs of 8 at the multiples of 31 here): one is left
    out of the sample's mean, the other stays.  A third, larger one lies outside the sample.  The redone sketch does not
    go by that mean: 2^29 units or more to a typical drift, or fp64."""
    import paper_2405_20988_amd as F
    d, g = 2_000, gen(K)
    w = (torch.randn((K, d), generator=g, device=DEV) * 1e-3).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    w[:, 22 * 31 + 3] = w[:, 48 * 31 + 2] = 1e-3 * 2.0 ** 34
    w[:, 23 * 31 + 9] = 1e-3 * 2.0 ** 40
    coef = S.hash_coefficients(K, l)
    mon = F.FdaMonitor(K, d, dtype, 3, l, m, 0.06, coef, device=DEV)
    assert mon.plan["partitions"] == 1
    zero = torch.zeros(d, device=DEV)
    ref = O.local_state(S.slab_to_numpy(w), dtype, zero.cpu().numpy(), zero.cpu().numpy(), coef, m)
    mon.local_state(w, zero, zero)
    sk = mon.state_numpy()[2]
    assert mon.last_state_path() == 2
    err = np.abs(sk.astype(np.float64) - ref["sk"])
    assert (err <= 2.0 ** -24 * np.abs(ref["sk"]) + ref["sk_cnt"][None] * 2.0 ** -30 * 0.8e-3 + 1e-45).all()
    mon.close()


@pytest.mark.parametrize("ratio", [2.0 ** 8, 2.0 ** 20])
@pytest.mark.parametrize("K,d,l,m,dtype", [(30, 900_001, 5, 250, "f32"), (8, 1_100_001, 7, 1000, "bf16"),
                                           (2, 4_300_003, 12, 300, "f32")])
def test_a_redone_long_chunk_keeps_29_bits_of_the_other_drifts(K, d, l, m, dtype, ratio):
    """Every workgroup meets a drift beyond its terms, of the last of its workers, and two `ratio` times the others in
    sampled runs of their own, of which one stays in the sample's mean.  A cell is off by its own fp32 rounding and by
    half a unit for each of its terms, with 2^29 units or more to a typical drift, or fp64; a sum by its fp32 rounding."""
    import paper_2405_20988_amd as F
    g = gen(K)
    coef = S.hash_coefficients(K, l)
    mon = F.FdaMonitor(K, d, dtype, 3, l, m, 0.06, coef, device=DEV)
    chunk, wpg = mon.plan["chunk"], mon.plan["workers_per_group"]
    assert chunk >= 8 * 2048 and K % wpg == 0
    u = torch.randn((K, d), generator=g, device=DEV) * 1e-3
    first = torch.arange(0, d - chunk, chunk, device=DEV)
    u[:, d - d % chunk:] = 0.0
    run = chunk // 64                                     # a sampled run of 8 at each multiple
    for k in range(wpg - 1, K, wpg):
        u[k, first + 10 * run] = u[k, first + 40 * run + 7] = 1e-3 * ratio
        u[k, first + 20 * run + 9] = 1e-3 * ratio * 64
    w = u.to(torch.float32 if dtype == "f32" else torch.bfloat16)
    zero, xi = torch.zeros(d, device=DEV), torch.randn(d, generator=g, device=DEV) / d ** 0.5
    ref = O.local_state(S.slab_to_numpy(w), dtype, zero.cpu().numpy(), xi.cpu().numpy(), coef, m)
    mon.local_state(w, zero, xi)
    n, p, sk = mon.state_numpy()
    assert mon.last_state_path() >= 1
    assert np.allclose(n, ref["n"], rtol=2.0 ** -23, atol=0)
    assert (np.abs(p - ref["p"]) <= 2.0 ** -23 * np.abs(ref["p"]) + 2.0 ** -40 * ref["p_abs"]).all()
    err = np.abs(sk.astype(np.float64) - ref["sk"])
    assert (err <= 2.0 ** -24 * np.abs(ref["sk"]) + ref["sk_cnt"][None] * 2.0 ** -30 * 0.8e-3 + 1e-45).all()
    mon.close()


@pytest.mark.parametrize("size,path", [(2.0 ** 14, 1), (1e12, 2)])       # 64-bit integers, fp64
@pytest.mark.parametrize("K,d,l,m,dtype", [
    (1, 50_001, 9, 250, "f32"), (1, 50_001, 1, 20_000, "bf16"),          # half of a worker's cells at a time
    (2, 50_001, 1, 15_000, "f32"),                                       # one worker at a time
    (5, 100_001, 5, 250, "f32"), (8, 50_001, 7, 1000, "bf16"), (4, 30_001, 5, 500, "f32"), (8, 30_001, 4, 300, "bf16"),  # all
    (3, 2_049, 1, 16, "f32"), (30, 60_001, 9, 250, "bf16"),
    (2, 1_500_003, 2, 64, "f32")])                                       # several tiles to a chunk
def test_redone_sketches_of_every_layout(K, d, l, m, dtype, size, path):
    """One workgroup in the middle and the one of the ragged end meet a drift that their terms cannot hold."""
    g = gen(K)
    w_t0 = torch.randn(d, generator=g, device=DEV).mul_(0.05).to(torch.bfloat16).float()
    w = (w_t0 + torch.randn((K, d), generator=g, device=DEV) * 1e-3).to(torch.float32 if dtype == "f32" else torch.bfloat16)
    w[K - 1, d - 1] = -1e-3 * size
    w[0, d // 2 + 37] = 1e-3 * size
    check_both(w, w_t0, torch.randn(d, generator=g, device=DEV) / d ** 0.5, dtype, l, m, K, path=(path,), mean_path=1)


def steps_of(K, d, dtype, g):
    """Drifts of either sign around 1.5 * 2^-10: one unit, 2^28, for every workgroup whose sample sees no others, whose
    terms end at 4."""
    u = (1.5 + 0.1 * torch.randn((K, d), generator=g, device=DEV).clamp_(-2, 2)) * 2.0 ** -10
    u *= torch.randint(0, 2, (K, d), generator=g, device=DEV) * 2 - 1
    return u.to(torch.float32 if dtype == "f32" else torch.bfloat16)


@pytest.mark.parametrize("K,d,l,m,dtype", [
    (1, 4_300_001, 3, 250, "f32"), (2, 4_300_003, 12, 300, "f32"),      # one worker slot; two row groups
    (2, 4_300_003, 2, 500, "bf16"), (8, 1_100_001, 7, 1000, "bf16"),    # placement groups of two rows, of four
    (11, 700_001, 3, 1500, "f32"), (30, 900_001, 9, 250, "bf16"),       # a spare slot; rows with a skew
    (31, 900_001, 5, 250, "f32"), (3, 1_500_001, 1, 20_000, "f32")])    # spare slots of six; plain rows of 16-bit fields
def test_outliers_of_a_long_chunk(K, d, l, m, dtype):
    """Long chunks, each with its own, outside the sampled runs: drifts just below and just beyond the terms, one, tens
    and hundreds beyond them, one of 2^39 units."""
    import paper_2405_20988_amd as F
    g = gen(K)
    plan = F.FdaMonitor(K, d, dtype, 3, l, m, 0.06, S.hash_coefficients(K, l), device=DEV).plan
    chunk, run = plan["chunk"], plan["chunk"] // 64       # a sampled run of 8 at each multiple
    assert chunk >= 8 * 2048
    w = steps_of(K, d, dtype, g)
    for i, x in enumerate((3.984375, 4.0, -3.984375, -4.0, 2040.0, -2040.0)):
        w[K - 1, chunk + run * i + 9] = x
        w[0, chunk + run * i + 11] = -x
    w[:, 2 * chunk - 1] = 37.0
    for p, n in ((3, 1), (5, 65), (8, 600)):
        i = torch.arange(n, device=DEV)
        w[K - 1, p * chunk + run * (i % 64) + 8 + torch.div(i, 64, rounding_mode="floor")] = 100.0
    w[K - 1, 10 * chunk + 9] = 2048.0
    xi = torch.randn(d, generator=g, device=DEV) / d ** 0.5
    check_both(w, torch.zeros(d, device=DEV), xi, dtype, l, m, K, path=(1,), mean_path=1)


def microseconds(call):
    """A pass among others: the best of five groups."""
    start, stop = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    best = float("inf")
    for _ in range(6):
        start.record()
        for _ in range(4):
            call()
        stop.record()
        stop.synchronize()
        best = min(best, start.elapsed_time(stop) * 250.0)
    return best


def test_a_redone_state_does_not_take_ten_times_the_pass():
    """One workgroup of 255 redoes its sketch: 5 times the pass without it (11 times with one worker and one element
    at a time)."""
    import paper_2405_20988_amd as F
    K, d = 30, 7_000_000
    mon = F.FdaMonitor(K, d, "f32", 3, 5, 250, 0.06, S.hash_coefficients(1, 5), device=DEV)
    w_t0 = torch.zeros(d, device=DEV)
    w = torch.randn((K, d), generator=gen(1), device=DEV) * 1e-3
    plain = microseconds(lambda: mon.local_state(w, w_t0, w_t0))
    assert mon.last_state_path() == 0
    w[1, d // 3 + 5] = 1e-3 * 2 ** 14
    redone = microseconds(lambda: mon.local_state(w, w_t0, w_t0))
    assert mon.last_state_path() == 1
    print("plain %.0f us, redone %.0f us" % (plain, redone))
    assert redone < 8.0 * plain
    mon.close()


def test_a_redone_average_state_does_not_take_four_times_the_pass():
    """Every workgroup redoes its sketch: twice the pass without it (5 times element by element)."""
    import paper_2405_20988_amd as F
    K, d = 30, 7_000_000
    mon = F.FdaMonitor(K, d, "f32", 3, 5, 250, 0.06, S.hash_coefficients(1, 5), device=DEV)
    w_t0 = torch.zeros(d, device=DEV)
    w = torch.randn((K, d), generator=gen(1), device=DEV) * 1e-3
    plain = microseconds(lambda: mon.mean_state(w, w_t0, w_t0))
    assert mon.last_mean_state_path() == 0
    w[:, 11::mon.plan["mean_chunk"] // 4] = 1e-3 * 2 ** 20
    redone = microseconds(lambda: mon.mean_state(w, w_t0, w_t0))
    assert mon.last_mean_state_path() == 1
    print("plain %.0f us, redone %.0f us" % (plain, redone))
    assert redone < 3.5 * plain
    mon.close()


@pytest.mark.parametrize("K,d,l,m,dtype", [(2, 5_001, 3, 40, "f32"), (5, 100_001, 5, 250, "f32"), (1, 1_100_003, 3, 250, "f32"),
                                           (8, 700_001, 7, 1000, "bf16"), (17, 400_003, 2, 33, "bf16")])
def test_partials_of_every_kind_merge(K, d, l, m, dtype):
    """Workgroups whose sketch stands, one that did it again in integers and one that did it in fp64: from 3 partitions
    (fewer than a batch of the merge) to hundreds, remainders among them."""
    g = gen(d)
    w_t0 = (torch.randn(d, generator=g, device=DEV) * 0.05).to(torch.bfloat16).float()
    w = torch.randn((K, d), generator=g, device=DEV) * 1e-3 + w_t0
    w[K - 1, d // 6 + 3] = 1e-3 * 2 ** 14
    w[0, d // 2 + 1] = 1e9
    w = w.to(torch.float32 if dtype == "f32" else torch.bfloat16)
    xi = torch.randn(d, generator=g, device=DEV)
    check_both(w, w_t0, xi / xi.norm(), dtype, l, m, seed=d, path=(2,), mean_path=1)
