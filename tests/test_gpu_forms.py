"""The forms a step is launched in, at the sizes where they can go wrong.

Several steps of one launch against the same steps launched one by one (the
arithmetic is the same, states are rounded to storage between steps either
way: bit for bit); tiles, waves and lists at their edges against the general
forms or the oracle.  Tolerances: one FP64 step agrees with the oracle to the
rounding of its sums (1e-13 of the largest population, the bound of the other
parity tests), a few steps to 1e-12; two forms that only rescale a moved node
differently agree to 1e-13.
"""
import numpy as np
import pytest

from paper_0704_0043_amd import workloads as wl
from tests.gpu_util import Pair, assert_ds_close, assert_masks_equal, lbm, orc, require_gpu, say, stats_equal

pytestmark = pytest.mark.gpu

D1Q3, D2Q9 = 1, 2
PERIODIC, CAVITY, TUBE, DIFFUSIVE = 0, 1, 2, 3
SMOOTH, RATIONAL, BUDGET = 8, 16, 32


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def rough(q, nx, ny, seed, amp=0.03):
    return wl.random_populations(q, nx, ny, seed=seed, amp=amp, spike_frac=0.05, spike_amp=0.3)


def close(a, b, rtol):
    err = np.abs(a - b).max() / np.abs(b).max()
    say(f"  max rel err {err:.2e} (bound {rtol:.0e})")
    assert err <= rtol


def run(doms, f0s, steps, storage=0, **kw):
    """Populations and sums of every domain, and the trace of those with a probe."""
    L = lbm()
    for d, f0 in zip(doms, f0s):
        d.f_init = f0
    with L.lbm_create(doms, L.Run(storage=storage, **kw)) as ctx:
        for n in steps:
            L.lbm_step(ctx, n)
        return [(L.lbm_get_populations(ctx, k), L.lbm_entropy_stats(ctx, k, allow_unstable=True),
                 L.lbm_probe_trace(ctx, k, sum(steps)) if d.probe else None) for k, d in enumerate(doms)]


def skip_small_cavity(bc, nx, ny):
    if bc != PERIODIC and min(nx, ny) < 4:
        pytest.skip("a cavity needs nx, ny >= 4")


def assert_same_runs(a, b):
    for (fa, sa, pa), (fb, sb, pb) in zip(a, b):
        assert np.array_equal(fa, fb, equal_nan=True)
        assert stats_equal(sa, sb)
        assert pa is None or np.array_equal(pa, pb)


# 190 sites a workgroup; 33 steps a launch, 64 a graph
@pytest.mark.parametrize("nx", [2, 63, 189, 190, 191, 381])
@pytest.mark.parametrize("bc", [PERIODIC, TUBE])
@pytest.mark.parametrize("limiter,storage", [(1, 0), (3, 0), (3, 1)])
def test_tube_steps_of_one_launch(nx, bc, limiter, storage):
    L = lbm()
    steps = [1, 2, 33, 34, 67]
    f0 = rough(3, nx, 1, seed=nx)
    d = L.Domain(lattice=D1Q3, nx=nx, ny=1, beta=0.98, qe=0, ds_form=0, limiter=limiter, bc=bc, delta_trim=1e-3,
                 delta_median=1e-5, probe=(nx // 2, 0))
    say(f"[tube] nx {nx} bc {bc} limiter {limiter} storage {storage}")
    many = run([d], [f0], steps, storage)
    assert_same_runs(many, run([d], [f0], steps, storage, flags=L.LBM_RUN_NO_GRAPH))
    if storage == 0:
        d.probe = None
        pr = Pair(d, f0, steps=4)
        close(pr.f, pr.fo, 1e-12)


# tiles of 10 x 10 and the like with one, two or three steps a launch; 200 x 200
# and the batch take single steps in FP64
@pytest.mark.parametrize("sizes", [[(3, 3)], [(4, 9)], [(11, 10)], [(33, 21)], [(100, 100)], [(101, 99)],
                                   [(200, 200)], [(70, 70), (13, 100), (64, 33)]])
@pytest.mark.parametrize("bc", [PERIODIC, CAVITY, DIFFUSIVE])
@pytest.mark.parametrize("storage,ds,qe", [(0, 0, 1), (1, 1, 0), (2, 1, 0)])
def test_tile_steps_of_one_launch(sizes, bc, storage, ds, qe):
    L = lbm()
    skip_small_cavity(bc, *min(sizes, key=min))
    steps = [1, 2, 5, 64, 39]
    say(f"[tiles] {sizes} bc {bc} storage {storage} ds {ds}")
    doms, f0s = [], []
    for k, (nx, ny) in enumerate(sizes):
        f0s.append(rough(9, nx, ny, seed=5 + k))
        doms.append(L.Domain(lattice=D2Q9, nx=nx, ny=ny, beta=0.9, qe=qe, ds_form=ds, limiter=3, bc=bc,
                             lid_ux=0.0 if bc == PERIODIC else 0.05, delta_trim=1e-3, delta_median=1e-5,
                             probe=(nx // 2, ny // 2)))
    many = run(doms, f0s, steps, storage)
    assert_same_runs(many, run(doms, f0s, steps, storage, flags=L.LBM_RUN_NO_GRAPH))
    if storage == 0:
        # one step against the walking form of the same step
        one = run(doms, f0s, [1], storage)
        walk = run(doms, f0s, [1], storage, tile_x=248, flags=L.LBM_RUN_NO_TUNE)
        for (fa, sa, _), (fb, sb, _) in zip(one, walk):
            close(fa, fb, 1e-13)
            for key in ("n_trimmed", "n_filtered", "n_fluid", "n_nonpositive"):
                assert sa[key] == sb[key], key


# the largest tiled domain (400000 nodes), and the smallest with two kernels
@pytest.mark.parametrize("nx", [640, 641])
def test_both_sides_of_the_tiled_size(nx):
    L = lbm()
    f0 = rough(9, nx, 625, seed=2)
    d = L.Domain(lattice=D2Q9, nx=nx, ny=625, beta=0.97, qe=0, ds_form=1, limiter=3, delta_trim=1e-4,
                 delta_median=1e-5)
    say(f"[tiled size] {nx}x625")
    a = run([d], [f0], [1], flags=L.LBM_RUN_NO_TUNE)[0]
    b = run([d], [f0], [1], tile_x=248, flags=L.LBM_RUN_NO_TUNE)[0]
    close(a[0], b[0], 1e-13)
    for key in ("n_trimmed", "n_filtered", "n_fluid"):
        assert a[1][key] == b[1][key], key


def test_tiled_batch_with_a_domain_without_median():
    """A batch takes the tiles when one of its domains has the median filter;
    the other alone takes the collision kernel."""
    L = lbm()
    f0s = [rough(9, 40, 30, seed=1), rough(9, 65, 31, seed=2)]
    doms = [L.Domain(lattice=D2Q9, nx=40, ny=30, beta=0.95, qe=0, ds_form=1, limiter=3, delta_trim=1e-4,
                     delta_median=1e-5),
            L.Domain(lattice=D2Q9, nx=65, ny=31, beta=0.95, qe=0, ds_form=1, limiter=1, delta_trim=1e-4)]
    both = run(doms, f0s, [7])
    for k in (0, 1):
        close(run([doms[k]], [f0s[k]], [7])[0][0], both[k][0], 1e-12)


# 256 consecutive nodes a workgroup, whatever the rows: rows of a wave, one less,
# one more, shorter than a wave, a last workgroup of one node
@pytest.mark.parametrize("nx,ny", [(1, 5), (2, 2), (3, 43), (63, 5), (64, 4), (65, 4), (128, 2), (257, 1), (255, 3)])
@pytest.mark.parametrize("bc", [PERIODIC, CAVITY])
def test_collision_over_consecutive_nodes(nx, ny, bc):
    skip_small_cavity(bc, nx, ny)
    L = lbm()
    d = L.Domain(lattice=D2Q9, nx=nx, ny=ny, beta=0.97, qe=0, ds_form=1, limiter=1, bc=bc, delta_trim=1e-4,
                 lid_ux=0.0 if bc == PERIODIC else 0.05)
    pr = Pair(d, rough(9, nx, ny, seed=nx + ny), steps=3)
    close(pr.f, pr.fo, 1e-12)
    f0s = [rough(9, nx, ny, seed=nx + ny), rough(9, ny + 2, nx + 2, seed=1)]
    e = L.Domain(lattice=D2Q9, nx=ny + 2, ny=nx + 2, beta=0.97, qe=0, ds_form=1, limiter=1, bc=bc, delta_trim=1e-4,
                 lid_ux=d.lid_ux)
    batch = run([d, e], f0s, [3])       # the next domain begins at a workgroup of its own
    assert np.array_equal(batch[0][0], run([d], f0s[:1], [3])[0][0])
    assert np.array_equal(batch[1][0], run([e], f0s[1:], [3])[0][0])


# the second pass's lists with nothing to move and with every node moved, at the
# edges of its waves (62 columns), workgroups (248) and short tiles
@pytest.mark.parametrize("nx,ny", [(3, 3), (62, 4), (63, 5), (64, 17), (249, 6), (300, 33)])
@pytest.mark.parametrize("bc", [PERIODIC, CAVITY])
@pytest.mark.parametrize("delta", [1e-12, 1e3])
def test_second_pass_lists(nx, ny, bc, delta):
    skip_small_cavity(bc, nx, ny)
    L = lbm()
    f0 = rough(9, nx, ny, seed=nx * ny)
    d = L.Domain(lattice=D2Q9, nx=nx, ny=ny, beta=0.97, qe=0, ds_form=1, limiter=2, bc=bc, delta_median=delta,
                 lid_ux=0.0 if bc == PERIODIC else 0.05)
    say(f"[lists] {nx}x{ny} bc {bc} delta {delta}")
    two = run([d], [f0], [1], flags=L.LBM_RUN_ADAPTIVE | L.LBM_RUN_NO_TUNE)[0]       # begins with two kernels
    walk = run([d], [f0], [1], tile_x=248, flags=L.LBM_RUN_NO_TUNE)[0]
    close(two[0], walk[0], 1e-13)
    assert two[1]["n_filtered"] == walk[1]["n_filtered"]
    if delta > 1.0:
        assert two[1]["n_filtered"] == 0


# the pass over every node of a smooth factor: rows across waves and workgroups
@pytest.mark.parametrize("nx,ny", [(3, 5), (63, 5), (64, 4), (65, 9), (130, 3), (257, 4)])
@pytest.mark.parametrize("bc", [PERIODIC, CAVITY])
@pytest.mark.parametrize("limiter,kw", [(SMOOTH, dict(ens_k=0.5, delta_ens=0.01)),
                                        (RATIONAL, dict(ens_c=2.0, ens_k=1.0))])
def test_dense_form_pass(nx, ny, bc, limiter, kw):
    skip_small_cavity(bc, nx, ny)
    L = lbm()
    d = L.Domain(lattice=D2Q9, nx=nx, ny=ny, beta=0.95, qe=0, ds_form=1, limiter=3 | limiter, bc=bc, delta_trim=1e-4,
                 delta_median=1e-5, lid_ux=0.0 if bc == PERIODIC else 0.05, **kw)
    pr = Pair(d, rough(9, nx, ny, seed=nx + 7 * ny), steps=1)
    assert_masks_equal(pr, ens_noise=True)
    close(pr.f, pr.fo, 1e-12)
    # beside a domain whose second pass is the list one
    e = L.Domain(lattice=D2Q9, nx=70, ny=20, beta=0.95, qe=0, ds_form=1, limiter=3 | BUDGET, ens_c=0.3, bc=bc,
                 delta_trim=1e-4, delta_median=1e-5, lid_ux=d.lid_ux)
    f0s = [rough(9, nx, ny, seed=nx + 7 * ny), rough(9, 70, 20, seed=3)]
    mixed = run([d, e], f0s, [1])
    for k, one in enumerate((d, e)):
        close(mixed[k][0], run([one], [f0s[k]], [1])[0][0], 1e-13)


# the arguments of the exact Delta S on both sides of its series' ends (FP64
# 1/85, 0.1, 0.5; FP32 1/64, 1/8, 0.5)
@pytest.mark.parametrize("amp", [1e-3, 0.011, 0.0125, 0.015, 0.017, 0.09, 0.11, 0.13, 0.45, 0.55, 0.95])
def test_exact_delta_s_over_its_ranges(amp):
    L = lbm()
    f0 = wl.random_populations(9, 130, 9, seed=7, amp=amp, spike_frac=0.0)
    d = L.Domain(lattice=D2Q9, nx=130, ny=9, beta=0.9, qe=1, ds_form=0, limiter=0)
    pr = Pair(d, f0, steps=1)
    assert_ds_close(pr, 1e-11)
    close(pr.f, pr.fo, 1e-13)
    # FP32: a deviation x = (f - f*)/f* of size amp/2 carries a rounding of some
    # 12 units of 6e-8 from the sums of f*, Delta S twice its relative error
    p32 = Pair(d, f0, steps=1, storage=1)
    fin = np.isfinite(p32.dso) & np.isfinite(p32.ds) & (p32.dso > 0.05 * np.median(p32.dso))
    err = np.abs(p32.ds[fin] - p32.dso[fin]) / p32.dso[fin]
    tol = 2 * 12 * 6e-8 / (amp / 2) * 5 + 1e-5      # 5: the smallest deviation let through is 0.05 ** 0.5 of the median's
    say(f"  amp {amp} FP32 Delta S max rel err {err.max():.2e} (bound {tol:.1e})")
    assert err.max() <= tol


# the entropic root from its series' start, from quasi-Newton and from Newton
@pytest.mark.parametrize("amp", [1e-6, 1e-3, 0.01, 0.08, 0.3, 0.7])
@pytest.mark.parametrize("lattice", [D1Q3, D2Q9])
def test_entropic_root_over_its_ranges(amp, lattice):
    L = lbm()
    nx, ny = (700, 1) if lattice == D1Q3 else (70, 9)
    f0 = wl.random_populations(3 if lattice == D1Q3 else 9, nx, ny, seed=11, amp=amp, spike_frac=0.0)
    d = L.Domain(lattice=lattice, nx=nx, ny=ny, beta=0.97, qe=1, ds_form=0, limiter=0, collision=1)
    pr = Pair(d, f0, steps=1)
    assert pr.stats["n_positivity"] == pr.so["n_positivity"]
    close(pr.f, pr.fo, 1e-12)
    p32 = Pair(d, f0, steps=1, storage=1)
    # a root at the rounding level of FP32 sums moves a population by a few units of its deviation
    close(p32.f, p32.fo, 2e-6 + 4e-6 * amp)


# one group of 16384 values, one more, and more groups than histogram workgroups
@pytest.mark.parametrize("nx,ny", [(64, 3), (128, 128), (129, 128), (2100, 2050)])
def test_budget_threshold_over_groups(nx, ny):
    L = lbm()
    f0 = rough(9, nx, ny, seed=9)
    c = 2 * 0.9 - 1
    d = L.Domain(lattice=D2Q9, nx=nx, ny=ny, beta=0.9, qe=0, ds_form=1, limiter=BUDGET, ens_c=0.1, f_init=f0)
    say(f"[budget] {nx}x{ny}")
    with L.lbm_create([d], L.Run(storage=0, flags=L.LBM_RUN_RECORD)) as ctx:
        L.lbm_step(ctx, 1)
        ds = L.lbm_limiter_mask(ctx)[1]
        st = L.lbm_entropy_stats(ctx)
    want = 0.1 * (1 - c * c) * ds.sum()
    t = st["ens_threshold"]
    assert np.maximum(ds - t, 0).sum() == pytest.approx(want, rel=1e-9)


def test_probe_ring_and_transfers():
    """A ring that wraps, fewer samples than it holds, and states on both sides
    of the pinned transfer (9 x 120 x 120 doubles are 1.04 MB, 1 MiB its limit)."""
    L = lbm()
    for n in (100, 120, 160):
        f0 = rough(9, n, n, seed=n)
        d = L.Domain(lattice=D2Q9, nx=n, ny=n, beta=0.9, qe=0, ds_form=1, limiter=1, delta_trim=1e-3, f_init=f0,
                     probe=(5, 7))
        with L.lbm_create([d], L.Run(storage=0, probe_capacity=8)) as ctx:
            want = []
            for k in range(13):
                rho, u = L.lbm_moments(ctx)
                want.append(u[:, 7, 5])
                L.lbm_step(ctx, 1)
                for ask in (1, 3, 8, 20):
                    got = L.lbm_probe_trace(ctx, 0, ask)
                    have = min(k + 1, 8, ask)
                    assert got.shape[0] == have
                    # the samples are FP32
                    assert np.allclose(got, np.array(want)[k + 1 - have:], rtol=1e-6, atol=1e-9)
            L.lbm_set_populations(ctx, f0)
            got = L.lbm_get_populations(ctx)
            rho, u = L.lbm_moments(ctx)
        close(got, f0, 4e-16)       # stored less the rest state, one rounding each way
        close(rho, f0.sum(0), 1e-14)


# several steps of one launch leave the states between them nowhere, but the
# buffer that does not hold the result holds the state before the last step
@pytest.mark.parametrize("lattice,nx,ny", [(D1Q3, 300, 1), (D2Q9, 60, 50)])
@pytest.mark.parametrize("n", [1, 2, 7, 40])
def test_static_buffers_after_several_steps(lattice, nx, ny, n):
    import torch
    L = lbm()
    d = L.Domain(lattice=lattice, nx=nx, ny=ny, beta=0.95, qe=0, ds_form=1, limiter=3, delta_trim=1e-3,
                 delta_median=1e-5)
    f = torch.from_numpy(rough(3 if lattice == D1Q3 else 9, nx, ny, seed=4)).cuda()

    def after(k):
        bufs = [f.clone(), torch.zeros_like(f)]
        L.lbm_step_static(d, 0, bufs[0].data_ptr(), bufs[1].data_ptr(), k, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        return bufs[k % 2], bufs[1 - k % 2]

    say(f"[static] lattice {lattice} {nx}x{ny} n {n}")
    assert torch.equal(after(n)[1], after(n - 1)[0])


W9 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)


# a node the positivity rule acts on has Delta S' = +inf; where every node has,
# E(Delta S') is 0 and the median infinite, so the rule's factor is the only one
@pytest.mark.parametrize("limiter,kw", [(SMOOTH, dict(ens_k=0.5, delta_ens=0.01)),
                                        (RATIONAL, dict(ens_c=2.0, ens_k=1.0))])
@pytest.mark.parametrize("median", [0, 2])
@pytest.mark.parametrize("storage", [0, 1])
def test_dense_form_pass_keeps_the_positivity_rule(limiter, kw, median, storage):
    L = lbm()
    f0 = np.empty((9, 8, 8))
    f0[:] = W9[:, None, None]
    f0[[1, 3]] *= 3.5
    d = L.Domain(lattice=D2Q9, nx=8, ny=8, beta=0.99, qe=0, ds_form=0, limiter=64 | limiter | median,
                 delta_median=1e-5, **kw)
    pr = Pair(d, f0, steps=1, storage=storage)
    assert_masks_equal(pr)
    assert pr.stats["n_positivity"] == pr.so["n_positivity"] == 64
    assert pr.stats["n_ensemble"] == pr.so["n_ensemble"] == 0
    # FP32: the rounding of the populations' excess over w_i, a few units of 6e-8 each
    close(pr.f, pr.fo, 1e-13 if storage == 0 else 2e-6)
    # one such node in an FP32 field at rest, whose other Delta S' are exactly 0:
    # the positivity rule alone
    if storage == 1 and not median:
        f1 = np.empty((9, 8, 8))
        f1[:] = W9[:, None, None]
        f1[[1, 3], 3, 5] *= 3.5
        lone = Pair(d, f1, steps=1, storage=1)
        d.limiter = 64
        alone = Pair(d, f1, steps=1, storage=1)
        assert lone.stats["n_positivity"] == 1 and lone.stats["mean_dS"] == 0.0
        assert np.array_equal(lone.mask, alone.mask)
        close(lone.f, alone.fo, 2e-6)


# beside a domain beyond the last-level cache the second pass rescales what is
# stored instead of forming the moved nodes anew: the same decisions, states to
# rounding (FP32: a few units of 6e-8 of a node's excess over w_i)
@pytest.mark.parametrize("nx,ny", [(15, 9), (63, 5), (65, 17), (257, 33)])
@pytest.mark.parametrize("storage,ds", [(0, 0), (1, 1)])
@pytest.mark.parametrize("limiter,kw", [(3, dict(delta_median=0.0)), (7, dict(ens_c=1.0, delta_median=1e-5)),
                                        (3, dict(delta_median=1e-5, top_k=40, trim_mode=1)),
                                        (66, dict(delta_median=1e-5))])
def test_moved_nodes_from_the_stored_state(nx, ny, storage, ds, limiter, kw):
    L = lbm()
    if limiter & 64 and ds:
        pytest.skip("the positivity rule needs the exact Delta S here")
    f0 = rough(9, nx, ny, seed=nx + ny)
    d = L.Domain(lattice=D2Q9, nx=nx, ny=ny, beta=0.97, qe=0, ds_form=ds, limiter=limiter, delta_trim=1e-5, **kw)
    far = L.Domain(lattice=D2Q9, nx=2600, ny=(1450, 4400)[storage], beta=0.97, qe=0, ds_form=ds, limiter=1)
    flags = L.LBM_RUN_NO_TUNE | (0 if limiter & 4 or d.top_k else L.LBM_RUN_ADAPTIVE)    # begins with two kernels
    say(f"[stored] {nx}x{ny} limiter {limiter} storage {storage}")
    anew = run([d], [f0], [1], storage, flags=flags)[0]
    stored = run([d, far], [f0, None], [1], storage, flags=flags)[0]
    close(stored[0], anew[0], 1e-13 if storage == 0 else 1e-6)
    for key in ("n_trimmed", "n_filtered", "n_ensemble", "n_positivity", "sum_dS_post", "max_dS"):
        assert anew[1][key] == stored[1][key], key
    assert anew[1]["n_filtered"] + anew[1]["n_ensemble"] + anew[1]["n_trimmed"] > nx * ny // 8
    # differences of the entropies of a node before and after
    assert stored[1]["limiter_production"] == pytest.approx(anew[1]["limiter_production"],
                                                            rel=1e-10 if storage == 0 else 1e-4)


def test_short_tiles_do_not_compute_what_lds_held():
    """Past a short tile there is LDS that nobody wrote; a halo node that took it
    in would hold its workgroup up in logarithms and roots.  64 steps of 40 x 40
    nodes with the exact homothety (3.8 us a step) take no longer
    than four times those with the quadratic form (2.6 us)."""
    import time
    L = lbm()

    def best(**kw):
        d = L.Domain(lattice=D2Q9, nx=40, ny=40, beta=0.97, qe=0, limiter=3, delta_trim=1e-4, delta_median=1e-5,
                     f_init=wl.random_populations(9, 40, 40, seed=8, amp=0.001, spike_frac=0.0), **kw)
        with L.lbm_create([d], L.Run(storage=0)) as ctx:
            L.lbm_step(ctx, 64)
            took = []
            for _ in range(30):
                L.lbm_synchronize(ctx)
                t = time.perf_counter()
                L.lbm_step(ctx, 64)
                L.lbm_synchronize(ctx)
                took.append(time.perf_counter() - t)
        return min(took)

    quadratic, exact = best(ds_form=1), best(ds_form=0, homothety=1)
    say(f"[short tiles] 64 steps: quadratic {quadratic * 1e6:.0f} us, exact homothety {exact * 1e6:.0f} us")
    assert exact < 4 * quadratic


# a workgroup's sites (188), one less and one more, two workgroups and one site
@pytest.mark.parametrize("nx", [187, 188, 377])
@pytest.mark.parametrize("limiter,storage", [(1, 0), (3, 1)])
def test_tube_workgroups(nx, limiter, storage):
    L = lbm()
    f0 = rough(3, nx, 1, seed=nx)
    d = L.Domain(lattice=D1Q3, nx=nx, ny=1, beta=0.98, qe=0, ds_form=0, limiter=limiter, bc=TUBE, delta_trim=1e-3,
                 delta_median=1e-5, probe=(nx // 2, 0))
    say(f"[tube workgroups] nx {nx} limiter {limiter} storage {storage}")
    steps = [1, 2, 33, 34, 67]
    assert_same_runs(run([d], [f0], steps, storage), run([d], [f0], steps, storage, flags=L.LBM_RUN_NO_GRAPH))
    if storage == 0:
        d.probe = None
        pr = Pair(d, f0, steps=4)
        close(pr.f, pr.fo, 1e-12)


@pytest.mark.parametrize("storage", [1, 2])
def test_limiter_production_of_tiles_in_fp64(storage):
    """The nodes' terms are FP32, their sum is FP64 in every form of the step."""
    L = lbm()
    f0 = rough(9, 100, 90, seed=3)
    d = L.Domain(lattice=D2Q9, nx=100, ny=90, beta=0.97, qe=0, ds_form=1, limiter=3, delta_trim=1e-4,
                 delta_median=1e-5)
    tiles = run([d], [f0], [1], storage)[0][1]
    walk = run([d], [f0], [1], storage, tile_x=248, flags=L.LBM_RUN_NO_TUNE)[0][1]
    assert tiles["n_filtered"] == walk["n_filtered"] > 0
    assert tiles["limiter_production"] == pytest.approx(walk["limiter_production"], rel=1e-13)


def test_budget_threshold_of_few_values_above_many():
    """A node of 300 v and two of 100 v above 512 x 512 of v, all but the first in
    the eight binary exponents that one thread of the selection adds up: the
    threshold lies between them, at (the sum of the three - budget) / 3, and owes
    nothing to the digits of the many."""
    import math
    L = lbm()
    n, beta = 512, 0.99
    c = 2 * beta - 1
    v = 1.3 * 2.0 ** -23
    e = np.full((n, n), math.sqrt(v / 18) / c)
    e[100, 300] *= 10
    e[301, 17] *= 10.1
    e[400, 400] *= 17.3
    f0 = np.empty((9, n, n))
    f0[:] = W9[:, None, None]
    f0[[1, 3]] += e
    f0[[2, 4]] -= e
    d = L.Domain(lattice=D2Q9, nx=n, ny=n, beta=beta, qe=0, ds_form=1, limiter=BUDGET,
                 ens_c=350 / (n * n * (1 - c * c)), f_init=f0)
    with L.lbm_create([d], L.Run(storage=0, flags=L.LBM_RUN_RECORD)) as ctx:
        L.lbm_step(ctx, 1)
        ds = L.lbm_limiter_mask(ctx)[1]
        t = L.lbm_entropy_stats(ctx)["ens_threshold"]
    budget = d.ens_c * (1 - c * c) * math.fsum(ds.ravel())
    big = ds[ds > 50 * v]
    want = (math.fsum(big) - budget) / 3
    assert big.size == 3 and 10 * v < want < big.min()
    say(f"[budget] threshold {t!r}, exactly {want!r}: rel {abs(t - want) / want:.1e}")
    # the sum over all nodes is 20 roundings deep; 7/3 of its relative error is the threshold's
    assert abs(t - want) <= 2.4 * 20 * 1.2e-16 * want


# the lists full: a threshold of 0 moves every fluid node, at the edges of the
# second pass's waves (64 columns), tiles (256) and list flushes (8 rows)
@pytest.mark.parametrize("nx", [63, 64, 65, 255, 256, 257])
@pytest.mark.parametrize("ny", [7, 8, 9])
@pytest.mark.parametrize("bc", [PERIODIC, CAVITY])
def test_second_pass_lists_with_every_node(nx, ny, bc):
    L = lbm()
    d = L.Domain(lattice=D2Q9, nx=nx, ny=ny, beta=0.97, qe=0, ds_form=1, limiter=4, ens_c=0.0, delta_ens=1e-9, bc=bc,
                 lid_ux=0.0 if bc == PERIODIC else 0.05)
    pr = Pair(d, rough(9, nx, ny, seed=nx + ny), steps=1)
    assert pr.stats["n_ensemble"] == pr.so["n_ensemble"] == pr.stats["n_fluid"]
    assert_masks_equal(pr)
    close(pr.f, pr.fo, 1e-13)
    assert pr.stats["limiter_production"] == pytest.approx(pr.so["limiter_production"], rel=1e-11)


# a node so fast that a population of its polynomial f* is negative: the rule's
# factor is negative too, and the smallest, whatever the mean says
@pytest.mark.parametrize("limiter,kw", [(SMOOTH, dict(ens_k=0.5, delta_ens=0.01)),
                                        (RATIONAL, dict(ens_c=2.0, ens_k=1.0))])
def test_dense_form_pass_with_a_negative_equilibrium(limiter, kw):
    L = lbm()
    f0 = rough(9, 70, 9, seed=4, amp=0.01)
    f0[:, 4, 20] = 0.01
    f0[1, 4, 20] = 2.0
    assert orc().equilibrium(2, 0, 2.08, 2.0 / 2.08, 0.0).min() < 0
    d = L.Domain(lattice=D2Q9, nx=70, ny=9, beta=0.97, qe=0, ds_form=0, limiter=64 | limiter, **kw)
    pr = Pair(d, f0, steps=1)
    assert pr.stats["n_positivity"] == pr.so["n_positivity"] > 0
    assert_masks_equal(pr, ens_noise=True)
    close(pr.f, pr.fo, 1e-13)
