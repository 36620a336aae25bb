"""GPU parity of the batched GNEB (geodesic init, iterations, climbing image,
ragged batching, hipGraph replay) against the FP64 oracle, plus the
Stoner-Wohlfarth closed-form barrier.

Tolerances: geodesic path 1e-13 per component; GNEB state after each of up
to 20 iterations <= 1e-9 per component (FP64 on both sides; observed drift is
rounding level); energies/distances 1e-10 relative; barrier 1e-8 meV.
"""
import math

import numpy as np
import pytest

import oracle
from tests.helpers import gpu_hamiltonian, oracle_model, require_gpu, to_dev
from workloads import Workload, random_sphere, uniform_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def frustrated(L, periodic=(0, 0, 0), K=0.05, B=(0.0, 0.0, 0.3)):
    return Workload(name="t", L=L, periodic=periodic, J_shell=(1.0, 0.188, -0.274, -0.161), K=K, B=B,
                    field_prec="fp64")


def endpoints(w, seed):
    A = random_sphere(w.N, seed)
    Bv = random_sphere(w.N, seed + 100)
    A[:, 0] = [0, 0, 1.0]
    Bv[:, 0] = [0, 0, -1.0]          # antiparallel pair
    if w.N > 1:
        Bv[:, 1] = A[:, 1]           # parallel pair
    return A, Bv


def gpu_path(w, A, B, n_img):
    Y = np.zeros((n_img, 3, w.N))
    Y[0], Y[-1] = A, B
    return to_dev(Y)


def test_geodesic_init_matches_oracle():
    import torch
    from paper_2605_26016_amd import spx
    w = frustrated((5, 4, 3))
    A, B = endpoints(w, 1)
    Yd = gpu_path(w, A, B, 9)
    g = spx.gneb_create([gpu_hamiltonian(w)], [Yd])
    spx.gneb_init_path(g)
    torch.cuda.synchronize()
    ref = oracle.geodesic_path(A, B, 9)
    assert np.max(np.abs(Yd.cpu().numpy() - ref)) < 1e-13


@pytest.mark.parametrize("ci_mode,engine", [(0, 0), (1, 0), (2, 0), (3, 0), (1, 1)],
                         ids=["mode0", "mode1", "mode2", "mode3", "mode1_gather"])
def test_gneb_iterations_match_oracle(ci_mode, engine):
    # engine 0: the batched z-march field pass; 1: pass A gathers neighbours
    import torch
    from paper_2605_26016_amd import spx
    w = frustrated((5, 4, 3))
    A, B = endpoints(w, 2)
    n_img = 7
    params = dict(spring_k=0.5, vp_dt=0.05, vp_mass=1.0, ci_mode=ci_mode, ci_on_below=10.0)
    Y0 = oracle.geodesic_path(A, B, n_img)
    Yd = to_dev(Y0)
    g = spx.gneb_create([gpu_hamiltonian(w, stencil_engine=engine)], [Yd], **params)
    st = oracle.GnebState(Y0, k_spring=0.5, dt=0.05, mass=1.0, ci_mode=ci_mode, ci_on_below=10.0)
    m = oracle_model(w)
    for it in range(12):
        E, dist, fmax, ci = oracle.gneb_iterate(m, st)
        spx.gneb_step(g, 1)
        s = spx.gneb_get_stats(g)
        got = Yd.cpu().numpy()
        assert np.max(np.abs(got - st.Y)) <= 1e-9, (it, np.max(np.abs(got - st.Y)))
        np.testing.assert_allclose(s["E"], E, rtol=1e-10, atol=1e-12)
        np.testing.assert_allclose(s["dist"], dist, rtol=1e-10, atol=1e-12)
        assert abs(s["max_force"] - fmax) <= 1e-9 * max(1.0, fmax)
        assert s["ci_index"] == ci and s["ci_on"] == st.ci_on.value and s["iterations"] == it + 1


def test_gneb_graph_replay_equals_single_steps():
    import torch
    from paper_2605_26016_amd import spx
    w = frustrated((4, 4, 4), periodic=(1, 1, 1))
    A, B = endpoints(w, 3)
    Y0 = oracle.geodesic_path(A, B, 6)
    Ya, Yb = to_dev(Y0), to_dev(Y0)
    ga = spx.gneb_create([gpu_hamiltonian(w)], [Ya], ci_mode=1, ci_on_below=5.0)
    gb = spx.gneb_create([gpu_hamiltonian(w)], [Yb], ci_mode=1, ci_on_below=5.0)
    spx.gneb_step(ga, 9)                  # one captured graph, replayed
    for _ in range(9):
        spx.gneb_step(gb, 1)              # direct launches
    torch.cuda.synchronize()
    assert torch.equal(Ya, Yb)
    assert spx.gneb_get_stats(ga)["iterations"] == 9


def test_gneb_graph_branches_equal_single_steps():
    # several instances: the captured iteration runs their passes on
    # parallel branches; replaying it must give the direct launches' images
    # bit for bit
    import torch
    from paper_2605_26016_amd import spx
    cases = [(frustrated((4, 4, 4)), 5, 21), (frustrated((5, 4, 3), periodic=(1, 0, 1)), 7, 22),
             (frustrated((6, 6, 2), K=0.2), 4, 23), (frustrated((8, 8, 8)), 6, 24)]
    ga_bufs, gb_bufs, hams_a, hams_b = [], [], [], []
    for w, n_img, seed in cases:
        A, B = endpoints(w, seed)
        Y0 = oracle.geodesic_path(A, B, n_img)
        ga_bufs.append(to_dev(Y0))
        gb_bufs.append(to_dev(Y0))
        hams_a.append(gpu_hamiltonian(w))
        hams_b.append(gpu_hamiltonian(w))
    ga = spx.gneb_create(hams_a, ga_bufs, ci_mode=1, ci_on_below=3.0)
    gb = spx.gneb_create(hams_b, gb_bufs, ci_mode=1, ci_on_below=3.0)
    spx.gneb_step(ga, 12)                 # captured once, replayed
    for _ in range(12):
        spx.gneb_step(gb, 1)              # direct launches, one instance after another
    torch.cuda.synchronize()
    for k in range(len(cases)):
        assert torch.equal(ga_bufs[k], gb_bufs[k]), k
        assert spx.gneb_get_stats(ga, k)["iterations"] == 12


def test_gneb_batched_ragged_instances_match_oracle():
    import torch
    from paper_2605_26016_amd import spx
    cases = [(frustrated((4, 4, 4)), 5, 11), (frustrated((5, 4, 3), periodic=(1, 0, 1)), 7, 12),
             (frustrated((6, 6, 2), K=0.2), 4, 13)]
    hams, bufs, refs = [], [], []
    for w, n_img, seed in cases:
        A, B = endpoints(w, seed)
        Y0 = oracle.geodesic_path(A, B, n_img)
        hams.append(gpu_hamiltonian(w))
        bufs.append(to_dev(Y0))
        refs.append((oracle_model(w), oracle.GnebState(Y0, k_spring=1.0, dt=0.05, mass=1.0, ci_mode=1,
                                                        ci_on_below=3.0)))
    g = spx.gneb_create(hams, bufs, spring_k=1.0, vp_dt=0.05, vp_mass=1.0, ci_mode=1, ci_on_below=3.0)
    n_it = 15
    spx.gneb_step(g, n_it)
    torch.cuda.synchronize()
    for k, (m, st) in enumerate(refs):
        for _ in range(n_it):
            E, dist, fmax, ci = oracle.gneb_iterate(m, st)
        got = bufs[k].cpu().numpy()
        assert np.max(np.abs(got - st.Y)) <= 1e-9, (k, np.max(np.abs(got - st.Y)))
        s = spx.gneb_get_stats(g, k)
        np.testing.assert_allclose(s["E"], E, rtol=1e-10)
        assert s["ci_index"] == ci and s["iterations"] == n_it


def test_gneb_stoner_wohlfarth_barrier():
    import torch
    from paper_2605_26016_amd import spx
    MU_B = oracle.constants()[0]
    K, h = 1.0, 0.3
    w = Workload(name="t", L=(1, 1, 1), J_shell=(0.0,), K=K, B=(0, 0, 2 * K * h / MU_B), field_prec="fp64")
    A = np.array([[0.0], [0.0], [-1.0]])
    B = np.array([[0.0], [0.0], [1.0]])
    Yd = gpu_path(w, A, B, 9)
    g = spx.gneb_create([gpu_hamiltonian(w)], [Yd], spring_k=1.0, vp_dt=0.2, vp_mass=1.0, ci_mode=1,
                        ci_on_below=1e-2, tol_force=1e-9)
    spx.gneb_init_path(g)
    spx.gneb_step(g, 3000)
    s = spx.gneb_get_stats(g)
    assert s["converged"] == 1 and s["ci_on"] == 1 and s["iterations"] < 3000
    ci = s["ci_index"]
    Y = Yd.cpu().numpy()
    assert abs(Y[ci, 2, 0] - (-h)) < 1e-6
    assert abs((s["E"][ci] - s["E"][0]) - K * (1 - h) ** 2) < 1e-8


def test_gneb_two_pass_and_item_instances_match_oracle():
    # one batch with every form of the iteration: instances of several
    # z-march tiles per image with ragged x/y/z tails, periodic and open (the
    # two z-march passes, one partial set per tile, no stored force), a thin
    # column with more tiles per image than 256-site items (the z-march stores
    # the field and the item passes read it), and a gather-engine instance
    # (item passes that gather the neighbours); their passes run side by side
    import torch
    from paper_2605_26016_amd import spx
    cases = [(frustrated((70, 10, 20), periodic=(1, 0, 1)), 5, 21, {}), (frustrated((66, 9, 18)), 4, 23, {}),
             (frustrated((2, 2, 40)), 4, 22, {}), (frustrated((5, 4, 3)), 5, 24, dict(stencil_engine=1))]
    hams, bufs, refs = [], [], []
    for w, n_img, seed, setup in cases:
        A, B = endpoints(w, seed)
        Y0 = oracle.geodesic_path(A, B, n_img)
        hams.append(gpu_hamiltonian(w, **setup))
        bufs.append(to_dev(Y0))
        refs.append((oracle_model(w), oracle.GnebState(Y0, k_spring=1.0, dt=0.05, mass=1.0, ci_mode=1,
                                                        ci_on_below=3.0)))
    g = spx.gneb_create(hams, bufs, spring_k=1.0, vp_dt=0.05, vp_mass=1.0, ci_mode=1, ci_on_below=3.0)
    for it in range(8):
        spx.gneb_step(g, 1)
        torch.cuda.synchronize()
        for k, (m, st) in enumerate(refs):
            E, dist, fmax, ci = oracle.gneb_iterate(m, st)
            got = bufs[k].cpu().numpy()
            assert np.max(np.abs(got - st.Y)) <= 1e-9, (it, k, np.max(np.abs(got - st.Y)))
            s = spx.gneb_get_stats(g, k)
            np.testing.assert_allclose(s["E"], E, rtol=1e-10, atol=1e-12)
            np.testing.assert_allclose(s["dist"], dist, rtol=1e-10, atol=1e-12)
            assert s["ci_index"] == ci and s["iterations"] == it + 1


def test_gneb_two_pass_tile_widths_match_oracle():
    # three-shell instances (256-thread blocks) on lattices whose padded area
    # is smallest at each tile width: 100 x 4 -> 64 x 4 tiles, 20 x 19 ->
    # 32 x 8 tiles (ragged x and y), 14 x 30 -> 16 x 16 tiles (ragged x and
    # y); odd image counts, so the image-fastest tile order wraps the XCD runs
    # unevenly, open and periodic faces
    import torch
    from paper_2605_26016_amd import spx

    def three(L, periodic):
        return Workload(name="t", L=L, periodic=periodic, J_shell=(1.0, -0.164, -0.082), K=0.05,
                        B=(0.0, 0.0, 0.3), field_prec="fp64")

    cases = [(three((100, 4, 5), (1, 0, 1)), 5, 31), (three((20, 19, 7), (1, 1, 0)), 7, 32),
             (three((14, 30, 5), (0, 0, 0)), 6, 33)]
    hams, bufs, refs = [], [], []
    for w, n_img, seed in cases:
        A, B = endpoints(w, seed)
        Y0 = oracle.geodesic_path(A, B, n_img)
        hams.append(gpu_hamiltonian(w))
        bufs.append(to_dev(Y0))
        refs.append((oracle_model(w), oracle.GnebState(Y0, k_spring=1.0, dt=0.05, mass=1.0, ci_mode=1,
                                                        ci_on_below=3.0)))
    g = spx.gneb_create(hams, bufs, spring_k=1.0, vp_dt=0.05, vp_mass=1.0, ci_mode=1, ci_on_below=3.0)
    for it in range(6):
        spx.gneb_step(g, 1)
        torch.cuda.synchronize()
        for k, (m, st) in enumerate(refs):
            E, dist, fmax, ci = oracle.gneb_iterate(m, st)
            got = bufs[k].cpu().numpy()
            err = float(np.max(np.abs(got - st.Y)))
            assert err <= 1e-9, (it, k, err)
            s = spx.gneb_get_stats(g, k)
            np.testing.assert_allclose(s["E"], E, rtol=1e-10, atol=1e-12)
            np.testing.assert_allclose(s["dist"], dist, rtol=1e-10, atol=1e-12)
            assert s["ci_index"] == ci and s["iterations"] == it + 1


FILMS = [("nn", dict(J_shell=(1.0,))), ("chiral", dict(J_shell=(1.0,), D_shell=(0.3,))),
         ("three", dict(J_shell=(1.0, -0.164, -0.082))), ("four", dict(J_shell=(1.0, 0.188, -0.274, -0.161)))]


@pytest.mark.parametrize("ci_mode", [1, 4], ids=["climbing", "string"])
@pytest.mark.parametrize("couplings", [f[1] for f in FILMS], ids=[f[0] for f in FILMS])
def test_gneb_films_match_oracle(couplings, ci_mode):
    # one plane, open in z: the passes march through the images.  One batch of
    # every tile width (16, 64 and 32) with ragged x and y tiles, image counts
    # that leave a short last run of images per block, wrapped and open edges,
    # an edge shorter than the couplings' reach, the least number of images,
    # and a film periodic in z (which marches through planes)
    import torch
    from paper_2605_26016_amd import spx
    cases = [((100, 97, 1), (1, 1, 0), 21), ((14, 30, 1), (0, 0, 0), 8), ((70, 4, 1), (1, 0, 0), 3),
             ((33, 9, 1), (0, 1, 0), 5), ((1, 2, 1), (0, 0, 0), 4), ((9, 12, 1), (1, 1, 1), 5)]
    hams, bufs, refs = [], [], []
    kw = dict(k_spring=1.0, dt=0.05, mass=1.0, ci_mode=ci_mode, ci_on_below=3.0)
    for k, (L, periodic, n_img) in enumerate(cases):
        w = Workload(name="t", L=L, periodic=periodic, K=0.05, B=(0.0, 0.0, 0.3), field_prec="fp64", **couplings)
        A, B = random_sphere(w.N, 41 + k), random_sphere(w.N, 141 + k)
        Y0 = oracle.geodesic_path(A, B, n_img)
        hams.append(gpu_hamiltonian(w))
        bufs.append(to_dev(Y0))
        refs.append((oracle_model(w), oracle.GnebState(Y0, **kw)))
    g = spx.gneb_create(hams, bufs, spring_k=1.0, vp_dt=0.05, vp_mass=1.0, ci_mode=ci_mode, ci_on_below=3.0)
    for it in range(4):
        spx.gneb_step(g, 1)
        torch.cuda.synchronize()
        for k, (m, st) in enumerate(refs):
            E, dist, fmax, ci = oracle.gneb_iterate(m, st)
            got = bufs[k].cpu().numpy()
            err = float(np.max(np.abs(got - st.Y)))
            assert err <= 1e-9, (it, k, err)
            s = spx.gneb_get_stats(g, k)
            np.testing.assert_allclose(s["E"], E, rtol=1e-10, atol=1e-10)
            np.testing.assert_allclose(s["dist"], dist, rtol=1e-10, atol=1e-10)
            np.testing.assert_allclose(s["max_force"], fmax, rtol=1e-9)
            assert s["ci_index"] == ci and s["iterations"] == it + 1


@pytest.mark.parametrize("ci_mode", [1, 4], ids=["climbing", "string"])
def test_gneb_long_graph_equals_single_steps(ci_mode):
    # from 128 iterations of a handle on, calls of eight or more replay a graph
    # of eight and single ones for the rest: bit for bit the direct launches,
    # with the program's own work between the replays
    import torch
    from paper_2605_26016_amd import spx
    cases = [(frustrated((17, 9, 1), periodic=(1, 1, 0)), 5, 31), (frustrated((6, 6, 4)), 4, 32),
             (frustrated((2, 2, 40)), 4, 33)]
    bufs, handles = ([], []), []
    for b in bufs:
        for w, n_img, seed in cases:
            b.append(to_dev(oracle.geodesic_path(random_sphere(w.N, seed), random_sphere(w.N, seed + 100), n_img)))
        handles.append(spx.gneb_create([gpu_hamiltonian(w) for w, _, _ in cases], b, ci_mode=ci_mode,
                                       ci_on_below=3.0, vp_dt=0.02))
    done = 0
    for n in (120, 8, 7, 21, 40, 1, 17):
        spx.gneb_step(handles[0], n)
        for _ in range(n):
            spx.gneb_step(handles[1], 1)
        done += n
        torch.cuda.synchronize()
        for k, (x, y) in enumerate(zip(*bufs)):
            assert torch.equal(x, y), (done, k)
            assert float(x.square().sum(1).sub(1.0).abs().max()) < 1e-12
            assert spx.gneb_get_stats(handles[0], k)["iterations"] == done


def test_statistics_from_several_threads():
    # threads that read the statistics of one handle's instances at the same
    # time, each on a stream of its own, each get their own instance's
    import threading

    import torch
    from paper_2605_26016_amd import spx
    cases = [(frustrated((4, 4, 4)), 3, 51), (frustrated((5, 4, 3)), 40, 52), (frustrated((3, 3, 3)), 17, 53),
             (frustrated((6, 5, 2)), 9, 54)]
    g = spx.gneb_create([gpu_hamiltonian(w) for w, _, _ in cases],
                        [to_dev(oracle.geodesic_path(random_sphere(w.N, s), random_sphere(w.N, s + 100), n))
                         for w, n, s in cases])
    spx.gneb_step(g, 3)
    torch.cuda.synchronize()
    want = [spx.gneb_get_stats(g, k) for k in range(len(cases))]
    streams = [torch.cuda.Stream() for _ in cases]
    wrong = []

    def read(k):
        for _ in range(500):
            s = spx.gneb_get_stats(g, k, stream=streams[k])
            if not (np.array_equal(s["E"], want[k]["E"]) and np.array_equal(s["dist"], want[k]["dist"])
                    and s["max_force"] == want[k]["max_force"]):
                wrong.append(k)
                return

    threads = [threading.Thread(target=read, args=(k,)) for k in range(len(cases))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


@pytest.mark.parametrize("n_img", [20, 130], ids=["passes", "items"])
@pytest.mark.parametrize("couplings", [f[1] for f in FILMS], ids=[f[0] for f in FILMS])
def test_ragged_lattices_of_few_and_many_images(couplings, n_img):
    # films periodic in z, whose tiles are more than their items: the two passes
    # up to 512 x 1024 sites x images of a batch, the item passes beyond (four
    # shells: the two passes)
    import torch
    from paper_2605_26016_amd import spx
    cases = [((65, 65, 1), (1, 1, 1)), ((33, 9, 1), (0, 1, 1))]
    hams, bufs, refs = [], [], []
    kw = dict(k_spring=1.0, dt=0.05, mass=1.0, ci_mode=1, ci_on_below=3.0)
    for k, (L, periodic) in enumerate(cases):
        w = Workload(name="t", L=L, periodic=periodic, K=0.05, B=(0.0, 0.0, 0.3), field_prec="fp64", **couplings)
        Y0 = oracle.geodesic_path(random_sphere(w.N, 61 + k), random_sphere(w.N, 161 + k), n_img)
        hams.append(gpu_hamiltonian(w))
        bufs.append(to_dev(Y0))
        refs.append((oracle_model(w), oracle.GnebState(Y0, **kw)))
    g = spx.gneb_create(hams, bufs, spring_k=1.0, vp_dt=0.05, vp_mass=1.0, ci_mode=1, ci_on_below=3.0)
    for it in range(2):
        spx.gneb_step(g, 1)
        torch.cuda.synchronize()
        for k, (m, st) in enumerate(refs):
            E, dist, fmax, ci = oracle.gneb_iterate(m, st)
            assert float(np.max(np.abs(bufs[k].cpu().numpy() - st.Y))) <= 1e-9, (it, k)
            s = spx.gneb_get_stats(g, k)
            np.testing.assert_allclose(s["E"], E, rtol=1e-10, atol=1e-10)
            np.testing.assert_allclose(s["dist"], dist, rtol=1e-10, atol=1e-10)
            np.testing.assert_allclose(s["max_force"], fmax, rtol=1e-9)
