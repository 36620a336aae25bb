"""GPU static minimisers (spx_min_*) against the FP64 oracle, iteration by
iteration, for every method and retraction; convergence to the closed-form
ferromagnet ground state; argument checks.

Tolerances: state after each of 12 iterations <= 1e-9 per component and the
reported max |F| to 1e-9 relative (FP64 on both sides; the GPU's reductions
sum in another order); ground-state energy 1e-8 meV per spin.
"""
import numpy as np
import pytest

import oracle
from tests.helpers import gpu_hamiltonian, oracle_model, require_gpu, to_dev
from workloads import Workload, random_sphere

pytestmark = pytest.mark.gpu

MU_B = 5.7883818060e-2
SETTINGS = {"vp": dict(dt=0.2), "bb": dict(dt=0.05), "lbfgs": dict(dt=0.05, history=3), "adam": dict(dt=0.05)}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


# the force pass runs inside the z-march field evaluation (one tile, or
# several with ragged x/y/z tails) or, with the gather engine, as its own
# pass after the field
LATTICES = {"one_tile": ((5, 4, 3), 0), "multitile": ((70, 9, 18), 0), "gather": ((5, 4, 3), 1)}


@pytest.mark.parametrize("lattice", list(LATTICES))
@pytest.mark.parametrize("method", ["vp", "bb", "lbfgs", "adam"])
@pytest.mark.parametrize("retraction", ["exp", "norm"])
def test_iterations_match_the_oracle(method, retraction, lattice):
    from paper_2605_26016_amd import spx
    L, engine = LATTICES[lattice]
    w = Workload(name="f", L=L, periodic=(1, 0, 1), J_shell=(1.0, 0.188, -0.274), K=0.3,
                 K_axis=(0.0, 0.6, 0.8), B=(0.5, 0.0, 1.0), field_prec="fp64")
    S0 = random_sphere(w.N, 7)
    S = to_dev(S0)
    kw = dict(SETTINGS[method])
    mn = spx.min_create(gpu_hamiltonian(w, stencil_engine=engine), method=method, retraction=retraction,
                        max_step=0.3, **kw)
    hist = kw.pop("history", 5)
    st = oracle.MinState(w.N, method, retraction, max_step=0.3, hist=hist, **kw)
    ref = S0.copy()
    m = oracle_model(w)
    for it in range(12):
        f = oracle.min_iterate(m, ref, st)
        spx.min_step(mn, S, 1)
        s = spx.min_get_stats(mn)
        err = float(np.max(np.abs(S.cpu().numpy() - ref)))
        assert err <= 1e-9, (it, err)
        assert abs(s["max_force"] - f) <= 1e-9 * max(1.0, f), (it, s["max_force"], f)
        assert s["iterations"] == it + 1


@pytest.mark.parametrize("method", ["vp", "bb", "lbfgs", "adam"])
def test_ferromagnet_converges_to_the_ground_state(method):
    # Adam with a constant step keeps moving by about dt per component near
    # the minimum (its steps are normalised by the gradient's own scale), so
    # it ends in an O(dt) neighbourhood: its bound is on the energy, with a
    # small step, not on convergence
    import torch
    from paper_2605_26016_amd import spx
    J, K, h = 1.0, 0.2, 6.0
    w = Workload(name="fm", L=(16, 16, 16), J_shell=(J,), K=K, B=(0.0, 0.0, h / MU_B), field_prec="fp64")
    S = to_dev(random_sphere(w.N, 9))
    ham = gpu_hamiltonian(w)
    kw = dict(SETTINGS[method])
    if method == "adam":
        kw["dt"] = 0.002
    mn = spx.min_create(ham, method=method, max_step=0.3, tol_force=0.0 if method == "adam" else 1e-9, **kw)
    spx.min_step(mn, S, 6000)
    s = spx.min_get_stats(mn)
    E = torch.zeros(1, dtype=torch.float64, device="cuda")
    spx.energy(ham, S, E)
    excess = float(E.item()) / w.N - (-(3 * J + K + h))
    if method == "adam":
        assert 0.0 <= excess < 1e-4, excess
    else:
        assert s["converged"] == 1 and s["iterations"] < 6000, s
        assert abs(excess) < 1e-8


def test_arguments_are_checked():
    from paper_2605_26016_amd import spx
    w = Workload(name="a", L=(3, 3, 3), J_shell=(1.0,), field_prec="fp64")
    h = gpu_hamiltonian(w)
    for kw in (dict(method=4), dict(retraction=2), dict(dt=0.0), dict(method="lbfgs", history=0),
               dict(method="lbfgs", history=33), dict(max_step=-1.0)):
        with pytest.raises(spx.SpxError):
            spx.min_create(h, **kw)
    w32 = Workload(name="b", L=(3, 3, 3), J_shell=(1.0,), field_prec="fp32")
    with pytest.raises(spx.SpxError):
        spx.min_create(gpu_hamiltonian(w32))


@pytest.mark.parametrize("history", [1, 2, 4, 5, 6, 8, 9])
def test_lbfgs_histories_match_the_oracle(history):
    # each size of the scalar recursion, exactly full and not, and the vector
    # recursion beyond it (9); a lattice of more sites than one block, with
    # tails; the history is full from iteration `history` + 1 on
    from paper_2605_26016_amd import spx
    w = Workload(name="f", L=(21, 10, 7), periodic=(1, 0, 1), J_shell=(1.0,), K=0.3, B=(0.5, 0.0, 1.0),
                 field_prec="fp64")
    S0 = random_sphere(w.N, 19)
    S = to_dev(S0)
    mn = spx.min_create(gpu_hamiltonian(w), method="lbfgs", dt=0.05, history=history, max_step=0.3)
    st = oracle.MinState(w.N, "lbfgs", "exp", max_step=0.3, hist=history, dt=0.05)
    ref = S0.copy()
    m = oracle_model(w)
    for it in range(13):
        oracle.min_iterate(m, ref, st)
        spx.min_step(mn, S, 1)
        err = float(np.max(np.abs(S.cpu().numpy() - ref)))
        assert err <= 1e-9, (it, err)


@pytest.mark.parametrize("engine", [0, 1], ids=["z_march", "gather"])
@pytest.mark.parametrize("method,history", [("vp", 1), ("bb", 1), ("lbfgs", 3), ("lbfgs", 9), ("adam", 1)])
@pytest.mark.parametrize("per_graph", [1, 3])
def test_captured_iterations_can_be_replayed(method, history, engine, per_graph):
    # a program may capture spx_min_step itself: an odd number of iterations a
    # graph, replayed several times with direct iterations in between, gives
    # the states of as many direct iterations, bit for bit
    import torch
    from paper_2605_26016_amd import spx
    w = Workload(name="c", L=(13, 6, 5), J_shell=(1.0, 0.2), K=0.3, B=(0.5, 0.0, 1.0), field_prec="fp64")
    S0 = to_dev(random_sphere(w.N, 23))
    h = gpu_hamiltonian(w, stencil_engine=engine)
    kw = dict(method=method, dt=0.05, history=history, max_step=0.3)
    ma, mb = spx.min_create(h, **kw), spx.min_create(h, **kw)
    Sa, Sb = S0.clone(), S0.clone()
    spx.min_step(mb, Sb, 1)  # the kernels are loaded before the capture
    spx.min_reset(mb)
    Sb.copy_(S0)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        spx.min_step(mb, Sb, per_graph)
    done = 0
    for rep in range(5):
        graph.replay()
        done += per_graph
        if rep in (1, 2):
            spx.min_step(mb, Sb, 1)
            done += 1
        spx.min_step(ma, Sa, done - spx.min_get_stats(ma)["iterations"])
        torch.cuda.synchronize()
        assert spx.min_get_stats(mb)["iterations"] == done
        assert torch.equal(Sa, Sb), rep


@pytest.mark.parametrize("engine", [0, 1], ids=["z_march", "gather"])
@pytest.mark.parametrize("method,history,vectors", [("vp", 1, 2), ("bb", 1, 3), ("lbfgs", 5, 15), ("lbfgs", 9, 24),
                                                    ("adam", 1, 3)])
def test_state_holds_only_what_the_method_reads(method, history, vectors, engine):
    # device memory taken by a minimiser in vectors of the state (12.6 MB; the
    # allocator's granularity and the scalars stay below one): two forces; the
    # previous step; 2 (history + 1) pairs; q of the vector recursion; Adam's
    # force and moments; the field where the force is a pass of its own
    import torch
    from paper_2605_26016_amd import spx
    w = Workload(name="m", L=(128, 64, 64), J_shell=(1.0,), field_prec="fp64")
    h = gpu_hamiltonian(w, stencil_engine=engine)
    free = torch.cuda.mem_get_info()[0]
    mn = spx.min_create(h, method=method, history=history, dt=0.05)
    used = (free - torch.cuda.mem_get_info()[0]) / (24 * w.N)
    S = to_dev(random_sphere(w.N, 3))
    spx.min_step(mn, S, 3)
    assert spx.min_get_stats(mn)["iterations"] == 3 and float((S * S).sum(0).sub(1.0).abs().max()) < 1e-12
    print(f"{method} {history}: {used:.2f} vectors", flush=True)
    assert used < vectors + engine + 1
