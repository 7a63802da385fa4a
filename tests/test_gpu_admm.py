"""GPU parity of the whole ADMM sweep against the CPU oracle, iteration by iteration, on the same seeded
inputs (tolerance 1e-4 relative on W, Z, U and the objective; step-size trajectories identical)."""
import copy

import numpy as np
import pytest

from oracle.admm import make_oracle
from paper_2112_09335_amd import synth
from parity import compare_iterate, expected_ties, record_case, say, step_with_relu_ties

pytestmark = pytest.mark.gpu


def low_rank_launches(solver):
    """How many gradients one more iteration keeps in low-rank form."""
    solver.profile(True)
    solver.run(1)
    n = solver.get_profile()["gemm_nn_gradz_kernel"]["records"]
    solver.profile(False)
    return n


def run_case(w, iters, tag, max_ties=None, tune=None):
    """Per-iteration parity of one workload.  A hidden pre-activation within fp32 rounding of zero (a ReLU tie, see
    step_with_relu_ties) is accepted only entry by entry, and in at most max_ties iterations of the case: the number
    of tied entries expected for its size and length (parity.expected_ties) rounded up, at least one."""
    max_ties = max(1, int(np.ceil(expected_ties(w.N, w.dims, iters)))) if max_ties is None else max_ties
    from paper_2112_09335_amd import binding
    say(f"[{tag}] N={w.N} M={w.M} dims={w.dims} E={w.E} iters={iters}")
    solver = binding.Solver.from_workload(w, 0)
    for key, value in (tune or {}).items():
        solver.tune(key, value)
    orc = make_oracle(w)
    ties, worst, done = [], 0.0, 0
    try:
        worst = compare_iterate(solver, orc, f"{tag} it0")
        for k in range(1, iters + 1):
            err, flipped = step_with_relu_ties(solver, orc, f"{tag} it{k}")
            worst = max(worst, err)
            if flipped:
                ties.append(dict(iter=k, entries=flipped))
            done = k
            say(f"[{tag}] it{k} ok, worst rel err so far {worst:.2e}")
        if "use_lowrank" in (tune or {}):                # (the case says which path it is for)
            assert (low_rank_launches(solver) > 0) == (tune["use_lowrank"] == 2)
        assert len(ties) <= max_ties, f"{len(ties)} iterations with ReLU ties in {iters} iterations"
    finally:
        solver.close()
        record_case(case=tag, N=int(w.N), dims=list(w.dims), iters=iters, iters_done=done, worst=worst, ties=ties,
                    max_ties=max_ties, expected_ties=expected_ties(w.N, w.dims, iters),
                    ok=bool(done == iters and len(ties) <= max_ties))
    return worst


def test_config1_tiny_sbm_all_iterations():
    w = synth.config(1)
    run_case(w, w.iters, "config1")


def test_config2_mid_sbm_scaled():
    w = synth.config(2, 0.1)             # N = 2000, 500 -> 128 -> 3
    run_case(w, 12, "config2/10")


def test_config3_three_layers_scaled():
    w = synth.config(3, 0.01)            # N = 2000, 32 communities, 128 -> 256 -> 256 -> 10
    run_case(w, 8, "config3/100")


def test_config4_powerlaw_scaled():
    w = synth.config(4, 0.002)           # N = 4000, 64 communities, hubs, 128 -> 256 -> 16
    run_case(w, 8, "config4/500")


def test_config5_deep_scaled():
    w = synth.config(5, 0.002, M=4)      # N = 1000, 8 layers of 512
    run_case(w, 4, "config5/500")


def test_unlabelled_nodes_least_squares_risk_one_community_and_ragged_sizes():
    w = synth.make_workload("ragged", 11, 1237, 5, [37, 50, 9, 6], 6, 6, graph="sbm", features="gaussian",
                            avg_degree=6, frac_intra=0.7, labelled_fraction=0.4)
    w.comm = np.where(w.comm == 3, 4, w.comm).astype(np.int32)      # community 3 is empty
    run_case(w, 6, "ragged-ce")
    w2 = copy.deepcopy(w)
    w2.hyper["risk"] = 1
    run_case(w2, 4, "ragged-lsq")
    w3 = synth.make_workload("single", 12, 600, 1, [20, 33, 4], 4, 5, graph="sbm", features="gaussian",
                             avg_degree=8, frac_intra=1.0)
    run_case(w3, 5, "one-community")
    w4 = synth.make_workload("noedges", 13, 300, 3, [10, 12, 3], 3, 3, graph="empty", features="gaussian")
    run_case(w4, 3, "empty-graph")


@pytest.mark.parametrize("dims,more", [([101, 301, 90, 6], {}), ([30, 90, 301, 70, 7], {"step_policy": 1}),
                                       ([67, 49, 261, 3], {"schedule": 1, "fista_mode": 1})])
def test_ragged_widths_across_column_tiles(dims, more):
    """Widths that are no multiple of four on both sides of the narrow-side rule: the searches' row sums are left by the
    64-column product over several tiles or by the aggregation in one tile, with a partial last quad in either."""
    w = synth.make_workload("ragged-wide", 21 + len(more), 1501, 5, dims, dims[-1], 4, graph="sbm", features="gaussian",
                            avg_degree=9, frac_intra=0.8, labelled_fraction=0.4)
    w.hyper.update(more)
    run_case(w, 4, "ragged-wide/" + "-".join(map(str, dims)))


def copies(w, n):
    """n disjoint copies of a workload: every copy goes through the same values, so a workload of any size has the ReLU ties
    of a small one."""
    at = np.repeat(np.arange(n, dtype=np.int64) * w.N, w.E)
    return synth.Workload(w.name, w.N * n, w.M, (np.tile(w.src, n) + at).astype(np.int32), (np.tile(w.dst, n) + at).astype(np.int32),
                          np.tile(w.comm, n), np.tile(w.X, (n, 1)), np.tile(w.labels, n), w.dims, w.W0, w.iters, dict(w.hyper))


@pytest.mark.parametrize("dims", [[24, 133, 46, 5], [24, 136, 48, 5], [201, 133, 46, 5]])
def test_many_rows_reach_the_128_column_products(dims):
    """From 512 tiles of 128 x 128 on: the first trial of tau_1 with its step, and the gradient of Z_1 with its row sums over
    a whole and a partial column tile, at widths with and without a partial last quad.  201 x 133: the gradient of W_1 in
    tiles of 256 x 128, chunks that end within a step."""
    w = copies(synth.make_workload("many-rows", 41, 101, 3, dims, dims[-1], 4, graph="sbm", features="gaussian", avg_degree=8,
                                   frac_intra=0.7), 325)
    assert -(-w.N // 128) * -(-dims[1] // 128) >= 512
    run_case(w, 6, "many-rows/" + "-".join(map(str, dims)))


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("dims,n", [([24, 133, 136, 5], 325), ([201, 480, 400, 5], 163)])
def test_two_wide_layers_of_many_rows_take_every_branch_of_the_w_step(dims, n, policy):
    """Layer 2 from 512 tiles of 128 x 128 on: the product that leaves G_2 beside its first trial, where the search takes no step,
    accepts what was taken ahead, and (steps that may shrink) rejects it.  480 x 400: the gradient of W_2 in several tiles of
    256 x 128, the last one partial in either direction."""
    from paper_2112_09335_amd import binding
    w = copies(synth.make_workload("many-rows", 41, 101, 3, dims, dims[-1], 4, graph="sbm", features="gaussian", avg_degree=8,
                                   frac_intra=0.7), n)
    w.hyper["step_policy"] = policy
    tiles = lambda a, b, t: -(-a // t) * -(-b // 128)
    assert tiles(w.N, dims[2], 128) >= 512
    if dims[1] > 256:
        K, C = dims[1:3]
        assert 2 * -(-K // 256) == -(-K // 128)                            # the rows of W fill tiles of 256
        assert min(1024 // tiles(K, C, 128), w.N * (K + C) // (2 * K * C)) * tiles(K, C, 128) >= 512      # and tiles of 128 would do
        assert tiles(K, C, 256) > 4 and K % 256 and C % 128
    say(f"[two-wide/{dims}/{policy}] N={w.N}")
    solver, orc, trials = binding.Solver.from_workload(w, 0), make_oracle(w), []
    try:
        for k in range(6):
            step_with_relu_ties(solver, orc, f"two-wide/{dims}/{policy} it{k + 1}")
            trials.append(int(solver.get_steps()[2][1]))
            say(f"it{k + 1} ok, candidates of the W search of layer 2: {trials[-1]}")
    finally:
        solver.close()
    ahead = [after for before, after in zip(trials, trials[1:]) if before == 1]         # what followed an accepted first candidate
    assert 0 in trials and (max(ahead) > 1 if policy else 1 in ahead), trials


@pytest.mark.parametrize("start,candidates", [(40, 21 + 16), (52, 21 + 32)])
@pytest.mark.parametrize("n", [20, 44, 60, 90])
def test_the_last_candidates_of_a_search_come_in_rounds(n, start, candidates):
    """tau_1 starts 2^start too small: the search accepts in the second round of sixteen candidates of its last pass or in a later
    one.  262 to 1181 workgroups a round: four, three or two rounds side by side, or one after the other; the smallest has all
    candidates in one pass, the others come to it behind passes of four and sixteen."""
    from paper_2112_09335_amd import binding
    w = copies(synth.make_workload("late", 41, 101, 3, [24, 133, 5], 5, 4, graph="sbm", features="gaussian", avg_degree=8,
                                   frac_intra=0.7), n)
    w.hyper.update(tau0=1e-3 * 2.0 ** -start, max_backtrack=64)
    say("late candidates", w.N, start)
    solver, orc, trials = binding.Solver.from_workload(w, 0), make_oracle(w), []
    try:
        for k in range(4):
            step_with_relu_ties(solver, orc, f"late{n}/{start} it{k + 1}")
            trials.append(int(solver.get_steps()[2][0]))
    finally:
        solver.close()
    assert max(trials) > candidates, trials


def test_backtracking_cap_status_and_resume_are_consistent():
    from paper_2112_09335_amd import binding
    w = synth.config(1, 0.5)
    w.hyper["max_backtrack"] = 2
    run_case(w, 3, "cap")                # both sides must raise the same status bit
    # resume: 4 iterations == 2 iterations, state out and in again, 2 more (bit for bit on the GPU side)
    # (the first layer's pre-activation is normally carried across iterations; a resumed run has to form
    # it anew, so for a bit-for-bit comparison every run forms it in every iteration)
    w = synth.config(1, 0.5)
    a = binding.Solver.from_workload(w, 0)
    a.tune("t1_refresh", 0)
    a.run(4)
    b = binding.Solver.from_workload(w, 0)
    b.tune("t1_refresh", 0)
    b.run(2)
    tau, theta, _, _ = b.get_steps()
    W = [b.get_W(l) for l in range(1, w.L + 1)]
    Z = [b.get_Z(l) for l in range(1, w.L + 1)]
    U = b.get_U()
    c = binding.Solver.from_workload(w, 0)
    c.tune("t1_refresh", 0)
    c.set_state(W=W, Z=Z, U=U, tau=tau, theta=theta)
    c.run(2)
    for l in range(1, w.L + 1):
        assert np.array_equal(a.get_W(l), c.get_W(l))
        assert np.array_equal(a.get_Z(l), c.get_Z(l))
    assert np.array_equal(a.get_U(), c.get_U())
    # and the run itself is reproducible bit for bit
    d = binding.Solver.from_workload(w, 0)
    d.tune("t1_refresh", 0)
    d.run(4)
    assert np.array_equal(a.get_Z(1), d.get_Z(1)) and a.eval()["objective"] == d.eval()["objective"]
    # carrying the first layer's pre-activation changes the iterates only by rounding
    e = binding.Solver.from_workload(w, 0)
    e.run(4)
    assert np.abs(e.get_Z(1) - a.get_Z(1)).max() <= 1e-5 * np.abs(a.get_Z(1)).max()
    e.close()
    for s in (a, b, c, d):
        s.close()


def test_graph_replay_equals_plain_launches_bit_for_bit():
    """cadmm_run replays a captured HIP graph; with readouts (eager kernels, synchronisations) between the
    replays every iterate must equal the one from plain launches exactly."""
    from paper_2112_09335_amd import binding
    w = synth.config(2, 0.1)
    a = binding.Solver.from_workload(w, 0)
    b = binding.Solver.from_workload(w, 0)
    b.tune("use_graph", 0)
    for k in range(6):
        a.run(1 if k % 2 == 0 else 2)
        b.run(1 if k % 2 == 0 else 2)
        sa, sb = a.eval(), b.eval()
        assert sa == sb, (k, sa, sb)
        for l in range(1, w.L + 1):
            assert np.array_equal(a.get_W(l), b.get_W(l)), (k, l)
            assert np.array_equal(a.get_Z(l), b.get_Z(l)), (k, l)
        assert np.array_equal(a.get_U(), b.get_U())
        ta, tb = a.get_steps(), b.get_steps()
        assert all(np.array_equal(x, y) for x, y in zip(ta, tb))
    a.close()
    b.close()


@pytest.mark.parametrize("name,more", [("three", {}), ("lowrank", {"step_policy": 1}), ("deep", {}), ("ragged", {"schedule": 1, "dual_form": 1})])
def test_step_floor_tested_first_gives_the_same_iterates_bit_for_bit(name, more):
    """From the forward pass on the layers far from the last one take no step at first: nothing of what only a step needs is
    formed then.  One community is cut off from the labels, so that only some communities of a layer step later on."""
    from paper_2112_09335_amd import binding
    w = {"three": lambda: synth.config(3, 0.01), "lowrank": lambda: synth.config(4, 0.002), "deep": lambda: synth.config(5, 0.002, M=4),
         "ragged": lambda: synth.make_workload("floor", 71, 1501, 5, [30, 90, 301, 90, 7], 7, 4, graph="sbm", features="gaussian",
                                               avg_degree=9, frac_intra=0.8)}[name]()
    w.hyper.update(more)
    keep = (w.comm[w.src] != 1) == (w.comm[w.dst] != 1)
    w.src, w.dst = w.src[keep].copy(), w.dst[keep].copy()
    w.labels[w.comm == 1] = -1
    got = []
    for mode in (0, 2):
        s = binding.Solver.from_workload(w, 0)
        s.tune("use_floor_first", mode)
        if name == "lowrank":
            s.tune("use_lowrank", 2)
        s.run(5)
        tau, theta, trials, _ = s.get_steps()
        got.append([s.get_W(l) for l in range(1, w.L + 1)] + [s.get_Z(l) for l in range(1, w.L + 1)] + [s.get_U(), tau, theta, trials])
        s.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("dims,more,split", [([40, 64, 48, 64, 64, 5], {}, 1), ([40, 64, 48, 64, 64, 5], {"step_policy": 1}, 1),
                                             ([70, 192, 130, 200, 160, 5], {"dual_form": 1}, 2), ([60, 400, 100, 33, 36, 4], {}, 1),
                                             ([48, 24, 40, 20, 64, 90, 5], {}, 1), ([40, 96, 12, 64, 16, 48, 6], {}, 1)])
def test_layers_at_rest_are_left_as_they_are_bit_for_bit(dims, more, split):
    """A layer whose steps were below resolution is not looked at again until something it depends on has changed
    (launch_rest_w, launch_rest_z): the same iterates, step parameters and trial counts as without, whatever else is
    called between the iterations and over two exact evaluations of the pre-activations."""
    from paper_2112_09335_amd import binding
    w = synth.make_workload("rest", 77, 1301, 4, dims, dims[-1], 4, graph="sbm", features="gaussian", avg_degree=8, frac_intra=0.8)
    w.hyper.update(more)
    got = []
    try:
        for mode in (0, 2):
            s = binding.Solver.from_workload(w, 0)
            s.tune("gemm_split", split)                  # (process-wide)
            s.init(w.W0)
            s.tune("use_floor_first", mode)
            s.tune("use_lowrank", 2)
            s.tune("t1_refresh", 4)
            seen = []
            for k in (1, 1, 1, 1, 2, 3, 1):
                s.run(k)
                seen += [*s.get_steps()]
                if k == 2:
                    s.predict()
                if k == 3:
                    seen += [s.eval()["objective"]]
                    s.profile(True)                      # (the next iteration is not replayed)
            s.profile(False)
            Z = s.get_Z(1)
            s.set_state(Z=[Z * np.float32(1.25)] + [None] * (w.L - 1))
            s.run(2)
            seen += [s.get_W(l) for l in range(1, w.L + 1)] + [s.get_Z(l) for l in range(1, w.L + 1)] + [s.get_U(), *s.get_steps()]
            s.init(w.W0)                                 # and from the start again
            s.run(3)
            seen += [s.get_W(l) for l in range(1, w.L + 1)] + [s.get_Z(l) for l in range(1, w.L + 1)] + [*s.get_steps()]
            got.append(seen)
            s.close()
    finally:
        probe = binding.Solver(device=-1)
        probe.tune("gemm_split", 1)
        probe.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def solver_in_cleared_memory(w):
    """As Solver.from_workload, in a workspace that starts as zeros (the block that was freed last is handed out again)."""
    import torch
    from paper_2112_09335_amd import binding
    s = binding.Solver(0)
    s.build_graph(w.N, w.src, w.dst, w.M, w.comm)
    s.set_model(w.dims, **w.hyper)
    torch.cuda.empty_cache()
    zeros = torch.zeros(s.workspace_bytes() + 256, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    at = zeros.data_ptr()
    del zeros
    s.set_workspace()
    assert s.workspace.data_ptr() == at
    s.set_data(w.X, w.labels)
    return s


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("who", ["this", "other"])
@pytest.mark.parametrize("key,values", [("spmm_tile_cols", (4, 0)), ("spmm_tile_cols", (0, 4, 0)), ("gemm_split", (0, 2)), ("gemm_split", (2, 1, 2))])
def test_process_wide_knobs_turned_during_a_run(key, values, who, graph):
    """What an iteration leaves for the next one under one setting (largest magnitudes of rows, layers at rest, captured iterations)
    is not taken for what another one would leave, whichever context turns the knob: the same iterates as from a run that keeps
    nothing.  A second round from the initial weights meets the settings with everything captured already."""
    from paper_2112_09335_amd import binding
    w = synth.make_workload("knobs", 79, 1301, 4, [70, 192, 130, 200, 160, 5], 5, 4, graph="sbm", features="gaussian", avg_degree=8, frac_intra=0.8)
    got = []
    other = binding.Solver(device=-1)
    try:
        for keep in (0, 2):
            other.tune("gemm_split", 2)
            other.tune("spmm_tile_cols", 0)
            s = solver_in_cleared_memory(w)
            s.tune("use_floor_first", keep)
            s.tune("use_graph", graph if keep else 0)
            seen = []
            for again in range(2):
                for i, value in enumerate(values):
                    (s if who == "this" else other).tune(key, value)
                    if i == 0:
                        s.init(w.W0)
                    s.run(1)
                s.run(2)
                seen += [s.get_W(l) for l in range(1, w.L + 1)] + [s.get_Z(l) for l in range(1, w.L + 1)] + [s.get_U(), *s.get_steps()]
            assert all(np.isfinite(x).all() for x in seen)
            got.append(seen)
            s.close()
    finally:
        other.tune("gemm_split", 1)
        other.tune("spmm_tile_cols", 0)
        other.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


# layers of fewer than 2^24 entries look at the step floor with the search, larger ones before it: in front of, between, and two
# layers before one that rests
@pytest.mark.parametrize("dims", [[8, 40, 424, 5], [8, 40, 424, 420, 5], [8, 424, 40, 424, 5], [8, 424, 36, 40, 424, 5]])
@pytest.mark.parametrize("M", [1, 3])
def test_a_run_owes_nothing_to_the_run_before_it(M, dims):
    """A layer that rests from the forward pass on leaves no gradient for the layer in front of it: that one must not take what an
    earlier run from other weights has left for one."""
    from paper_2112_09335_amd import binding
    w = synth.make_workload("again", 87, 40000, M, dims, dims[-1], 3, graph="sbm", features="gaussian", avg_degree=4, frac_intra=0.8 if M > 1 else 1.0)
    got = []
    for mode in (0, 1):
        s = binding.Solver.from_workload(w, 0)
        s.tune("use_floor_first", mode)
        for first in (True, False):
            s.init([W * np.float32(3.0) for W in w.W0] if first else w.W0)
            s.run(4)
        got.append([s.get_W(l) for l in range(1, w.L + 1)] + [s.get_Z(l) for l in range(1, w.L + 1)] + [s.get_U(), *s.get_steps()])
        assert s.eval()["status"] == 0
        s.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("entry", [np.inf, np.nan, 3e38])
@pytest.mark.parametrize("split", [1, 2])
def test_layers_do_not_rest_on_numbers_that_are_not_finite(entry, split):
    """The gradients behind a forward pass are zero only where its pre-activations are finite (3e38 overflows in them)."""
    from paper_2112_09335_amd import binding
    w = synth.make_workload("rest-inf", 78, 700, 3, [70, 160, 140, 150, 5], 5, 4, graph="sbm", features="gaussian", avg_degree=8, frac_intra=0.8)
    w.X = w.X.copy()
    w.X[11, 3:9] = entry
    got = []
    probe = binding.Solver(device=-1)
    try:
        probe.tune("gemm_split", split)                  # (process-wide)
        for mode in (0, 2):
            s = binding.Solver.from_workload(w, 0)
            s.tune("use_floor_first", mode)
            s.run(3)
            got.append([s.get_W(l) for l in range(1, w.L + 1)] + [s.get_Z(l) for l in range(1, w.L + 1)] + [*s.get_steps(), s.eval()["status"]])
            s.close()
    finally:
        probe.tune("gemm_split", 1)
        probe.close()
    assert got[0][-1] != 0                               # (the first layer's search meets them)
    for a, b in zip(*got):
        assert np.array_equal(a, b, equal_nan=True)


def test_the_profile_books_only_what_ran():
    """From the forward pass on most layers take no step at first, and what only a step needs returns at once: neither its flops
    nor its bytes are booked, and its records are no records of its kernel's class."""
    from paper_2112_09335_amd import binding
    w = synth.config(5, 0.002, M=4)
    s = binding.Solver.from_workload(w, 0)
    try:
        s.tune("use_floor_first", 2)
        nnz, seen = s.graph_sizes()[0], set()
        for it in range(10):
            s.profile(True)
            s.run(1)
            prof = s.get_profile()
            s.profile(False)
            trials = s.get_steps()[2]
            moved_W = trials[:w.L] > 0
            moved_Z = (trials[w.L:].reshape(w.L - 1, w.M) > 0).any(axis=1)           # layers 1 .. L-1
            trial = next(p for name, p in prof.items() if name.endswith("+finish"))
            hidden = [l for l in range(1, w.L) if moved_W[l - 1]]
            assert trial["records"] == len(hidden)
            assert trial["flops"] == sum(2.0 * w.N * w.dims[l - 1] * w.dims[l] for l in hidden)
            seg, stepped = prof["spmm_rows_kernel[segments]"], [l for l in range(1, w.L) if moved_Z[l - 1]]
            assert seg["records"] == len(stepped)
            assert seg["flops"] == sum(2.0 * nnz * w.dims[l + 1] for l in stepped)
            assert prof["z_step_kernel"]["records"] == len(stepped)
            assert prof["t_carry_kernel"]["records"] == len([l for l in stepped if l + 1 < w.L])
            seen |= set(moved_W[:-1]) | set(moved_Z)
        assert seen == {True, False}                     # (both were met)
    finally:
        s.close()


@pytest.mark.parametrize("dims", [[40, 64, 96, 128, 132, 5], [48, 64, 12, 72, 16, 96, 5], [40, 200, 160, 132, 92, 5]])
def test_a_layer_at_rest_forms_no_gradient(dims):
    """Whichever way the gradient of Z_l is formed (the aggregation last, in front of a wider layer; the product last; low rank, in front
    of a narrow one), none of its launches does anything where the layer rests: the profile books those of the other layers alone."""
    from paper_2112_09335_amd import binding
    w = synth.make_workload("rest", 83, 1501, 4, dims, dims[-1], 4, graph="sbm", features="gaussian", avg_degree=8, frac_intra=0.8)
    s = binding.Solver.from_workload(w, 0)
    L, met = w.L, set()
    # the class of a layer's last launch that forms the gradient, as the widths decide it
    kind = {l: "gemm_nn_gradz_kernel" if dims[l + 1] <= 16 else "split_kernel<1>" if dims[l + 1] < dims[l] else "[rows,gradz]"
            for l in range(1, L)}
    try:
        s.tune("use_floor_first", 2)
        s.tune("use_lowrank", 2)
        s.run(1)                                         # (behind the forward pass layers of at most 32 units do not rest yet)
        moved_Z = [False] * (L + 1)
        for it in range(1, 2 * L):
            before, moved_W = moved_Z, [False] * (L + 2)
            s.profile(it >= 2)
            s.run(1)
            prof = s.get_profile() if it >= 2 else None
            s.profile(False)
            trials = s.get_steps()[2]
            moved_W = [False] + list(trials[:L] > 0)
            moved_Z = [False] + list((trials[L:].reshape(L - 1, w.M) > 0).any(axis=1)) + [True]
            if it < 2:
                continue
            runs = [l for l in range(1, L) if l + 1 == L or before[l - 1] or before[l] or before[l + 1] or moved_W[l] or moved_W[l + 1]]
            for name in set(kind.values()):
                booked = sum(p["records"] for full, p in prof.items() if full.endswith(name))
                assert booked == sum(kind[l] == name for l in runs), (it, name, runs)
            met |= {(kind[l], l in runs) for l in range(1, L)}
        assert {(k, True) for k in kind.values()} <= met and any(not runs for _, runs in met)
    finally:
        s.close()


def test_the_column_tile_knob_reaches_captured_iterations():
    """The tile width decides the order of an aggregation's sums and who leaves the row sums of the Z search: iterations
    captured before the knob was turned must not be replayed after it."""
    import torch
    from paper_2112_09335_amd import binding
    w = synth.config(3, 0.01)
    a, b = binding.Solver.from_workload(w, 0), binding.Solver.from_workload(w, 0)
    b.tune("use_graph", 0)
    try:
        X = torch.randn(w.N, 256, device="cuda")
        whole = a.op_aggregate(X)
        for tile in (0, 32, 0):
            a.tune("spmm_tile_cols", tile)               # process-wide: b follows
            assert torch.equal(a.op_aggregate(X), whole) == (tile == 0)
            a.run(3)
            b.run(3)
            for l in range(1, w.L + 1):
                assert np.array_equal(a.get_W(l), b.get_W(l)) and np.array_equal(a.get_Z(l), b.get_Z(l)), (tile, l)
    finally:
        a.tune("spmm_tile_cols", 0)
        a.close()
        b.close()


# below the staged sizes, one piece of 8 MB that is not full, full, two with the second one row, three
@pytest.mark.parametrize("N", [65535, 65536, 98305, 131072, 131073, 262145])
def test_large_readouts_come_out_whole(N):
    """64 bytes a row: what is read is what was set, through whichever pieces of pinned memory it leaves (from the second on)."""
    from paper_2112_09335_amd import binding
    s = binding.Solver(0)
    s.build_graph(N, np.zeros(0, np.int32), np.zeros(0, np.int32), 1, np.zeros(N, np.int32))
    s.set_model([2, 16, 3], **synth.DEFAULT_HYPER)
    s.set_workspace()
    s.set_data(np.ones((N, 2), np.float32), np.zeros(N, np.int32))
    s.init([np.ones((2, 16), np.float32), np.ones((16, 3), np.float32)])
    Z = np.random.default_rng(N).standard_normal((N, 16)).astype(np.float32)
    s.set_state(Z=[Z, None])
    for _ in range(3):
        assert np.array_equal(s.get_Z(1), Z)
    s.close()


def test_inference_matches_the_oracle_between_iterations():
    from paper_2112_09335_amd import binding
    w = synth.config(3, 0.01)
    solver = binding.Solver.from_workload(w, 0)
    orc = make_oracle(w)
    accs = []
    for k in range(0, 7):
        if k:
            solver.run(1)
            orc.iterate(1)
        pg, lg, ag = solver.predict()
        po, lo, ao = orc.predict()
        scale = np.abs(lo).max()
        assert np.abs(lg - lo).max() <= 1e-4 * scale
        top2 = np.sort(lo, axis=1)[:, -2:]
        clear = (top2[:, 1] - top2[:, 0]) > 1e-3 * scale          # rows whose class is not a near tie
        assert clear.mean() > 0.9
        assert np.array_equal(pg[clear], po[clear])
        assert abs(ag - ao) <= (~clear).mean() + 1e-12
        accs.append(ag)
        # predict leaves the iterate alone
        assert abs(solver.eval()["objective"] - orc.stats()["objective"]) <= 1e-4 * orc.stats()["objective"]
    say("accuracy per iteration", accs)
    solver.close()


@pytest.mark.parametrize("n,dims", [(700, [20, 33, 32, 5]), (701, [37, 3, 130, 4]), (40007, [16, 200, 129, 7]), (70001, [9, 5, 31, 3])])
def test_forward_pass_of_init_and_inference_over_product_shapes(n, dims):
    """The products leave relu(T_l) themselves: 64- and 128-column tiles, narrow ones for few and many rows, partial quads, and
    a hidden layer that aggregates on its narrow side.  Three fp32 contractions of at most 200 terms: far below 1e-5."""
    from oracle.graph import OracleGraph
    from paper_2112_09335_amd import binding
    w = synth.make_workload("forward", 61, n, 3, dims, dims[-1], 1, graph="sbm", features="gaussian", avg_degree=6, frac_intra=0.8)
    A = OracleGraph(w.N, w.src, w.dst, w.M, w.comm)
    solver = binding.Solver.from_workload(w, 0)
    try:
        X = w.X.astype(np.float64)
        for l, W in enumerate(w.W0, 1):
            X = (A.A @ (X[A.perm] @ W.astype(np.float64)))[A.inv_perm]
            X = np.maximum(X, 0.0) if l < w.L else X
            assert np.linalg.norm(solver.get_Z(l) - X) <= 1e-5 * np.linalg.norm(X), l
        _, logits, _ = solver.predict()
        assert np.linalg.norm(logits - X) <= 1e-5 * np.linalg.norm(X)
    finally:
        solver.close()


def test_dual_ascent_on_new_iterates_variant():
    w = synth.config(1, 0.5)
    w.hyper["dual_form"] = 1
    run_case(w, 6, "dual-form-1")
    w = synth.config(3, 0.005)
    w.hyper["dual_form"] = 1
    run_case(w, 5, "dual-form-1/3-layer")


def test_low_rank_gradient_path_and_its_stored_twin():
    """Narrow next layers (up to 16 units) keep the Z gradient in low-rank form (at this size if asked to); both that path and the
    stored-gradient path must match the oracle, three layers so that both hidden layers use it."""
    from paper_2112_09335_amd import binding
    w = synth.make_workload("lowrank", 21, 1500, 6, [36, 48, 12, 4], 4, 6, graph="sbm", features="gaussian",
                            avg_degree=9, frac_intra=0.8)
    run_case(w, 6, "low-rank", tune={"use_lowrank": 2})
    # the gradient kernel takes 32 columns at a time: a last step of four own columns, the factor's and zeros
    run_case(synth.make_workload("lowrank", 22, 1500, 6, [36, 100, 12, 4], 4, 5, graph="sbm", features="gaussian",
                                 avg_degree=9, frac_intra=0.8), 5, "low-rank/partial-step", tune={"use_lowrank": 2})
    a = binding.Solver.from_workload(w, 0)
    b = binding.Solver.from_workload(w, 0)
    a.tune("use_lowrank", 2)
    b.tune("use_lowrank", 0)
    a.run(5)
    b.run(5)
    for l in range(1, w.L + 1):
        za, zb = a.get_Z(l), b.get_Z(l)
        assert np.abs(za - zb).max() <= 1e-5 * np.abs(zb).max()
    ta, tb = a.get_steps(), b.get_steps()
    assert np.array_equal(ta[0], tb[0]) and np.array_equal(ta[1], tb[1]) and np.array_equal(ta[2], tb[2])
    assert low_rank_launches(a) == 2 and low_rank_launches(b) == 0
    a.close()
    b.close()


def test_layer_by_layer_schedule_matches_the_oracle():
    """Serial baseline of Section 4.1 (schedule 1): W_l then Z_l, layer after layer, newest values everywhere."""
    w = synth.config(1, 0.5)
    w.hyper["schedule"] = 1
    run_case(w, 8, "layer-by-layer/config1")
    w = synth.config(3, 0.01)                       # three layers: both kinds of hidden Z update
    w.hyper["schedule"] = 1
    run_case(w, 6, "layer-by-layer/config3")
    w = synth.config(4, 0.002)                      # narrow-side association, low-rank gradient, hub rows
    w.hyper["schedule"] = 1
    w.hyper["dual_form"] = 1
    run_case(w, 6, "layer-by-layer/config4/dual-form-1", tune={"use_lowrank": 2})
    w = synth.make_workload("serial", 14, 900, 1, [24, 40, 12, 5], 5, 5, graph="sbm", features="gaussian",
                            avg_degree=8, frac_intra=1.0)
    w.hyper["schedule"] = 1                         # the paper's serial run: one community
    run_case(w, 6, "layer-by-layer/one-community")


def test_step_parameters_that_may_shrink_again():
    """step_policy 1: every search starts one notch below the value accepted last time."""
    w = synth.config(1, 0.5)
    w.hyper["step_policy"] = 1
    run_case(w, 8, "step-policy-1/config1")
    w = synth.config(3, 0.01)
    w.hyper["step_policy"] = 1
    run_case(w, 6, "step-policy-1/config3")
    w = synth.config(4, 0.002)
    w.hyper["step_policy"] = 1
    w.hyper["schedule"] = 1
    run_case(w, 6, "step-policy-1/config4/layer-by-layer")


def test_fp32_matrix_core_path_matches_the_oracle_too():
    """The sweep with the wide products on the fp32 MFMA kernels (gemm_split = 0) instead of the bf16-split ones."""
    from paper_2112_09335_amd import binding
    w = synth.config(3, 0.01)
    probe = binding.Solver(device=-1)
    try:
        probe.tune("gemm_split", 0)              # process-wide switch
        run_case(w, 5, "fp32-mfma/config3")
    finally:
        probe.tune("gemm_split", 1)
        probe.close()


# three to sixteen units behind the last hidden layer, in whole quads and not; contractions of whole and partial steps; split rows
@pytest.mark.parametrize("dims,hubs", [([30, 64, 3], 0), ([33, 100, 36, 5], 0), ([40, 132, 16], 2), ([24, 256, 13], 2), ([50, 68, 40, 10], 2)])
def test_low_rank_gradient_behind_any_few_units(dims, hubs):
    w = synth.make_workload("low-rank", 51 + dims[-1], 1301, 4, dims, dims[-1], 4, graph="sbm", features="gaussian", avg_degree=8,
                            frac_intra=0.8, labelled_fraction=0.7)
    if hubs:
        w = synth.add_hubs(w, 5, hubs, 600, 0.5)
    run_case(w, 5, "low-rank/" + "-".join(map(str, dims)), tune={"use_lowrank": 2})


def test_low_rank_gradient_of_the_power_law_sample():
    run_case(synth.config(4, 0.002), 6, "low-rank/config4", tune={"use_lowrank": 2})


@pytest.fixture
def pairs_everywhere():
    """The products on pairs of fp16 wherever their form allows, not from a size on (process-wide)."""
    from paper_2112_09335_amd import binding
    probe = binding.Solver(device=-1)
    probe.tune("gemm_split", 2)
    yield
    probe.tune("gemm_split", 1)
    probe.close()


# One column tile, and a part of a second; contractions of one step, of whole and of partial ones; the gradient
# of Z by the product and by the aggregation; split rows, whose largest magnitude the combine kernel leaves
@pytest.mark.parametrize("dims,more,hubs", [([101, 301, 90, 6], {}, 0), ([64, 97, 97, 256, 257, 7], {"step_policy": 1}, 0),
                                            ([96, 256, 256, 10], {"schedule": 1}, 3), ([67, 449, 261, 65, 3], {"dual_form": 1}, 3)])
def test_products_on_pairs_inside_the_sweep(pairs_everywhere, dims, more, hubs):
    w = synth.make_workload("pairs", 31 + len(dims), 1501, 5, dims, dims[-1], 4, graph="sbm", features="gaussian",
                            avg_degree=9, frac_intra=0.8, labelled_fraction=0.7)
    if hubs:
        w = synth.add_hubs(w, 5, hubs, 700, 0.5)
    w.hyper.update(more)
    run_case(w, 4, "pairs/" + "-".join(map(str, dims)))


def first_layer(X, W1):
    """relu(X W_1): without edges A~ is the identity, and this is what the forward pass leaves as Z_1."""
    from paper_2112_09335_amd import binding
    N, (K, C) = X.shape[0], W1.shape
    s = binding.Solver(0)
    s.build_graph(N, np.zeros(0, np.int32), np.zeros(0, np.int32), 1, np.zeros(N, np.int32))
    s.set_model([K, C, 3], **synth.DEFAULT_HYPER)
    s.set_workspace()
    s.set_data(X, np.zeros(N, np.int32))
    s.init([W1, np.ones((C, 3), np.float32)])
    got = s.get_Z(1)
    s.close()
    return got


@pytest.mark.parametrize("N,K,C", [(1, 64, 129), (127, 65, 130), (128, 95, 192), (129, 96, 193), (1000, 97, 255), (300, 512, 256),
                                   (257, 129, 257), (640, 1000, 513)])
def test_product_on_pairs_of_scaled_rows_and_columns(pairs_everywhere, N, K, C):
    """Rows of X and columns of W_1 from 1e-12 to 1e12 (and zero rows) keep the accuracy of a 32-bit product, since each has a scale
    of its own."""
    rng = np.random.default_rng(N + K + C)
    X = rng.standard_normal((N, K)) * 10.0 ** rng.integers(-12, 13, (N, 1)) * (rng.random((N, 1)) < 0.95)
    X, W1 = X.astype(np.float32), (rng.standard_normal((K, C)) * 10.0 ** rng.integers(-12, 13, (1, C))).astype(np.float32)
    got = first_layer(X, W1)
    exact, mag = X.astype(np.float64) @ W1.astype(np.float64), np.abs(X).astype(np.float64) @ np.abs(W1).astype(np.float64)
    # (the tolerance of the other split products: a few roundings of 32-bit sums)
    assert np.all(np.abs(got - np.maximum(exact, 0.0)) <= 2e-6 * mag)


# (the aggregation of 40000 rows in one community goes in tiles of 32 columns: nineteen words a row)
@pytest.mark.parametrize("kind,N,K,C", [(kind, *shape) for kind in ("even", "outlier", "opposed", "one-hot", "tiny columns", "few", "one row", "one column")
                                        for shape in ((128, 95, 192), (300, 512, 256), (257, 129, 257), (640, 1000, 513))] +
                         [(kind, 40000, 608, 130) for kind in ("even", "opposed", "one row")])
def test_product_on_pairs_of_unlike_columns_and_rows(pairs_everywhere, kind, N, K, C):
    """Where the largest entries of a row meet zeros of a column, or small ones (a feature 1e8 times the others that has no weight,
    features as much larger as their weights are smaller, weights that pick one feature), parts of a row's largest entry are not
    parts of what a result is made of.  Such tiles of 128 x 256 results come from operands in all 24 bits, to the bit as the kernel-level
    product; the others stay on pairs."""
    rng = np.random.default_rng(N + K + C)
    X, W1 = rng.standard_normal((N, K)), rng.standard_normal((K, C))
    rows, cols = slice(0, N), slice(0, C)                # of the results that are not for pairs
    if kind == "even":
        rows = slice(0, 0)
    elif kind == "outlier":
        X[:, 3] *= 1e8
        W1[3] = 0.0
    elif kind == "opposed":
        size = np.exp(4.0 * rng.standard_normal(K))
        X, W1 = X * size, W1 / size[:, None]
    elif kind == "one-hot":
        X *= 10.0 ** rng.integers(-9, 4, K)
        W1 = np.where(np.arange(K)[:, None] == np.arange(C) % K, W1, 0.0)
    elif kind == "tiny columns":                         # a few features far below the rest, and weights that ask for nothing else
        X[:, 7:12] *= 1e-13
        W1 = np.where((np.arange(K) >= 7)[:, None] & (np.arange(K) < 12)[:, None], W1, 0.0)
    elif kind == "few":                                  # three entries in a row, weights of all sizes
        X[rng.random((N, K)) > 3.0 / K] = 0.0
        W1 *= np.exp(4.0 * rng.standard_normal((K, C)))
    elif kind == "one row":                              # of the last tile
        X[N - 1, 5] = 1e9
        rows = slice((N - 1) // 128 * 128, N)
    elif kind == "one column":
        W1[5, 0] = 1e9
        cols = slice(0, min(C, 256))
    X, W1 = X.astype(np.float32), W1.astype(np.float32)
    import torch
    from paper_2112_09335_amd import binding
    got = first_layer(X, W1)
    s = binding.Solver(0)
    triples = np.maximum(s.op_transform(torch.from_numpy(X).cuda(), torch.from_numpy(W1).cuda()).cpu().numpy(), 0.0)       # (has no counts)
    s.close()
    exact, mag = X.astype(np.float64) @ W1.astype(np.float64), np.abs(X).astype(np.float64) @ np.abs(W1).astype(np.float64)
    assert np.all(np.abs(got - np.maximum(exact, 0.0)) <= 2e-6 * mag)
    assert np.array_equal(got[rows, cols], triples[rows, cols])
    on_pairs = np.ones((N, C), bool)
    on_pairs[rows, cols] = False
    assert not on_pairs.any() or (got != triples)[on_pairs].mean() > 0.1


@pytest.mark.parametrize("more,hubs", [({}, 0), ({"schedule": 1}, 2), ({"dual_form": 1}, 0)])
def test_tiles_that_are_not_for_pairs_inside_the_sweep(pairs_everywhere, more, hubs):
    """A feature far larger than the others with weights as much smaller, weights whose rows differ by powers of ten, and as they are in
    some of the layers: both ways of forming a tile in every product of the sweep."""
    w = synth.make_workload("unlike", 41, 1501, 5, [96, 256, 200, 256, 10], 10, 4, graph="sbm", features="gaussian", avg_degree=9,
                            frac_intra=0.8, labelled_fraction=0.7)
    if hubs:
        w = synth.add_hubs(w, 5, hubs, 700, 0.5)
    w.X, w.W0 = w.X.copy(), [W.copy() for W in w.W0]
    w.X[:, 0] *= 256.0
    w.W0[0][0] /= 256.0
    w.W0[1] *= np.float32(2.0) ** -np.random.default_rng(5).integers(0, 40, (256, 1)).astype(np.float32)
    w.W0[1] *= 4.0
    w.hyper.update(more)
    run_case(w, 4, "pairs/unlike/" + ("+".join(more) or "default"))


def test_hub_rows_and_hub_segments_are_split_inside_the_sweep():
    """Rows and (row, community) segments above the aggregation's split threshold (384 entries), as the power-law graph
    has them at full size, inside whole iterations: the aggregation that carries the penalty term nu (Z_l - relu(T_l))
    of the Z gradient (Appendix A, Eqs. 3, 4) on split rows and its combine kernel, the low-rank form of the gradient,
    the segment products of the theta search and the carried pre-activations."""
    base = synth.make_workload("hub", 31, 2400, 5, [24, 32, 32, 8], 8, 6, graph="sbm", features="gaussian",
                               avg_degree=8, frac_intra=0.8)
    w = synth.add_hubs(base, 32, 3, 700, 0.65)
    deg = np.bincount(w.src, minlength=w.N) + np.bincount(w.dst, minlength=w.N)
    assert np.sort(deg)[-3] > 500
    # layer 1: C_2 >= C_1, so G_2 W_2^T is aggregated at width 32 with the penalty epilogue; layer 2: low-rank form
    run_case(w, 6, "hubs/epilogue-aggregation+low-rank", tune={"use_lowrank": 2})
    # widths that are no multiple of four (one column per lane) through the same path
    base = synth.make_workload("hub", 33, 2000, 4, [20, 30, 30, 5], 5, 6, graph="sbm", features="gaussian",
                               avg_degree=8, frac_intra=0.8)
    run_case(synth.add_hubs(base, 34, 2, 600, 0.7), 5, "hubs/odd-widths")
    # an aggregated gradient of two column tiles, the second one with a partial last quad: the row sums come tile by tile from
    # the aggregation, and those of the split rows from the combine kernel, all in the first tile's place
    base = synth.make_workload("hub", 37, 1500, 4, [20, 261, 300, 5], 5, 4, graph="sbm", features="gaussian",
                               avg_degree=8, frac_intra=0.8)
    run_case(synth.add_hubs(base, 38, 3, 600, 0.7), 3, "hubs/two-column-tiles")
    # two layers, narrow last layer: low-rank gradient and narrow-side association of layer 2 on hub rows
    base = synth.make_workload("hub", 35, 2400, 6, [24, 40, 8], 8, 6, graph="dcsbm", features="gaussian",
                               avg_degree=10, frac_intra=0.8, exponent=2.5)
    w = synth.add_hubs(base, 36, 3, 650, 0.7)
    run_case(w, 6, "hubs/low-rank-two-layers", tune={"use_lowrank": 2})
    run_case(w, 5, "hubs/stored-gradient-two-layers", tune=dict(use_lowrank=0))


def test_carried_pre_activations_across_their_refresh():
    """T_l = A~ Z_{l-1} W_l is carried from one iteration to the next by update formulas and formed anew every
    t1_refresh iterations: compare with the oracle at every age, across several refreshes, and over more than one
    full period of the default."""
    w = synth.config(1, 0.5)
    run_case(w, 11, "carry/config1/refresh4", tune=dict(t1_refresh=4))
    w = synth.config(3, 0.005)                       # three layers: T_2, T_3 carried through the Z steps
    run_case(w, 10, "carry/config3/refresh3", tune=dict(t1_refresh=3))
    w = synth.config(4, 0.002)                       # narrow-side association: the carried T_2 skips an aggregation
    run_case(w, 10, "carry/config4/refresh4", tune=dict(t1_refresh=4))
    w = synth.config(1)                              # default period of 16: ages 1..16, the refresh, and beyond
    run_case(w, 19, "carry/config1/default-period")
    w = synth.config(3, 0.005)
    run_case(w, 18, "carry/config3/default-period")


def test_last_layer_by_fista_with_backtracking():
    """fista_mode 1: Z_{L,m} by FISTA with backtracking on the block (one L per community and step, found on the device);
    iterates, the L every solve ends with and the number of candidates it tested must match the oracle."""
    w = synth.config(1, 0.5)
    w.hyper["fista_mode"] = 1
    run_case(w, 8, "fista-backtracking/config1")
    w = synth.config(3, 0.005)                       # three layers, ten classes
    w.hyper["fista_mode"] = 1
    run_case(w, 6, "fista-backtracking/config3")
    w = synth.make_workload("ragged", 11, 1237, 5, [37, 50, 9, 6], 6, 6, graph="sbm", features="gaussian",
                            avg_degree=6, frac_intra=0.7, labelled_fraction=0.4)
    w.comm = np.where(w.comm == 3, 4, w.comm).astype(np.int32)      # community 3 is empty; most rows have no label
    w.hyper["fista_mode"] = 1
    run_case(w, 5, "fista-backtracking/ragged-ce")
    w2 = copy.deepcopy(w)
    w2.hyper["risk"] = 1
    w2.hyper["dual_form"] = 1
    run_case(w2, 4, "fista-backtracking/ragged-lsq/dual-form-1")
    w = synth.config(4, 0.002)                       # 16 classes, 64 communities
    w.hyper["fista_mode"] = 1
    run_case(w, 4, "fista-backtracking/config4")
    # a cap on the multiplications that binds: L cannot reach the curvature, both sides must raise the status bit (the
    # solve then overshoots and the iteration amplifies rounding within a few iterations, so only two are compared)
    w.hyper["max_backtrack"] = 6
    run_case(w, 2, "fista-backtracking/config4/cap")
    w = synth.make_workload("wide-last", 41, 900, 3, [20, 24, 40], 40, 4, graph="sbm", features="gaussian",
                            avg_degree=8, frac_intra=0.8)   # 40 classes: sixteen lanes per row
    w.hyper["fista_mode"] = 1
    w.hyper["schedule"] = 1
    run_case(w, 4, "fista-backtracking/40-classes/layer-by-layer")
    # from 300000 entries of Z_L on a step starts with one candidate, and four more follow where it fails
    w = copies(synth.make_workload("many-rows", 42, 101, 3, [12, 16, 10], 10, 4, graph="sbm", features="gaussian", avg_degree=8,
                                   frac_intra=0.7), 300)
    w.hyper["fista_mode"] = 1
    run_case(w, 4, "fista-backtracking/many-rows")


def test_more_communities_than_a_workgroup_keeps_step_parameters_for():
    """The Z-step and carry kernels keep 1/theta of up to 1024 communities in LDS and look the parameters up in memory
    beyond that: 1100 communities of a few nodes each, on the low-rank path (two layers) and on the stored-gradient
    path (three layers)."""
    run_case(synth.config(4, 0.002, M=1100), 3, "many-communities/config4", tune={"use_lowrank": 2})       # N = 4000
    run_case(synth.config(3, 0.008, M=1100), 3, "many-communities/config3")       # N = 1600, three layers


def test_communities_from_the_library_partitioner_feed_the_sweep():
    """A graph that comes without communities: cadmm_partition (bit-exact against its CPU twin) supplies them, the graph
    built from them is bit-exact against the oracle's, and the sweep on them matches the oracle iteration by iteration."""
    from oracle.graph import OracleGraph
    from oracle.partition import partition as twin_partition
    from paper_2112_09335_amd import binding
    w = synth.config(2, 0.1)                          # N = 2000, planted blocks thrown away
    host = binding.Solver(device=-1)
    comm = host.partition(w.N, w.src, w.dst, w.M)
    host.close()
    assert np.array_equal(comm, np.asarray(twin_partition(w.N, w.src, w.dst, w.M), dtype=np.int32))
    assert comm.min() >= 0 and comm.max() < w.M and not np.array_equal(comm, w.comm)
    w.comm = comm
    s = binding.Solver.from_workload(w, 0)
    g = s.get_graph()
    og = OracleGraph(w.N, w.src, w.dst, w.M, w.comm)
    assert np.array_equal(g["perm"], og.perm) and np.array_equal(g["row_ptr"], og.row_ptr)
    assert np.array_equal(g["col"], og.col) and np.array_equal(g["val"], og.val.astype(np.float32))
    assert np.array_equal(g["seg_ptr"], og.seg_ptr) and np.array_equal(g["seg_comm"], og.seg_comm)
    assert np.array_equal(g["neighbour"], og.neighbour)
    s.close()
    run_case(w, 6, "library-partitioner/config2")
