"""What a user of this library has it do, as cases that can be timed.

A case names one kind of work and its sizes:

  train      a training run: initial weights, a number of ADMM iterations, then what a training program reads back
             (`every` > 0: the objective and the residuals are read after that many iterations, as a program that
             watches convergence does; `checkpoint`: the whole state is read at the end, as one that saves it does)
  predict    inference on a trained solver: classes, logits and accuracy of all nodes
  session    a whole program on host data: communities if it has none, graph, solver, data, training, inference
  aggregate  one product with the normalised adjacency on device data
  wgrad      one weight-gradient product on device data, through the entry point that allocates nothing

The graphs are stochastic block models in a scrambled node order (`powerlaw`: with node weights of exponent 2.5), the
features Gaussian or sparse binary, the labels follow the communities: the recipes of paper_2112_09335_amd/synth.py,
drawn on the GPU because they are drawn often.
"""
import numpy as np
import torch

from paper_2112_09335_amd import binding, synth

DEV = "cuda:0"
HYPER = ("dual_form", "schedule", "step_policy", "fista_mode", "risk")


def _net(N, M, dims, degree, intra, **more):
    return dict(N=N, M=M, dims="-".join(str(d) for d in dims), degree=degree, intra=intra, powerlaw=False, sparse=False,
                labelled=1.0, nu=1e-3, **{h: 0 for h in HYPER}, **more)


def listed():
    deep = [512] * 8 + [10]
    computers = [767, 1000, 10]
    return [
        # the smallest call: one product of a few thousand rows inside somebody else's loop; launches and host calls count
        dict(name="wgrad_small", kind="wgrad", n=2000, K=256, C=64),
        # features of a mid-sized graph propagated once, as a preprocessing step does; gather-bound
        dict(name="aggregate_wide", kind="aggregate", width=256, **_net(200000, 32, [256, 16], 15, 0.85)),
        # the smallest training run: every iteration is launch-bound
        dict(name="train_tiny", kind="train", iters=5, every=0, checkpoint=True, **dict(_net(2000, 4, [256, 64, 7], 12, 0.85), sparse=True)),
        # an ordinary one: twenty thousand nodes, three classes (ragged last layer), the state saved at the end
        dict(name="train_mid", kind="train", iters=5, every=0, checkpoint=True, **_net(20000, 8, [500, 128, 3], 10, 0.9)),
        # the shape of the paper's speed-up experiment (thousand hidden units, three communities), watched after every iteration
        dict(name="train_watched", kind="train", iters=5, every=1, checkpoint=False, **dict(_net(13752, 3, computers, 36, 0.9), sparse=True)),
        # the other options together: layer-by-layer schedule, shrinking steps, last layer by backtracking, dual step on
        # the new iterates, few labels, odd sizes, the state saved at the end
        dict(name="train_options", kind="train", iters=5, every=0, checkpoint=True,
             **dict(_net(30011, 7, [301, 97, 50, 6], 9, 0.8), labelled=0.4, dual_form=1, schedule=1, step_policy=1, fista_mode=1)),
        # three layers, two hundred thousand nodes
        dict(name="train_large", kind="train", iters=5, every=0, checkpoint=False, **_net(200000, 32, [128, 256, 256, 10], 15, 0.85)),
        # skewed degrees: hub rows, many (row, community) segments
        dict(name="train_powerlaw", kind="train", iters=5, every=0, checkpoint=False, **dict(_net(2000000, 64, [128, 256, 16], 25, 0.8), powerlaw=True)),
        # eight layers of 512 units: the largest, bound by the matrix cores
        dict(name="train_deep", kind="train", iters=5, every=0, checkpoint=False, **_net(500000, 16, deep, 12, 0.85)),
        # inference on the three-layer graph
        dict(name="predict_large", kind="predict", **_net(200000, 32, [128, 256, 256, 10], 15, 0.85)),
        # whole programs on host data: the paper's shape with its communities given, and a larger graph that has none
        dict(name="session_given", kind="session", iters=5, partition=False, **dict(_net(13752, 3, computers, 36, 0.9), sparse=True)),
        dict(name="session_partitioned", kind="session", iters=5, partition=True, **_net(200000, 32, [128, 256, 256, 10], 15, 0.85)),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "train", "predict", "session", "aggregate", "wgrad"])
    if kind == "wgrad":
        return dict(kind=kind, n=_log(rng, 500, 500000), K=_log(rng, 8, 512), C=_log(rng, 3, 512))
    M = _log(rng, 1, 64)
    N = max(_log(rng, 1000, 100000 if kind == "session" else 300000), 16 * M)
    degree = rng.randint(6, 30 if N < 100000 else 15)
    c = _net(N, M, [1], degree, round(rng.uniform(0.7, 0.95), 2))
    c["powerlaw"] = rng.random() < 0.35
    c["kind"] = kind
    if kind == "aggregate":
        c["width"] = _log(rng, 3, 512 if N < 100000 else 256)
        c["dims"] = "%d-%d" % (c["width"], 8)
        return c
    classes = rng.choice([3, 6, 7, 8, 10, 16, 40])
    layers = rng.choice([2, 2, 2, 3, 3, 4])
    top = 1024 if N < 20000 else 512 if N < 100000 else 256
    c["dims"] = "-".join(str(d) for d in [_log(rng, 32, top)] + [_log(rng, 16, top) for _ in range(layers - 1)] + [classes])
    c["sparse"] = rng.random() < 0.4
    c["labelled"] = rng.choice([1.0, 1.0, 0.3])
    c["nu"] = rng.choice([1e-3, 1e-3, 1e-4])
    for h in HYPER:
        c[h] = 1 if rng.random() < 0.15 else 0
    if kind == "train":
        c["iters"] = rng.randint(3, 5)
        c["every"] = rng.choice([0, 0, 1, 2])
        c["checkpoint"] = N < 50000 and rng.random() < 0.3
    elif kind == "session":
        c["iters"] = rng.randint(3, 5)
        c["partition"] = rng.random() < 0.5
    return c


def _dims(case):
    return [int(d) for d in case["dims"].split("-")]


def _graph(case, g):
    """(src, dst, comm) on the host: endpoint pairs inside a community with probability `intra`, else across two; repeats
    and self pairs stay in, as a file of edges has them."""
    N, M = case["N"], case["M"]
    E = N * case["degree"] // 2
    bounds = (torch.arange(M + 1, device=DEV) * N) // M
    c1 = (torch.rand(E, generator=g, device=DEV, dtype=torch.float64) * M).long().clamp_(max=M - 1)
    other = (c1 + 1 + (torch.rand(E, generator=g, device=DEV, dtype=torch.float64) * (M - 1)).long()) % M
    c2 = torch.where(torch.rand(E, generator=g, device=DEV) < case["intra"], c1, other)
    cum = None
    if case["powerlaw"]:
        w = (1.0 - torch.rand(N, generator=g, device=DEV, dtype=torch.float64)) ** (-1.0 / 1.5)
        w = w.clamp_(max=float(N * case["degree"]) ** 0.5).cpu().numpy()
        cum = torch.from_numpy(np.concatenate([[0.0], np.cumsum(w)])).to(DEV)

    def ends(c):
        lo, hi = bounds[c], bounds[c + 1]
        u = torch.rand(E, generator=g, device=DEV, dtype=torch.float64)
        if cum is None:
            return torch.minimum(lo + (u * (hi - lo)).long(), hi - 1)
        at = torch.searchsorted(cum, cum[lo] + u * (cum[hi] - cum[lo]), right=True) - 1
        return torch.minimum(torch.maximum(at, lo), hi - 1)

    a, b = ends(c1), ends(c2)
    name = torch.randperm(N, generator=g, device=DEV).int()
    comm = torch.empty(N, dtype=torch.int32, device=DEV)
    comm[name.long()] = torch.repeat_interleave(torch.arange(M, dtype=torch.int32, device=DEV), bounds[1:] - bounds[:-1])
    return name[a].cpu().numpy(), name[b].cpu().numpy(), comm.cpu().numpy()


def _workload(case, g):
    src, dst, comm = _graph(case, g)
    N, dims = case["N"], _dims(case)
    if case["sparse"]:
        X = (torch.rand((N, dims[0]), generator=g, device=DEV) < 0.01).float().cpu().numpy()
    else:
        X = torch.randn((N, dims[0]), generator=g, device=DEV).cpu().numpy()
    u = torch.rand((3, N), generator=g, device=DEV).cpu().numpy()
    home = comm % dims[-1]
    far = (home + 1 + (u[1] * (dims[-1] - 1)).astype(np.int32)) % dims[-1]
    labels = np.where(u[2] < case["labelled"], np.where(u[0] < 0.8, home, far), -1).astype(np.int32)
    W0 = [((torch.rand((dims[l - 1], dims[l]), generator=g, device=DEV) * 2 - 1) * (6.0 / (dims[l - 1] + dims[l])) ** 0.5).cpu().numpy()
          for l in range(1, len(dims))]
    hyper = dict(synth.DEFAULT_HYPER, nu=case["nu"], rho=case["nu"], **{h: case[h] for h in HYPER})
    return synth.Workload("case", N, case["M"], src, dst, comm, X, labels, dims, W0, case.get("iters", 0), hyper)


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    kind = case["kind"]
    if kind == "wgrad":
        A = torch.randn((case["n"], case["K"]), generator=g, device=DEV)
        G = torch.randn((case["n"], case["C"]), generator=g, device=DEV) * 1e-3
        out = torch.empty((case["K"], case["C"]), device=DEV)
        return dict(case=case, solver=binding.Solver(0), A=A, G=G, out=out)
    if kind == "aggregate":
        src, dst, comm = _graph(case, g)
        s = binding.Solver(0)
        s.build_graph(case["N"], src, dst, case["M"], comm)
        h = synth.DEFAULT_HYPER
        s.set_model([case["width"], 8, 8], **h)
        s.set_workspace()
        return dict(case=case, solver=s, X=torch.randn((case["N"], case["width"]), generator=g, device=DEV))
    w = _workload(case, g)
    if kind == "session":
        return dict(case=case, w=w)
    s = binding.Solver.from_workload(w, 0)
    w.X = w.src = w.dst = None                      # the solver has its own copies
    if kind == "predict":
        s.run(3)
    return dict(case=case, w=w, solver=s)


def _numbers(e):
    return {k: (e[k] if k != "layer_penalty" else np.asarray(e[k])) for k in
            ("objective", "lagrangian", "risk", "primal_res", "dual_res", "layer_penalty", "iter", "status")}


def _train(s, w, case):
    """The iterations, and the readouts of a program that watches them."""
    every, seen = case.get("every", 0), []
    if every:
        for k in range(0, case["iters"], every):
            s.run(min(every, case["iters"] - k))
            seen.append(s.eval())
    else:
        s.run(case["iters"])
    out = dict(stats=_numbers(s.eval()), W=[s.get_W(l) for l in range(1, w.L + 1)])
    if seen:
        out["objectives"] = np.array([e["objective"] for e in seen])
    return out


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "wgrad":
        return state["solver"].op_wgrad_noalloc(state["A"], state["G"], state["out"])
    if kind == "aggregate":
        return state["solver"].op_aggregate(state["X"])
    if kind == "predict":
        classes, logits, accuracy = state["solver"].predict()
        return dict(classes=classes, logits=logits, accuracy=accuracy)
    w = state["w"]
    if kind == "session":
        s = binding.Solver(0)
        h = w.hyper
        comm = s.partition(w.N, w.src, w.dst, w.M) if case["partition"] else w.comm
        s.build_graph(w.N, w.src, w.dst, w.M, comm)
        s.set_model(w.dims, **h)
        s.set_workspace()
        s.set_data(w.X, w.labels)
        s.init(w.W0)
        out = _train(s, w, case)
        out["classes"], out["logits"], out["accuracy"] = s.predict()
        out["comm"] = comm
        s.close()
        return out
    s = state["solver"]
    s.init(w.W0)
    out = _train(s, w, case)
    out["Z_last"], out["U"] = s.get_Z(w.L), s.get_U()
    if case["checkpoint"]:
        out["Z"] = [s.get_Z(l) for l in range(1, w.L)]
        out["tau"], out["theta"], _, _ = s.get_steps()
    return out


def work(case):
    """What one pass cannot do without: its inputs read once and its results written once; for a training run, in each
    iteration the graph and the first layer's input read and the state (Z, U) read and written.  Products: in every layer
    the weight gradient and the step's change of the pre-activation, in a hidden one also the gradient with respect to Z
    and the change of the next pre-activation, and the aggregations of the latter two."""
    kind = case["kind"]
    if kind == "wgrad":
        n, K, C = case["n"], case["K"], case["C"]
        return {"bytes": 4.0 * (n * K + n * C + K * C), "flops": 2.0 * n * K * C}
    N, dims = case["N"], _dims(case)
    nnz = float(N) * (case["degree"] + 1)
    if kind == "aggregate":
        return {"bytes": 8.0 * nnz + 8.0 * N * case["width"], "flops": 2.0 * nnz * case["width"]}
    weights = float(sum(a * b for a, b in zip(dims, dims[1:])))
    forward = 2.0 * N * weights + 2.0 * nnz * sum(min(a, b) for a, b in zip(dims, dims[1:]))
    if kind == "predict":
        return {"bytes": 8.0 * nnz + 4.0 * (N * (dims[0] + dims[-1] + 1) + weights), "flops": forward}
    hidden = float(sum(a * b for a, b in zip(dims[1:], dims[2:])))
    flops = 4.0 * N * weights + 4.0 * N * hidden + 4.0 * nnz * sum(min(a, b) for a, b in zip(dims[1:], dims[2:]))
    state = sum(dims[1:]) + dims[-1]
    bytes_ = 8.0 * nnz + 4.0 * N * (dims[0] + 2.0 * state) + 12.0 * weights
    once = 4.0 * N * dims[0] + 8.0 * nnz + 4.0 * N * dims[-1] + 4.0 * weights
    if kind == "session":
        once += 4.0 * N * case["degree"] + 4.0 * N * (dims[0] + 2)
        return {"bytes": once + case["iters"] * bytes_, "flops": 2.0 * forward + case["iters"] * flops}
    if case["checkpoint"]:
        once += 4.0 * N * state
    return {"bytes": once + case["iters"] * bytes_, "flops": forward + case["iters"] * flops}


def tolerance(case):
    """Products and sums of a single call are 32-bit ones.  A training run passes its rounding errors on: a pre-activation
    within rounding of zero may fall on either side of the ReLU (a few of 10^7 entries in an iteration do), which moves
    single entries of Z by percents of the root mean square, and every later iteration roughly doubles the distance.  Two
    correct runs are 1e-7 to 3e-4 apart after five iterations (32-bit products against three-way split 16-bit ones, 100
    graphs), which is also why the runs here are not longer.  Two nearly equal logits may change a class."""
    if case["kind"] in ("wgrad", "aggregate"):
        return {"rel": 1e-5}
    if case["kind"] == "predict":
        return {"rel": 1e-4, "differ": 1e-3}
    return {"rel": 1e-3, "max": 0.1, "differ": 1e-3}
