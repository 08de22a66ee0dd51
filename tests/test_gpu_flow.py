"""Plans whose step is one launch with both passes of every tensor in it: the same sets through the launches by phases
(LPMM_FLOW=0) and through the one launch (LPMM_FLOW_MIN=0: small sets, too), with the tiles of the second pass waiting for
the first one, and with every tile of it deferred to the tensor's last workgroup (LPMM_FLOW_SPIN=-1: no poll at all).
The rank-1 results are the same bits on every route; the factorized statistics are sums in another order (tolerance: see
test_gpu_factor)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2309_01507_amd as lpmm
import workloads
from gpu_util import DEV, PARAM_ATOL, PARAM_RTOL, to_dev
from test_gpu_factor import STAT_RTOL
from test_gpu_multi import _mini_transformer, _run_set

pytestmark = pytest.mark.gpu
HP = oracle.Hyper()
ROUTE = ("LPMM_FLOW", "LPMM_FLOW_MIN", "LPMM_FLOW_SPIN", "LPMM_MULTI_STREAMS", "LPMM_PHASE_MPARAMS", "LPMM_FORCE_GENERAL")
PHASES = {"LPMM_FLOW": "0"}
ONE = {"LPMM_FLOW_MIN": "0"}
DEFERRED = {"LPMM_FLOW_MIN": "0", "LPMM_FLOW_SPIN": "-1"}

# every kind of tile: whole blocks, rows that are no multiple of 128, narrow ones, one workgroup and many, a wide one
RANK1 = [("rank1", (300, 512)), ("rank1", (130, 4224)), ("rank1", (37, 200)), ("rank1", (1030, 129)), ("rank1", (40, 96)),
         ("rank1", (1, 5000)), ("rank1", (257, 1023)), ("offset", (70, 1280)), ("nd", (24, 16, 3, 3)), ("nd", (8, 1, 2, 128)),
         ("nd", (5, 3, 1024)), ("b128", (1, 70001)), ("fp32", (1, 3000)), ("rank1", (2050, 640))]
FACTOR = [("factor", (300, 512)), ("factor", (37, 100)), ("factor", (1, 6400)), ("factor", (1030, 640)), ("fp32", (1, 768)),
          ("b128", (1, 8192)), ("factor", (2057, 127))]
RAGGED_FACTOR = [("factor", (300, 512)), ("factor", (37, 200))]       # ragged factorized matrices: by phases


def _steps(monkeypatch, env, tensors, bf16, steps=3, capture=False, one_launch=None):
    """`steps` steps of one plan; all parameters and states, as arrays.  one_launch: the route that the plan has to take,
    by default the one that the environment asks for."""
    for k in ROUTE:
        monkeypatch.delenv(k, raising=False)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    lpmm.ensure_init(8192)
    ws, gs, states, descs = [], [], [], []
    for tid, (kind, shape) in enumerate(tensors):
        rows, cols = shape[0], int(np.prod(shape[1:]))
        w = to_dev(workloads.weights(81, tid, rows, cols).reshape(-1))
        g = torch.empty(rows * cols, dtype=torch.bfloat16 if bf16 else torch.float32, device=DEV)
        if kind == "nd":
            st = lpmm.new_state_nd(shape, DEV)
        elif kind == "b128":
            st = lpmm.new_state_b128(cols, DEV)
        elif kind == "factor":
            st = lpmm.new_state_factor(rows, cols, DEV)
        elif kind == "fp32":
            st = (torch.zeros(cols, device=DEV), torch.zeros(cols, device=DEV))
        else:
            st = lpmm.new_state(rows, cols, DEV)
            if kind == "offset":                    # column maxima off the 16-byte grid: no whole-block tiles
                st.v_colmax = torch.zeros(cols + 4, device=DEV)[1:cols + 1]
        descs.append(lpmm.make_desc(w, g, st, rows, cols) if kind == "fp32" else lpmm.make_desc(w, g, st))
        ws.append(w)
        gs.append(g)
        states.append(st)
    plan = lpmm.new_plan(descs, 1 if bf16 else 0, DEV)
    assert (lpmm.lpmm_adamw4_plan_launches(plan) == 1) == (env is not PHASES if one_launch is None else one_launch)
    lr, step = torch.full((1,), HP.lr, device=DEV), torch.zeros(1, dtype=torch.int64, device=DEV)

    def one():
        lpmm.lpmm_adamw4_step_multi_capturable(plan, lr, step, HP.beta1, HP.beta2, HP.eps, HP.weight_decay)

    graph = None
    if capture:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            one()
    for t in range(1, steps + 1):
        for tid, ((kind, shape), g) in enumerate(zip(tensors, gs)):
            x = workloads.grads(81, tid, t, shape[0], int(np.prod(shape[1:])), "outlier_sparse" if tid % 3 == 2 and shape[0] > 1
                                else "col_lognormal", bf16)
            g.copy_(to_dev(x.reshape(-1), bf16))
        step.fill_(t)
        graph.replay() if capture else one()
        torch.cuda.synchronize()
    lpmm.lpmm_adamw4_plan_release(plan)
    out = []
    for w, st in zip(ws, states):
        parts = list(st) if isinstance(st, tuple) else [v for v in vars(st).values() if torch.is_tensor(v)]
        out.append([w.cpu().numpy()] + [v.cpu().numpy() for v in parts])
    return out


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("env", [ONE, DEFERRED], ids=["waiting", "deferred"])
def test_the_oracle_step_by_step(monkeypatch, env, bf16):
    for k in ROUTE:
        monkeypatch.delenv(k, raising=False)
    launches, release = [], lpmm.lpmm_adamw4_plan_release
    monkeypatch.setattr(lpmm, "lpmm_adamw4_plan_release",
                        lambda plan: (launches.append(lpmm.lpmm_adamw4_plan_launches(plan)), release(plan)))
    _run_set(_mini_transformer(), "col_lognormal", bf16, steps=3, seed=82, env=env)
    assert launches == [1]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("env,capture", [(ONE, False), (DEFERRED, False), (ONE, True)], ids=["waiting", "deferred", "graph"])
def test_same_bits_as_the_launches_by_phases(monkeypatch, env, capture, bf16):
    want = _steps(monkeypatch, PHASES, RANK1, bf16)
    got = _steps(monkeypatch, env, RANK1, bf16, capture=capture)
    for (kind, shape), a, b in zip(RANK1, want, got):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y, err_msg=f"{kind} {shape}")


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("env,capture,tensors", [(ONE, False, FACTOR), (DEFERRED, False, FACTOR), (ONE, True, FACTOR),
                                                 (ONE, True, RAGGED_FACTOR)], ids=["waiting", "deferred", "graph", "ragged"])
def test_factorized(monkeypatch, env, capture, tensors, bf16):
    """With a ragged matrix in the set the plan keeps the launches by phases (see flow_possible), here from a graph."""
    want = _steps(monkeypatch, PHASES, tensors, bf16)
    got = _steps(monkeypatch, env, tensors, bf16, capture=capture, one_launch=tensors is FACTOR)
    for (kind, shape), a, b in zip(tensors, want, got):
        np.testing.assert_allclose(b[0], a[0], rtol=PARAM_RTOL, atol=PARAM_ATOL, err_msg=f"{kind} {shape}")
        for x, y in zip(a[1:], b[1:]):
            if x.dtype == np.uint8 or kind != "factor" or x.size not in shape:      # first moment: nothing of it is a sum
                np.testing.assert_array_equal(x, y, err_msg=f"{kind} {shape}")
            else:
                np.testing.assert_allclose(y, x, rtol=STAT_RTOL, atol=0, err_msg=f"{kind} {shape}")


def test_statistics_beyond_one_workgroup_keep_the_phases(monkeypatch):
    """Inner dimensions with more statistics than the one launch has room for: the plan is stepped by phases."""
    tensors = [("nd", (4, 2400, 2)), ("rank1", (64, 256))]
    want = _steps(monkeypatch, PHASES, tensors, False)
    got = _steps(monkeypatch, ONE, tensors, False, one_launch=False)
    for a, b in zip(want, got):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("rows,n_first", [(40, "fewer than"), (1024, "as many as"), (1056, "one more than"), (9000, "many more than")])
def test_counts_of_finished_workgroups(monkeypatch, rows, n_first):
    """First passes of fewer workgroups than the counters of the first level (32), as many, one more and many more, with
    the tiles of the second pass waiting: the last one in is the one that lets the second pass go on, step after step.
    (32 rows to a tile of the first pass in a set this small, one strip.)"""
    tensors = [("rank1", (rows, 128)), ("rank1", (64, 256))]
    want = _steps(monkeypatch, PHASES, tensors, True, steps=4)
    got = _steps(monkeypatch, ONE, tensors, True, steps=4)
    for a, b in zip(want, got):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y, err_msg=n_first)


@pytest.mark.parametrize("bf16", [False, True])
def test_deferred_by_the_workgroup_with_the_last_ticket(monkeypatch, bf16):
    """Tensors of one or two update tiles: the workgroup that defers a tile takes the tensor's last ticket, too, and so
    writes the word again from which its waves have just read that the tile is deferred."""
    tensors = [("rank1", (8, 128)), ("rank1", (8, 256)), ("rank1", (3, 128)), ("rank1", (5, 130)), ("rank1", (20, 96)),
               ("rank1", (24, 128))] * 8
    want = _steps(monkeypatch, PHASES, tensors, bf16)
    got = _steps(monkeypatch, DEFERRED, tensors, bf16)
    for (kind, shape), a, b in zip(tensors, want, got):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y, err_msg=f"{kind} {shape}")


@pytest.mark.parametrize("env", [{}, {"LPMM_FLOW_SPIN": "-1"}], ids=["waiting", "deferred"])
def test_updates_of_convolutions_at_the_end(monkeypatch, env):
    """A set between 12.6 and 33.5 million parameters: all updates but the convolutions' come first, ragged tiles are of middle
    height."""
    tensors = [("nd", (512, 256, 3, 3)), ("rank1", (2944, 2944)), ("nd", (736, 368, 3, 3)), ("rank1", (1000, 1472)), ("fp32", (1, 736)),
               ("nd", (16, 3, 7, 7))]
    want = _steps(monkeypatch, PHASES, tensors, False, steps=2)
    got = _steps(monkeypatch, env, tensors, False, steps=2)
    for (kind, shape), a, b in zip(tensors, want, got):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y, err_msg=f"{kind} {shape}")


@pytest.mark.parametrize("kind,shape", [("rank1", (300, 512)), ("rank1", (257, 1023)), ("rank1", (300, 96)), ("nd", (24, 16, 3, 3)),
                                        ("factor", (300, 512)), ("factor", (300, 96)), ("rank1", (8192, 2048)),
                                        ("rank1", (16000, 1000)), ("factor", (8192, 2048))])
@pytest.mark.parametrize("spin,deferred", [("-1", True), ("20000", False)])
def test_which_tiles_are_deferred(monkeypatch, kind, shape, spin, deferred):
    """LPMM_FLOW_SPIN=-1 defers every tile of the second pass: the plan's list of them, zeros when it is built and not cleared by a
    step, holds every number of a workgroup of that pass once afterwards (0 cannot be told from an empty place), and the rest
    of the plan's workspace is zeros again.  (In the large ones most of the second pass begins when the first has ended.)  With polls a second pass that waits is not deferred."""
    for k in ROUTE:
        monkeypatch.delenv(k, raising=False)
    monkeypatch.setenv("LPMM_FLOW_MIN", "0")
    monkeypatch.setenv("LPMM_FLOW_SPIN", spin)
    lpmm.ensure_init(8192)
    rows, cols = shape[0], int(np.prod(shape[1:]))
    w, g = torch.zeros(rows * cols, device=DEV), torch.ones(rows * cols, device=DEV)
    st = {"rank1": lambda: lpmm.new_state(rows, cols, DEV), "nd": lambda: lpmm.new_state_nd(shape, DEV),
          "factor": lambda: lpmm.new_state_factor(rows, cols, DEV)}[kind]()
    plan = lpmm.new_plan([lpmm.make_desc(w, g, st)], 0, DEV)
    assert lpmm.lpmm_adamw4_plan_launches(plan) == 1
    words = plan[:plan.numel() // 4 * 4].view(torch.int32)
    before = words.clone()
    lpmm.lpmm_adamw4_step_multi(plan, HP.lr, HP.beta1, HP.beta2, HP.eps, HP.weight_decay, 1)
    torch.cuda.synchronize()
    listed = sorted(words[words != before].tolist())
    lpmm.lpmm_adamw4_plan_release(plan)
    least = rows * cols // (16 * 1024)                    # no update tile of such a set has more elements
    assert listed == list(range(1, len(listed) + 1)) and (len(listed) + 1 >= max(2, least) if deferred else not listed)


def test_launches_of_a_step(monkeypatch):
    """The host's count of a step's kernels on every route: both passes of one group, with two kernels between them for
    tensors of more than two dimensions; groups on two streams, one after the other and fused; and no plan at all."""
    lpmm.ensure_init(8192)
    keep = []

    def launches(tensors, **env):
        for k in ROUTE:
            monkeypatch.delenv(k, raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        descs = []
        for kind, shape in tensors:
            n = int(np.prod(shape))
            w, g = torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
            st = {"nd": lambda: lpmm.new_state_nd(shape, DEV), "b128": lambda: lpmm.new_state_b128(n, DEV),
                  "rank1": lambda: lpmm.new_state(*shape, DEV), "sgdm": lambda: lpmm.new_state_sgdm(n, DEV)}[kind]()
            keep.append((w, g, st))
            descs.append(lpmm.make_desc_sgdm(w, g, st) if kind == "sgdm" else lpmm.make_desc(w, g, st))
        plan = lpmm.new_plan(descs, 0, DEV)
        n = lpmm.lpmm_adamw4_plan_launches(plan)
        lpmm.lpmm_adamw4_plan_release(plan)
        with pytest.raises(lpmm.LpmmError):
            lpmm.lpmm_adamw4_plan_launches(plan)
        return n

    two, nd = [("rank1", (1024, 1024)), ("rank1", (1024, 512))], [("nd", (16, 16, 3, 3))]
    assert launches(two) == 2 and launches(two, LPMM_FLOW_MIN="0") == 1
    assert launches(nd) == 1 and launches(nd, LPMM_FLOW="0") == 4
    assert launches([("b128", (1, 5000))]) == 1 and launches([("sgdm", (1, 5000))]) == 1
    groups = {"LPMM_PHASE_MPARAMS": "1"}
    assert launches(two, **groups) == 4 and launches(two, LPMM_MULTI_STREAMS="0", **groups) == 4
    assert launches(two, LPMM_MULTI_STREAMS="1", **groups) == 3


def test_memory_without_a_work_list(monkeypatch):
    """A plan built into memory that was sized with the one launch switched off: by phases, the same bits."""
    tensors = [("rank1", (300, 512)), ("nd", (24, 16, 3, 3)), ("rank1", (37, 200))]
    want = _steps(monkeypatch, PHASES, tensors, False)
    sized = lpmm.binding.lpmm_adamw4_plan_bytes

    def without(descs):
        with monkeypatch.context() as m:
            m.setenv("LPMM_FLOW", "0")
            return sized(descs)

    monkeypatch.setattr(lpmm.binding, "lpmm_adamw4_plan_bytes", without)
    got = _steps(monkeypatch, ONE, tensors, False, one_launch=False)
    for a, b in zip(want, got):
        for x, y in zip(a, b):
            np.testing.assert_array_equal(x, y)
