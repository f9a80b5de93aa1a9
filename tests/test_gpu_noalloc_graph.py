"""mlmc_level_noalloc captured into graphs: replays between eager calls, and
sums that a failed call left in the static records.

Such sums are made by a captured call whose last launch (the fold, which reads
and clears the records) is taken out of its graph: the replay stands for a
call whose level launches were enqueued and whose fold was not."""
import ctypes as C

import pytest

from paper_1505_00965_amd import mlmc, workloads as W

pytestmark = pytest.mark.gpu

# level, M, N, precision: one launch a call but the last, whose samples lie on
# both sides of 2^32 (a launch each)
CASES = [(2, 4, 20000, 32, 0), (5, 4, 331, 32, 0), (3, 4, 1000, 64, 0), (2, 4, 5000, 32, (1 << 32) - 1700)]
SEED, THREAD_LOCAL, RELAXED = 5, 1, 2


class Runtime:
    """The HIP calls that torch does not expose, on the runtime it has loaded."""

    def __init__(self):
        path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
        self.lib = C.CDLL(path)

    def __call__(self, name, *args):
        e = getattr(self.lib, name)(*args)
        assert e == 0, (name, e)


class Graph:
    """A captured call; without_fold: its last node taken out."""

    def __init__(self, hip, stream, call, without_fold=False):
        self.hip, self.stream = hip, C.c_void_p(stream.cuda_stream)
        self.graph, self.exec = C.c_void_p(), C.c_void_p()
        hip("hipStreamBeginCapture", self.stream, RELAXED)
        call()
        hip("hipStreamEndCapture", self.stream, C.byref(self.graph))
        if without_fold:
            n = C.c_size_t(0)
            hip("hipGraphGetNodes", self.graph, None, C.byref(n))
            nodes = (C.c_void_p * n.value)()
            hip("hipGraphGetNodes", self.graph, nodes, C.byref(n))
            last = []
            for node in nodes:
                k = C.c_size_t(0)
                hip("hipGraphNodeGetDependentNodes", C.c_void_p(node), None, C.byref(k))
                if k.value == 0:
                    last.append(node)
            assert len(last) == 1 and n.value >= 2      # a chain of launches
            hip("hipGraphDestroyNode", C.c_void_p(last[0]))
        hip("hipGraphInstantiate", C.byref(self.exec), self.graph, None, None, C.c_size_t(0))

    def replay(self):
        self.hip("hipGraphLaunch", self.exec, self.stream)

    def close(self):
        self.hip("hipGraphExecDestroy", self.exec)
        self.hip("hipGraphDestroy", self.graph)


class Bench:
    def __init__(self, case):
        import torch
        l, M, N, prec, off = case
        self.hip, self.stream = Runtime(), torch.cuda.Stream()
        self.out = torch.zeros(9, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()                # the fill runs on another stream
        gm, gp = mlmc.model(**W.GBM_MODEL), mlmc.payoff(**W.ASIAN)
        self.call = lambda: mlmc.mlmc_level_noalloc(gm, gp, l, M, N, SEED, self.out, path_offset=off,
                                                    precision=prec, stream=self.stream)
        self.other = lambda: mlmc.mlmc_level_noalloc(gm, gp, 1, M, 777, SEED, self.out, stream=self.stream)

    def read(self):
        self.stream.synchronize()
        return mlmc.level_result_from(self.out)

    def eager(self):
        self.call()
        return self.read()


def same(a, b):
    # the same samples, added into the records in another order
    assert a["n"] == b["n"] and a["n_nonfinite"] == b["n_nonfinite"]
    for k, k2 in (("sum_y", "sum_y2"), ("sum_pf", "sum_pf2"), ("sum_pc", "sum_pc2")):
        assert abs(a[k] - b[k]) <= 1e-12 * (b["n"] * b[k2]) ** 0.5, (k, a[k], b[k])
        assert abs(a[k2] - b[k2]) <= 1e-12 * b[k2], (k2, a[k2], b[k2])


@pytest.mark.parametrize("case", CASES)
def test_replays_between_eager_calls(case):
    b = Bench(case)
    ref = b.eager()
    g = Graph(b.hip, b.stream, b.call)
    for _ in range(3):
        g.replay()
        same(b.read(), ref)
        b.other()                               # eager, of another size
        g.replay()
        g.replay()
        same(b.read(), ref)
        same(b.eager(), ref)
    g.close()


@pytest.mark.parametrize("case", CASES)
def test_replay_after_a_call_that_failed_midway(case):
    b = Bench(case)
    ref = b.eager()
    full, cut = Graph(b.hip, b.stream, b.call), Graph(b.hip, b.stream, b.call, without_fold=True)
    for _ in range(2):
        cut.replay()                            # sums left in the records
        full.replay()
        same(b.read(), ref)
    same(b.eager(), ref)
    full.close()
    cut.close()


def test_captured_call_does_not_settle_an_earlier_failure():
    b = Bench(CASES[0])
    ref = b.eager()
    cut = Graph(b.hip, b.stream, b.call, without_fold=True)
    # a call on a stream whose capture has been broken fails
    st, graph = C.c_void_p(b.stream.cuda_stream), C.c_void_p()
    b.hip("hipStreamBeginCapture", st, THREAD_LOCAL)
    assert b.hip.lib.hipStreamQuery(st) != 0    # not allowed in a capture: breaks it
    with pytest.raises(mlmc.MLMCError) as e:
        b.call()
    assert e.value.status == mlmc.MLMC_EDEVICE
    assert b.hip.lib.hipStreamEndCapture(st, C.byref(graph)) != 0 and not graph.value
    b.hip.lib.hipGetLastError()
    cut.replay()                                # the sums that such a call may leave
    never = Graph(b.hip, b.stream, b.call)      # captured, not replayed
    same(b.eager(), ref)
    same(b.eager(), ref)
    never.close()
    cut.close()
