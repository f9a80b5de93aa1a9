"""Calls that return results to the host are refused while the context's
stream is being captured: nothing is recorded, and nothing that the context
would have noted as done (uploaded descriptors, tables, zeroed buffers) makes
a later call read what never ran."""
import ctypes as C

import numpy as np
import pytest

from paper_1505_00965_amd import mlmc, workloads as W

pytestmark = pytest.mark.gpu

GM, HM = W.GBM_MODEL, W.HESTON_MODEL


def calls(ctx):
    """(name, call returning plain numbers) of every kind, and the networks that they use."""
    gm, hm, mil = mlmc.model(**GM), mlmc.model(**HM), mlmc.model(**dict(GM), scheme=1)
    pay = {k: mlmc.payoff(**v) for k, v in W.PAYOFFS.items()}
    r = np.random.default_rng(4)

    def net(d, tab):
        cv = mlmc.ControlVariate(ctx, d)
        cv.set_params(r.uniform(-0.2, 0.2, cv.nparams).astype(np.float32))
        cv.set_tabulated(tab)
        return cv

    nets = {(d, tab): net(d, tab) for d in (2, 3) for tab in (False, True)}
    sums = lambda x: [x["sum_y"], x["sum_y2"], x["n"]]
    run = lambda x: [x["estimate"]] + x["N"]
    return nets.values(), [
        ("level", lambda: sums(ctx.mlmc_level(gm, pay["call"], 3, 4, 5000, 7))),
        ("level, network", lambda: sums(ctx.mlmc_level(gm, pay["call"], 0, 4, 5000, 7, cv=nets[2, False]))),
        ("level, table", lambda: sums(ctx.mlmc_level(hm, pay["asian"], 2, 4, 5000, 7, cv=nets[3, True]))),
        ("stdmc", lambda: sums(ctx.mlmc_stdmc(hm, pay["asian"], 2, 2, 5000, 7))),
        ("batch", lambda: sum((sums(x) for x in ctx.mlmc_levels_batch(gm, [pay["asian"]], 4, 2, [[700, 80, 9]], 5)[0]), [])),
        ("randomised", lambda: [ctx.mlmc_rhee_glynn(mil, pay["call"], 4, 4, 0.125, 9001, 3)["estimate"]]),
        ("randomised fp64", lambda: [ctx.mlmc_rhee_glynn(mil, pay["call"], 4, 3, 0.125, 901, 3, precision=64)["estimate"]]),
        ("run", lambda: run(ctx.mlmc_run(gm, pay["call"], 0.3, seed=3, n_pilot=2000))),
        ("run planned", lambda: run(ctx.mlmc_run(gm, pay["call"], 0.3, seed=3, n_pilot=2000, persistent=True))),
        ("run, table", lambda: run(ctx.mlmc_run(gm, pay["call"], 0.3, seed=3, n_pilot=2000, persistent=True,
                                                cv=nets[2, True]))),
        ("counts", lambda: list(ctx.mlmc_optimal_n([1.0, 0.1], [1.0, 5.0], 0.01))),
        ("gradient", lambda: [nets[2, False].loss_grad(gm, pay["call"], 4, 1, 100, 3, 2)[0]]),
        ("training", lambda: list(nets[3, False].train(hm, pay["call"], 4, 1, 2, 100))),
    ]


# each as its context's first call
@pytest.mark.parametrize("k", range(13))
def test_refused_and_without_effect(k):
    import torch
    path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
    hip = C.CDLL(path)
    s = torch.cuda.Stream()
    st, graph, status = C.c_void_p(s.cuda_stream), C.c_void_p(), C.c_int(-1)
    with mlmc.Context(0) as ref_ctx, mlmc.Context(0) as ctx:
        ref_nets, ref_calls = calls(ref_ctx)
        name, ref_call = ref_calls[k]
        print("case", name, flush=True)
        ref = ref_call()
        nets, own = calls(ctx)
        call = own[k][1]
        ctx.set_stream(s)
        assert hip.hipStreamBeginCapture(st, 2) == 0            # relaxed
        with pytest.raises(mlmc.MLMCError) as e:
            call()
        assert e.value.status == mlmc.MLMC_EDEVICE and "captured" in str(e.value)
        assert hip.hipStreamIsCapturing(st, C.byref(status)) == 0 and status.value == 1   # unharmed
        assert hip.hipStreamEndCapture(st, C.byref(graph)) == 0
        n = C.c_size_t(99)
        assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0 and n.value == 0
        hip.hipGraphDestroy(graph)
        got = call()
        # the same samples: sums in another order of their additions (training
        # returns fp32 losses)
        assert np.allclose(got, ref, rtol=1e-6 if name == "training" else 1e-10, atol=0)
        ctx.set_stream(None)
        for cv in (*ref_nets, *nets):
            cv.close()
