"""Captured batch iterations after something they baked in has changed: a
replay must give what the same calls give eagerly."""
import numpy as np
import pytest

from paper_2609_13115_amd import workloads, xls

pytestmark = pytest.mark.gpu


def boxes():
    return [workloads.small_dirichlet(ns=10, index=1, shape=(13, 9, 20), h=0.6),
            workloads.small_periodic(n=12, ns=8, index=3)]


# odd degrees keep the block's parity from one iteration to the next, so that
# every iteration after the first of a call has the key of a captured one
PARAMS = [xls.chefsi_params(d, 4, xls.XLS_BOUNDS_LANCZOS) for d in (7, 11)]


def results(b, use_graph):
    ritz, resid, iters, _ = b.xls_batch_chefsi(PARAMS, use_graph=use_graph)
    return ritz, resid, iters, [b.xls_batch_subdomain(i).xls_subdomain_get_block() for i in range(len(PARAMS))]


# One row and one plane a tile: more residual partial sums than any chosen
# shape, so the FP64 tune moves their buffer.  Then the first shape again, whose
# graph would write to the buffer that is gone.
@pytest.mark.parametrize("prec", [xls.XLS_PREC_FP32, xls.XLS_PREC_FP64])
def test_replay_after_retuning_the_fp64_sweep(prec):
    shapes = [(256, 0, 5, 1), (256, 1, 1, 1), (256, 0, 5, 1)]
    out = []
    for use_graph in (False, True):
        print(f"[case] replay after retune prec={prec} graph={use_graph}", flush=True)
        with xls.Batch(boxes(), filter_prec=prec) as b:
            runs = []
            for shape in shapes:
                for i in range(len(PARAMS)):
                    b.xls_batch_subdomain(i).xls_subdomain_tune(xls.XLS_PREC_FP64, *shape)
                runs.append(results(b, use_graph))
            out.append(runs)
            stats = b.xls_batch_stats()
    assert stats["captures"] == len(shapes) and stats["replays"] == 3 * len(shapes)
    for eager, graph in zip(*out):
        assert list(eager[2]) == list(graph[2])
        for x, y in zip(eager[0] + eager[1] + eager[3], graph[0] + graph[1] + graph[3]):
            assert np.array_equal(x, y)


# Slot residency releases every working set at the end of a call and allocates
# it anew in the next.  Other handles of the same sizes, made in between, take
# the released addresses: the next call's sets lie elsewhere, and what the first
# calls captured or tabled must not be run on them.
@pytest.mark.parametrize("use_graph", [False, True])
def test_slot_batch_whose_working_sets_moved(use_graph):
    print(f"[case] slots moved graph={use_graph}", flush=True)
    sds = boxes()
    with xls.Batch(sds) as b:
        ref = results(b, False)[:3]
    others, start = [], []
    with xls.Batch(sds, slots=0) as b:
        for n in range(4):
            ritz, resid, iters, _ = b.xls_batch_chefsi(PARAMS, use_graph=use_graph)
            assert list(iters) == list(ref[2])
            for x, y in zip(ritz + resid, ref[0] + ref[1]):
                assert np.array_equal(x, y)
            for s, X in zip(others, start):
                assert np.array_equal(s.xls_subdomain_get_block(), X)
            if n in (1, 2):
                others += [xls.Subdomain(sd) for sd in sds]
                start = [s.xls_subdomain_get_block() for s in others]
    for s in others:
        s.close()


# Four zeros give a tuned handle the shape back that it started with: the graph
# captured before the first tune serves it again.
def test_tune_with_zeros_restores_the_first_shape():
    with xls.Batch(boxes(), filter_prec=xls.XLS_PREC_FP32) as b:
        captures = []
        for shape in (None, (0, 0, 0, 0), (256, 2, 4, 1), (0, 0, 0, 0)):
            print(f"[case] tune {shape}", flush=True)
            for i in range(len(PARAMS)):
                if shape:
                    b.xls_batch_subdomain(i).xls_subdomain_tune(xls.XLS_PREC_FP32, *shape)
            results(b, True)
            captures.append(b.xls_batch_stats()["captures"])
    assert captures == [1, 1, 2, 2]
