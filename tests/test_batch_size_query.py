"""The size query of a large ensemble, without a GPU."""
import ctypes as C
import time

import synth
import paper_1410_2569_amd as L


def _query_seconds(count, shapes, walls, tune):
    arr = (L.Params * count)()
    for i in range(count):
        nx, ny = shapes[i % len(shapes)]
        arr[i] = L.make_params(synth.base_params(nx=nx, ny=ny)) if i < len(shapes) \
            else arr[i % len(shapes)]
        arr[i].walls, arr[i].ghost_psi = walls, 0
    n, best = C.c_size_t(), float("inf")
    for _ in range(3):
        t = time.perf_counter()
        assert L.lib().lbm_batch_workspace_size(arr, count, C.byref(tune), C.byref(n)) == 0
        best = min(best, time.perf_counter() - t)
    return best


def test_split_into_segments_costs_little_beside_the_layout():
    """The rule that splits an ensemble's lattices into marching segments weighs about a thousand
    heights. Its cost must follow the distinct lattices, of which an ensemble has few, not the
    instances: the query of 3,000 instances stays within a few times that of as many solid masks,
    whose layout is the same and which have no such rule (a weighing of every instance takes
    hundreds of times as long)."""
    shapes = [(50, 1100 + 40 * k) for k in range(6)]
    tune = L.lbm.Tune(1, 0, 0, 2)
    with_rule = _query_seconds(3000, shapes, 1, tune)
    without = _query_seconds(3000, shapes, 3, tune)
    assert with_rule <= 10 * without + 1e-3, (with_rule, without)
