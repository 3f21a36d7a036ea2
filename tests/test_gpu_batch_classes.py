"""Untuned slices of one coil class share one persistent launch per direction,
also where the single solves' rule would give them different held tiles: the
captured solve has as many nodes as with every slice pinned to four tiles, and
the results are those of the single solves to the bit."""
import ctypes

import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _nodes(graph):
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    n = ctypes.c_size_t()
    assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


def test_one_launch_per_coil_class():
    from paper_2604_09233_amd import nfs

    probs, ms = [], []
    for i, (L, K, G) in enumerate([(9216, 9001, 12), (16900, 15003, 16), (2303, 6007, 9), (23409, 25013, 14)]):
        d = synth.random_problem(L, K, G, 9, seed=60 + i)
        probs.append(nfs.Problem(*(d[k] for k in ("sens", "fields", "b0", "kcoef", "t"))))
        ms.append(torch.from_numpy(d["m"]).cuda())
    shapes = [nfs.tuned_shape(p, "bf16") for p in probs]
    assert any(len({s[op][0] for s in shapes}) > 1 for op in ("E", "EH")), shapes
    single = [nfs.cg_solve(p, m, 3, precision="bf16") for p, m in zip(probs, ms)]

    def nodes():
        nfs.cg_solve_batched(probs, ms, 3, precision="bf16")  # streams and events exist before the capture
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g):
            out = nfs.cg_solve_batched(probs, ms, 3, precision="bf16")
        n = _nodes(g)
        for _ in range(3):
            g.replay()
            torch.cuda.synchronize()
            for i, one in enumerate(single):
                assert torch.equal(out[0][i], one[0]) and torch.equal(out[1][i], one[1])
        return n

    nfs.set_batch_mode(0, "persistent")
    try:
        n = nodes()
        for p, s in zip(probs, shapes):
            for op in ("E", "EH"):
                nfs.set_shape(p, "bf16", op, 4, s[op][1])
        assert n == nodes()
    finally:
        nfs.set_batch_mode(0, "streams")
