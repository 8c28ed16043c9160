"""Workgroups of several waves that set a layer's status agree on it before they use barriers.

The orders of a layer run in one launch and share its status entry. A kernel in which every wave read the
entry for itself could have some waves leave, because another order failed meanwhile, while the others wait at
a barrier or use what the missing wave should have written. Shown on the sources: every kernel that stores to
the status and has barriers takes its decision by layer_failed, and the general form of that function hands
one thread's reading over through LDS. The GPU test has many orders of a layer fail in one launch."""

import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_1707_05882_amd", "csrc")


def _source(name):
    with open(os.path.join(CSRC, name)) as f:
        return re.sub(r"//[^\n]*", "", f.read())


def _functions(text):
    """(head, body) of every function defined in the text, by brace matching."""
    for m in re.finditer(r"(?:__global__|__device__)[^;{}]*\{", text):
        depth, i = 1, m.end()
        while depth:
            depth += {"{": 1, "}": -1}.get(text[i], 0)
            i += 1
        yield text[m.start():m.end()], text[m.end():i]


def _name(head):
    names = re.findall(r"(\w+|operator\W)\s*\(", head)
    return [x for x in names if x not in ("__launch_bounds__", "__attribute__")][0]


def test_kernels_that_set_the_status_agree_on_it():
    seen = 0
    for f in sorted(os.listdir(CSRC)):
        if not f.endswith(".hip"):
            continue
        functions = [(h, _name(h), b) for h, b in _functions(_source(f))]
        stores = {n for _, n, b in functions if re.search(r"status\[[^\]]*\]\s*=[^=]", b)}
        waits = {n for _, n, b in functions if "__syncthreads" in b}
        calls = {n: set(re.findall(r"\b(\w+)(?:<[^;()]*>)?\s*\(", b)) for _, n, b in functions}

        def reaches(n, what, todo=None):
            done, todo = set(), [n]
            while todo:
                x = todo.pop()
                if x in what:
                    return True
                done.add(x)
                todo += [c for c in calls.get(x, ()) if c in calls and c not in done]
            return False

        for head, name, body in functions:
            if "__global__" not in head or not (reaches(name, stores) and reaches(name, waits)):
                continue
            seen += 1
            assert "layer_failed(status" in body, (f, name)
            assert not re.search(r"status\[[^\]]*\]\s*!=", body), (f, name)
    # LU in two files, V, the eigensolvers and their persistent forms
    assert seen >= 8


def test_one_thread_reads_for_all():
    body = dict((_name(h), b) for h, b in _functions(_source("vbrdf_internal.hpp")))["layer_failed"]
    read, wait = body.index("threadIdx.x == 0"), body.index("__syncthreads")
    assert body.index("__shared__") < read < wait < body.index("return")
    assert body.count("__hip_atomic_load") == 1


@pytest.mark.gpu
@pytest.mark.parametrize("N", [8, 20, 32, 40])
def test_layers_whose_orders_fail_in_one_launch(N):
    """A cap of a few sweeps per problem fails some orders of each layer sooner than others; every call ends, its
    layers are reported NUMERIC, and the plan without the cap gives the same bits afterwards as before."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        raise RuntimeError("GPU tests need a ROCm device")
    from paper_1707_05882_amd import binding
    from paper_1707_05882_amd.api import BRDFSolver
    from workloads.layers import hg_like_coefficients

    nl, M, L = 4, 40, 48
    rng = np.random.default_rng(900 + N)
    coefs = [hg_like_coefficients(rng, L)[0] for _ in range(nl)]
    tau, om = [0.5, 2.0, 8.0, 30.0], [0.7, 0.9, 0.99, 0.999]
    shape = ([N] * nl, [L] * nl, [M] * nl, [5] * nl)
    whole = BRDFSolver(*shape)
    before = [F.clone() for F in whole(tau, om, coefs)]
    for cap in (1, 3, 10):
        for sched in (binding.EIGEN_PLAN_ORDER, binding.EIGEN_LONGEST_FIRST, binding.EIGEN_PERSISTENT):
            s = BRDFSolver(*shape, qr_sweep_cap=cap)
            s.plan.set_tuning(sched, 16)
            print(f"N = {N}, cap {cap}, schedule {sched}", flush=True)
            s.solve_device(*s.upload(tau, om, coefs))
            torch.cuda.synchronize()
            assert s.status.cpu().tolist() == [binding.E_NUMERIC] * nl
    assert all(torch.equal(a, b) for a, b in zip(whole(tau, om, coefs), before))
