"""GPU test of the planner's per-thread memory (needs an MI355X): calls that
differ only in one number of the plan's key, in an order that hits and misses,
from several threads on streams of their own, each against the oracle.
"""

import threading

import numpy as np
import pytest
import torch

from oracle import qlin_ref as ref
from paper_2607_04244_amd import qlin
from synth import gen

from test_parity import dev, host_bits, make

pytestmark = pytest.mark.gpu


def test_plans_remembered_per_thread_fit_their_call():
    """The same rows and members with the whole workspace, half of it and
    none, forced and automatic, one member and two: a plan remembered for one
    must not serve another (a split that does not fit would be refused or
    overrun its workspace)."""
    M, K = 48, 2560
    cases = [gen.random_case(810 + i, M, K, N) for i, N in enumerate((320, 1040))]
    refs = [ref.forward(cases[0]["x"], c["packed"], c["scales"], c["zeros"]) for c in cases]
    errors = []

    def work(seed):
        try:
            lins = [make(c) for c in cases]
            rng = np.random.default_rng(seed)
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                x = dev(cases[0]["x"])
                stream.synchronize()
                for _ in range(40):
                    rows = int(rng.choice([3, 16, 17, M]))
                    mem = [[0], [1], [0, 1]][int(rng.integers(0, 3))]
                    path, split = [(0, 0), (2, 3), (3, 4), (3, 0)][int(rng.integers(0, 4))]
                    group = [lins[i] for i in mem]
                    need, _ = qlin.group_plan(group, rows, path, split)
                    nb = need if split else [need, need // 2 // 16 * 16, 0][int(rng.integers(0, 3))]
                    ws = qlin.new_workspace(nb) if nb else None
                    ys = qlin.forward_group(group, x[:rows], path=path, split_k=split, workspace=ws)
                    stream.synchronize()
                    for i, y in zip(mem, ys):
                        r = ref.compare(host_bits(y), refs[i][:rows])
                        assert r["ok"], (rows, mem, path, split, nb, r)
            for l in lins:
                l.close()
        except BaseException as e:      # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(s,)) for s in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    if errors:
        raise errors[0]
