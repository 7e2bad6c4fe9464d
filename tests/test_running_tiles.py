"""Default tile of compiled passes: the fewest passes of the plan that the call
runs - out of place, or in place when the workspace holds no second state or an
out-of-place sweep of the caller's own state would end in the other buffer - and
(5, 8, 5) where no other tile has fewer."""
import random

import pytest

from paper_1804_04797_amd import qsv, workloads

TILES = [(5, 8, 5), (5, 8, 4), (5, 9, 5), (5, 9, 4)]


def _circuits():
    rng = random.Random(3)
    for _ in range(20):
        n, depth, lb = rng.randrange(24, 31), rng.randrange(8, 25), rng.choice((0, 1, 1, 3))
        rows, cols, pres = workloads.lattice_for_qubits(n)
        yield pytest.param(n, (rows, cols, pres, depth, rng.randrange(1000)), lb, id=f"{n}q-d{depth}-from{lb}")


@pytest.mark.parametrize("n,lattice,lb", _circuits())
def test_fewest_passes_that_run(n, lattice, lb):
    c = qsv.circuit_create(*lattice)
    for in_place in (True, False):
        for ws in (0, (8 << n) - 1, 8 << n):
            for oop in (0, 1, -1):
                if oop == 1 and ws < 8 << n:
                    continue

                def run(tile):
                    o = dict(out_of_place=oop)
                    if tile:
                        o.update(jit=1, reg_qubits=tile[0], thread_qubits=tile[1], low_qubits=tile[2])
                    return qsv.sv_debug_fused_plan(c, lb, -1, o, in_place, ws)

                counts = [run(t)[1] for t in TILES]
                want = TILES[counts.index(min(counts))]
                assert run(None) == (want, min(counts)), (in_place, ws, oop, counts)
