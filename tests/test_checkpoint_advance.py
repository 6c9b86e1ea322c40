"""The executor against a lattice that advances from snapshot to snapshot, as
Lattice does (CPU only): schedules replayed on a fake lattice whose state is its
step index.  An advance into a snapshot leaves the lattice's own state at any
earlier step, so nothing may read it afterwards."""
import pytest

from paper_1703_04594_amd import checkpoint as ck


class Slot:
    def __init__(self):
        self.n = None

    def copy_(self, other):
        self.n = other.n


class Advancing:
    def __init__(self):
        self.n = 0
        self.expect = None
        self.steps = self.copies = self.pending = self.takes = 0

    def new_state(self):
        return Slot()

    def get_state(self, out):
        assert self.n is not None
        out.n = self.n
        self.copies += 1
        return out

    def set_state(self, s):
        self.n = s.n
        self.copies += 1

    def step(self, k):
        self.n += k
        self.steps += k

    def advance_state(self, src, dst, k):
        assert k >= 1 and (src is None or src is not dst)
        n = (self.n if src is None else src.n) + k
        self.steps += k
        if dst is None:
            self.n = n
        else:
            dst.n = n
            self.n = None      # not kept

    def step_state(self, src, dst):
        raise AssertionError("advance_state covers it")

    def adjoint_step(self, s, dacc):
        assert s.n == self.expect and dacc is None
        self.expect -= 1
        self.pending += 1

    def take_dtau(self, dacc):
        assert self.pending > 0
        self.pending = 0
        self.takes += 1


@pytest.mark.parametrize("kind", ["sqrt", "binomial1", "binomial2", "binomial3", "binomial7"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 7, 10, 16, 17, 36, 61])
def test_every_reverse_step_gets_its_state(N, kind):
    sch = ck.sqrt_schedule(N) if kind == "sqrt" else ck.binomial_schedule(N, int(kind[-1]))
    fwd, bwd = sch.split_at_first_adjoint()
    lat = Advancing()
    ex = ck.Executor(lat, None)
    ex.run(fwd)
    ex.final_step()                # the rollout's last step
    assert lat.n == N and ex.where == ck.Executor.LATTICE
    lat.expect = N - 1
    ex.run(bwd)
    assert lat.expect == -1 and lat.pending == 0 and lat.takes == 1
    assert ex.adjoint_steps == N
    assert ex.forward_steps == sch.forward_steps()
    assert lat.steps == sch.forward_steps() + 1
    assert ex.peak_slots <= sch.slots_needed
    # no copies but of the initial state, and of one stored where it stands
    assert lat.copies <= 2


def test_an_advance_stored_in_its_own_slot_goes_through_the_lattice():
    lat = Advancing()
    ex = ck.Executor(lat, None)
    ex.run([("store", 0, 0), ("restore", 0, 0), ("advance", 0, 3), ("store", 3, 0), ("restore", 3, 0), ("advance", 3, 3),
            ("store", 3, 1)])
    assert ex.slots[0].n == 3 and ex.slots[1].n == 3
