"""Carrying a population forward: the whole buffer in one copy, and array by array where a caller has
put an array of its own into a population (no GPU needed)."""
import pytest
import torch

from paper_2407_17296_amd import driver


@pytest.fixture
def run():
    r = driver.SMC2Run.__new__(driver.SMC2Run)
    shapes = dict(theta=(2, 3, 2), logpost=(2, 3), grad_logpost=(2, 3, 2), loglik=(2, 3), logw=(2, 3))

    def pop():
        sizes = [torch.Size(s).numel() for s in shapes.values()]
        flat = torch.zeros(sum(sizes), dtype=torch.float64)
        return flat, {k: v.view(s) for v, (k, s) in zip(torch.split(flat, sizes), shapes.items())}
    r._cur_flat, r.cur = pop()
    r._prev_flat, r.prev = pop()
    for i, v in enumerate(r.cur.values()):
        v.copy_(torch.arange(v.numel(), dtype=torch.float64).view(v.shape) + 100 * i)
    return r


def _carried(run):
    return all(torch.equal(run.prev[k], run.cur[k]) for k in run.cur)


def test_carry(run):
    run._carry()
    assert _carried(run)
    assert torch.equal(run._prev_flat, run._cur_flat)


@pytest.mark.parametrize("side", ["cur", "prev"])
@pytest.mark.parametrize("key", ["theta", "logpost", "logw"])
def test_carry_with_a_replaced_array(run, side, key):
    pop = getattr(run, side)
    pop[key] = torch.full_like(pop[key], -7.0)
    run._carry()
    assert _carried(run)


def test_carry_with_an_added_array(run):
    run.cur["extra"], run.prev["extra"] = torch.ones(3), torch.zeros(3)
    run._carry()
    assert _carried(run)


def test_carry_with_storage_swapped_under_a_view(run):
    run.cur["theta"].data = torch.full((2, 3, 2), 5.0, dtype=torch.float64)
    run._carry()
    assert _carried(run)
