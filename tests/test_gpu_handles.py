"""Tensor handles in unusual states: moved-from operands, operands and results
that share memory."""
import ctypes

import numpy as np
import pytest

from paper_2512_23917_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    from paper_2512_23917_amd import tci
    return tci


@pytest.fixture(scope="module")
def ctx(T):
    c = T.Context(0)
    yield c
    c.close()


def draw(shape, seed):
    return synth.complex_gaussian(synth.rng(41, seed), shape)


@pytest.mark.parametrize("side", [0, 1])
def test_moved_from_operand_is_refused(T, ctx, side):
    """A handle keeps its dimensions when its data is moved away; an update that gets it fails on the host."""
    ops = [[T.Tensor.from_numpy(ctx, draw(s, i), T.C128) for i in range(2)] for s in ((3, 2, 4), (4, 2, 3))]
    taken = ctypes.c_void_p()
    T._check(T.lib().tci_move(ctx.h, ctypes.byref(ops[side][1].h), ctypes.byref(taken)), "tci_move")
    p = T.update_params(chi_min=1, chi_max=4, direction=T.DIR_LEFT)
    with pytest.raises(T.TciError):
        T.two_site_update_batched(ctx, ops[0], ops[1], None, p)
    T._check(T.lib().tci_destroy(ctx.h, taken), "tci_destroy")
    # the context goes on
    out = T.two_site_update_batched(ctx, ops[0][:1], ops[1][:1], None, p) if side else None
    assert out is None or out[3][0].chi == 4
