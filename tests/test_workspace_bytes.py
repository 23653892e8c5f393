"""Workspace sizes of test-particle mode (host only): the second set of lists and
the planets' slots of every step are taken only where a graph has two branches,
from 8192 particles on and with encounters."""
import ctypes

import pytest

from paper_1404_2324_amd import genga as G

LIST = 4 * 6 + 8 * 7  # bytes of a particle in the second set of lists


def _bytes(ntp, **kw):
    p = G.default_params(**kw)
    return G.lib().genga_workspace_bytes(G.GENGA_TEST, ctypes.byref(p), 8, ntp, 0, 0)


@pytest.mark.parametrize("ntp", [8192, 20000, 1000000])
def test_no_second_lists_without_encounters(ntp):
    assert _bytes(ntp, encounter_free=1) + LIST * ntp <= _bytes(ntp)


def test_no_second_lists_with_few_particles():
    assert _bytes(8191) + LIST * 8191 <= _bytes(8192)
    # what one set of everything takes: 345 bytes a particle and 8 planets, and
    # the planets' share, under 1 MB
    assert _bytes(3001) <= 3001 * 345 + (1 << 20)
