"""What an autotuner's cache entry belongs to: the meaning of the knobs when it was found, and the
spheres themselves (their columns decide which plane kernels fit), not only their sizes."""
import dataclasses
import types

import numpy as np

from paper_2501_08697_amd import autotune
from paper_2501_08697_amd import workload as W


def problem(miller=None):
    p = W.make_problem(W.tiny_config(fft=16, ecut=12.0, kfrac=((0.0, 0.0, 0.0), (0.5, 0.0, 0.0))))
    if miller is not None:
        p = dataclasses.replace(p, miller=miller(p.miller.copy()))
    return types.SimpleNamespace(prob=p, fft=p.fft, npw=p.npw, nproj=p.nproj)


def test_key_names_the_spheres():
    a, b = problem(), problem(lambda m: np.ascontiguousarray(m[:, [1, 0, 2]]))   # the same sizes, x and y exchanged
    assert autotune.key(a, 4, 0) == autotune.key(problem(), 4, 0)
    assert autotune.key(a, 4, 0) != autotune.key(b, 4, 0)
    assert autotune.key(a, 4, 0) != autotune.key(a, 5, 0)
    assert autotune.key(a, 4, 0) != autotune.key(a, 4, 1)


def test_key_of_other_knob_meanings_is_another():
    """An entry from before plane mode 0 meant the column passes would pin the slab passes."""
    d = problem()
    old = f"fft={d.fft};npw={list(map(int, d.npw))};nproj={d.nproj};nb=4;prec=0"
    k = autotune.key(d, 4, 0)
    assert k != old and f"knobs={autotune.KNOBS}" in k.split(";")
