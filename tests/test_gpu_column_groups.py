"""Band groups of the column passes that are part full: batches which the bands of a z-pass or a
plane work-group do not divide, several groups per k-point, in one stream and two, each against the
oracle and with the kernels that ran named. Bars as in test_gpu_apply_h and test_gpu_density:
relative max-norm 1e-12 in FP64, 1e-5 in FP32.
"""
import contextlib
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2501_08697_amd import workload as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

K3 = ((0.0, 0.0, 0.0), (0.5, 0.0, 0.0), (0.25, 0.375, 0.5))
COLUMNS, SLABS = {"z_inv", "plane", "z_fwd"}, {"yz_inv", "xpass", "yz_fwd"}
TOL = {0: 1e-12, 1: 1e-5}


def cell(n1, n2, nb, kfrac=K3):
    a1, a2 = 0.28 * n1, 0.28 * n2
    lat = np.diag([a1, a2, a2])
    p = W.make_problem(W.tiny_config(a=a1, ecut=26.0, fft=max(n1, n2), kfrac=kfrac, natom=3, lmax=1, nb=nb, seed=8),
                       lattice=lat)
    fft = (n1, n2, n2)
    return dataclasses.replace(p, fft=fft, vloc=np.ascontiguousarray(W.gaussian_vloc(lat, fft, p.tau, p.depth)))


@contextlib.contextmanager
def recorded(b, names, **knobs):
    """Runs the block with the knobs set and adds the names of the kernels that it launched."""
    try:
        b.set_tuning(**knobs)
        b.profile_enable()
        b.profile_read()
        yield
        names.update(b.profile_read())
    finally:
        b.profile_enable(False)
        b.set_tuning()


def err(y, ref):
    return np.max(np.abs(y.cpu().numpy() - ref)) / np.max(np.abs(ref))


@pytest.mark.parametrize("n1,n2,prec,kernels", [(32, 32, 0, COLUMNS), (32, 32, 1, COLUMNS), (48, 54, 0, COLUMNS),
                                                (48, 54, 1, SLABS), (72, 120, 0, COLUMNS), (80, 80, 1, COLUMNS),
                                                (90, 90, 1, SLABS)])
def test_part_full_groups(n1, n2, prec, kernels):
    from paper_2501_08697_amd import binding as b
    p = cell(n1, n2, 13, K3 if n1 < 72 else K3[:2])   # 72 x 120: a plane alone on its CU
    print(f"[column groups] fft={p.fft} npw={list(p.npw)} prec={prec}", flush=True)
    dp, x = b.DeviceProblem(p), torch.from_numpy(p.psi).cuda()
    x = x.to(torch.complex64) if prec else x
    ref = oracle.apply_h(p, p.psi)
    # groups of 3, 3 and 1 and of 5 and 2; of 2 with one left; a batch of 8 and one of 5
    for knobs in (dict(band_batch=7, yz_bands=3, x_bands=5), dict(yz_bands=2, x_bands=4),
                  dict(band_batch=8, yz_bands=4, x_bands=3, overlap=1)):
        names = set()
        with recorded(b, names, **knobs):
            y = b.apply_h(dp, x, prec)
        assert err(y, ref) < TOL[prec], knobs
        assert kernels <= names and not ((COLUMNS | SLABS) - kernels) & names, names


@pytest.mark.parametrize("n,kernel", [(32, "density_plane"), (45, "density_plane"), (80, "density_x")])
def test_part_full_groups_density(n, kernel):
    from paper_2501_08697_amd import binding as b
    p = cell(n, n, 13, K3 if n < 80 else K3[:1])
    occ = W.band_weights(p, 3)
    dp, x = b.DeviceProblem(p), torch.from_numpy(p.psi).cuda()
    ref = oracle.density(p, p.psi, occ)
    for knobs in ({}, dict(band_batch=7, yz_bands=3), dict(band_batch=8, yz_bands=4, overlap=1)):
        names = set()
        with recorded(b, names, **knobs):
            rho = b.density(dp, x, occ)
        assert err(rho, ref) < 1e-12, knobs
        assert kernel in names, names


@pytest.mark.parametrize("prec", [0, 1])
def test_default_groups_with_a_remainder(prec):
    """131 bands at two k-points of 72^3: z passes of four bands a work-group, three in the last."""
    from paper_2501_08697_amd import binding as b
    p = cell(72, 72, 131, K3[1:])
    print(f"[column groups] npw={list(p.npw)} nb={p.nb} prec={prec}", flush=True)
    dp, x = b.DeviceProblem(p), torch.from_numpy(p.psi).cuda()
    names = set()
    with recorded(b, names):
        y = b.apply_h(dp, x.to(torch.complex64) if prec else x, prec).cpu().numpy()
    assert COLUMNS <= names
    take = [0, 3, 4, 127, 128, 129, 130]
    for k in range(p.nk):
        xs = p.psi_k(k)[take]
        ref = oracle.apply_h(oracle._single_k(p, k), xs.reshape(-1), nb=len(take)).reshape(len(take), -1)
        assert np.max(np.abs(p.psi_k(k, y)[take] - ref)) < TOL[prec] * np.max(np.abs(ref)), k


def test_compact_rows_at_128():
    """The compact-row slab kernels of a 128^3 plane in FP64, which plane mode 2 still runs."""
    from paper_2501_08697_amd import binding as b
    p = W.make_problem(W.tiny_config(fft=128, ecut=10.0, a=8.0, nb=2, natom=1))
    names = set()
    with recorded(b, names, yz_mode=2):
        y = b.apply_h(b.DeviceProblem(p), torch.from_numpy(p.psi).cuda())
    assert err(y, oracle.apply_h(p, p.psi)) < 1e-12
    assert SLABS <= names, names
