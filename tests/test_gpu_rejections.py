"""What a rejected classification leaves behind: the geometry in force, whole."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2206_11634_amd import binding as B
from paper_2206_11634_amd import workloads as W
from test_gpu_parity import FORCE_TOL, POP_TOL, _compare_geometry

pytestmark = pytest.mark.gpu

LAT, PS = W.tiny_case(21, dims=(34, 30, 32), periodic=(1, 0, 1), n_particles=3,
                      diameter_range=(5.0, 8.0), speed=0.08, spin=0.004, u0=(0.02, 0.0, 0.01))


def _rejected(P, why):
    """Device particles at P that the boxes' check rejects."""
    parts = B.DeviceParticles(P)
    if why == "centre":
        parts.t["pos"][1, 0] = float("nan")
    elif why == "weight":
        parts.t["K"][-1] = -1.0
    else:   # a control point far from its body
        parts.t["world_pts"][0, 1] += 400.0
    return parts


def _reject(gpu, P, why):
    with pytest.raises(B.LbmError) as e:
        gpu.classify(_rejected(P, why))
    assert e.value.code == B.LBM_EINVAL


def _step(gpu, ora, parts, P, what):
    gpu.step(parts)
    Fo, To = ora.step(P)
    F, T = (t.cpu().numpy()[:P.n] for t in gpu.forces())
    assert np.abs(Fo).max() > 1e-6, what
    assert np.abs(F - Fo).max() <= FORCE_TOL["f64"] * np.abs(Fo).max(), what
    assert np.abs(T - To).max() <= FORCE_TOL["f64"] * np.abs(To).max(), what
    fluid = ora.owner == 0
    assert np.abs(gpu.populations() - ora.f)[:, fluid].max() <= POP_TOL["f64"], what


@pytest.mark.parametrize("classify", ["balls", "sweep"])
@pytest.mark.parametrize("why", ["centre", "weight", "reach"])
@pytest.mark.parametrize("last", [0, 2])
def test_steps_and_snapshots_after_a_rejected_classification(classify, why, last):
    """After the first classification, and after one with refills: owners, links,
    refills and the snapshot are those of before the rejected one, and the steps
    that follow it match the oracle's, links and forces included."""
    import torch
    gpu, ora = B.Lattice.for_particles(LAT, PS, storage="f64", classify=classify), O.Oracle(LAT)
    parts = B.DeviceParticles(PS)
    for n in range(last + 1):
        P = W.prescribed_state(PS, LAT, float(n))
        parts.set_state(P)
        gpu.classify(parts)
        ora.classify(P)
        if n < last:
            _step(gpu, ora, parts, P, n)
    assert last == 0 or len(ora.refill_nodes) > 0
    snaps = [torch.zeros(gpu.geometry_bytes()[0], dtype=torch.uint8, device="cuda") for _ in range(2)]
    gpu.geometry_save(snaps[0])
    for _ in range(2):
        _reject(gpu, P, why)
    _compare_geometry(gpu, ora, why)
    gpu.geometry_save(snaps[1])
    assert torch.equal(*snaps)
    for k in range(2):
        _step(gpu, ora, parts, P, (why, k))
    gpu.close()


@pytest.mark.parametrize("classify", ["balls", "sweep"])
@pytest.mark.parametrize("rejections", [1, 2, 3])
def test_classification_after_a_rejected_one(classify, rejections):
    """Bodies that moved little since the classification in force (the sweep mode
    then works from its candidate lists): flags, through the populations of the
    nodes that left a body, and refills of the next classifications match the
    oracle's."""
    gpu, ora = B.Lattice.for_particles(LAT, PS, storage="f64", classify=classify), O.Oracle(LAT)
    parts, refilled = B.DeviceParticles(PS), 0
    for n in range(6):
        P = W.prescribed_state(PS, LAT, float(n))
        if n in (2, 4):
            for _ in range(rejections):
                _reject(gpu, P, "weight")
        parts.set_state(P)
        gpu.classify(parts)
        ora.classify(P)
        _compare_geometry(gpu, ora, n)
        refilled += len(ora.refill_nodes) if n in (2, 4) else 0
        _step(gpu, ora, parts, P, n)
    assert refilled > 0
    gpu.close()
