"""What wave_alloc accepts of a velocity model and an eta array (host checks
only: the arena is NULL, which is looked at last)."""
import numpy as np
import pytest

from paper_2009_04619_amd import wave as W

NAN_SIGN = np.array([0xFFC00000], np.uint32).view(np.float32)[0]


def alloc(vel, eta=None):
    nz, ny, nx = vel.shape
    d = W.make_desc(nx, ny, nz, 3, 10, 10, 10, 1e-3, eta_array=eta is not None)
    rc, _ = W.wave_alloc(d, vel, eta, 0, 0, 0)
    return rc, W.wave_last_error()


@pytest.mark.parametrize("bad", [0.0, -0.0, -1.0, np.inf, -np.inf, np.nan, NAN_SIGN])
@pytest.mark.parametrize("where", [0, 5, -1])
def test_velocity_values(bad, where):
    vel = np.full((7, 9, 11), 2000.0, np.float32)
    assert "arena" in alloc(vel)[1]
    vel.reshape(-1)[where] = bad
    rc, msg = alloc(vel)
    assert rc == W.WAVE_EINVAL and "velocity" in msg


def test_largest_velocity_is_found():
    vel = np.full((7, 9, 11), 1e-42, np.float32)     # subnormal values are positive
    assert "arena" in alloc(vel)[1]
    vel[6, 8, 10] = 9000.0                            # dt 1 ms: above the stability bound
    assert alloc(vel)[0] == W.WAVE_EUNSTABLE


@pytest.mark.parametrize("value,ok", [(0.0, True), (-0.0, True), (1e-45, True), (-1e-45, False),
                                      (np.inf, False), (-np.inf, False), (np.nan, False), (NAN_SIGN, False)])
def test_eta_values(value, ok):
    vel = np.full((7, 9, 11), 2000.0, np.float32)
    eta = np.full((7, 9, 11), 0.1, np.float32)
    eta[3, 4, 5] = value
    rc, msg = alloc(vel, eta)
    assert ("arena" in msg) if ok else (rc == W.WAVE_EINVAL and "eta" in msg)
    eta[3, 4, 5] = 4.9
    assert alloc(vel, eta)[0] == W.WAVE_EUNSTABLE
