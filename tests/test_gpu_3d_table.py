"""The phase tables of 3D meshes.  complex64: entries hold exp(-i phi) times the cosines a
step's tangent-form factors leave out, in fixed point, and must keep 2^-31 of their own
modulus per part at any angle, as entries of modulus 1 do at 2^30 units: the error of an
entry repeats at every step.  complex128: for the same reason an entry rounds once: half
an ulp, and what the small parts of the product round (a tail of the cosine below 0.017,
that of the sine is smaller; six roundings of at most 2^-53 of it, beside a cosine of
0.7 and more: 0.15 ulp; 0.8 leaves as much again)."""
import math

import numpy as np
import pytest
import torch

import paper_1208_2407_amd as tsq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("angle", [0.0, 1e-7, 0.025, 0.1, 0.3, 0.5, 0.8, 0.95, 0.999])  # rad per step and axis
def test_entries_keep_their_bits_at_any_angle(angle):
    n, dt = 32, 0.1
    dx = np.sqrt(dt / (2 * angle)) if angle else 1.0
    if angle == 0.0:
        dt = 0.0
    V = np.random.default_rng(1).uniform(-20, 20, (n, n, n))
    plan = tsq.Plan(n, n, dt, "c64", nz=n, dx=dx, dy=dx, dz=dx)
    plan.set_potential(torch.from_numpy(V).cuda())
    torch.cuda.synchronize()
    at = n ** 3 * 8  # behind the second psi buffer
    ws = plan.workspace()
    table = ws[at:at + n ** 3 * 8].view(torch.int32).view(-1, 2).cpu().numpy().astype(np.float64)
    entries = (table[:, 0] + 1j * table[:, 1]).reshape(V.shape)
    # the cosines of a step's three odd and six even factors, from the rounded tangents
    odd, even = (float(np.float32(np.tan(tau / (2.0 * dx ** 2)))) for tau in (dt, dt / 2))
    g = (1 + odd ** 2) ** -1.5 * (1 + even ** 2) ** -3.0
    modulus = g * 2.0 ** np.round(np.log2(np.sqrt(np.mean(np.abs(entries) ** 2)) / g))
    assert 2.0 ** 30 * (1 - 2.0 ** -31) <= modulus < 2.0 ** 31
    err = entries / modulus - np.exp(-1j * dt * (V + 3.0 / dx ** 2))
    # rounded to whole units (one where a part meets the largest integer), and doubles
    worst = float(max(np.abs(err.real).max(), np.abs(err.imag).max()))
    assert worst <= 2.0 ** -31 * 1.001


@pytest.mark.parametrize("angle", [0.01, 0.05, 0.3, 0.95])
@pytest.mark.parametrize("scale", [1.0, 30.0, 1e6])
def test_complex128_entries_round_once(angle, scale):
    n, dt = 32, 0.1
    dx = float(np.sqrt(dt / (2 * angle)))
    V = np.random.default_rng(3).uniform(-scale, scale, (n, n, n))
    plan = tsq.Plan(n, n, dt, "c128", nz=n, dx=dx, dy=dx, dz=dx)
    plan.set_potential(torch.from_numpy(V).cuda())
    torch.cuda.synchronize()
    at = n ** 3 * 16
    entries = plan.workspace()[at:at + n ** 3 * 16].view(torch.float64).view(-1, 2).cpu().numpy()
    # the angle in the operations of the library, then 64-bit mantissas
    J = 1.0 / (dx * dx)
    x = dt * (V + (J + J + J)) / 1.0
    tan = [np.longdouble(math.tan(tau * (1.0 / (2.0 * dx * dx)) / 1.0)) for tau in (dt, 0.5 * dt)]
    g = (1 + tan[0] ** 2) ** np.longdouble(-1.5) * (1 + tan[1] ** 2) ** np.longdouble(-3)
    x = x.ravel().astype(np.longdouble)
    for got, want in ((entries[:, 0], g * np.cos(x)), (entries[:, 1], -g * np.sin(x))):
        worst = float(np.max(np.abs(got - want) / np.spacing(np.abs(got))))
        assert worst <= 0.8
