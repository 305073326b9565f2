"""chi^2 in one pass (residual and norm by the library, the gradient's factor in
the gather) against the separate steps it replaces and against FP64: the values,
the gradient scaled by what follows the loss, a repeated backward, skipped
records, odd sizes; and the calls that keep the separate steps (observations
with a gradient, of another type, conjugated or strided)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2111_04141_amd import autograd as AG
from paper_2111_04141_amd import workload as W
from tests import helpers as H

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _setup(npol, nrec, n=90, support=7, beta=4, seed=3):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    rng = np.random.Generator(np.random.PCG64(seed + nrec))
    uvw = np.concatenate([rng.uniform(-n / 2 - 2, n / 2 + 2, (nrec, 2)), np.zeros((nrec, 1))], 1)
    taps = W.pswf_taps(support, beta).astype(np.float32)
    spec = api.GridSpec(n, n, npol, beta, 1.0, 1.0)
    bank = api.KernelBank("separable", torch.from_numpy(taps).cuda(), support=support)
    plan = api.Plan(spec, bank, torch.from_numpy(uvw).cuda())
    geom = oracle.Geometry(nu=n, nv=n, beta=beta, scale_u=1.0, scale_v=1.0, support=support)

    def cplx(*shape):
        return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    return plan, geom, taps.astype(np.float64), uvw, cplx(npol, n, n), cplx(nrec, npol)


def _separate(m, plan, obs, sigma):
    r = obs - AG.Degrid.apply(m, plan)
    return (r.real.double() ** 2 + r.imag.double() ** 2).sum() / (sigma * sigma)


@pytest.mark.parametrize("npol,nrec", [(4, 1), (1, 63), (3, 1025), (2, 20_011), (4, 300_001)])
def test_chi2_one_pass(npol, nrec):
    plan, geom, taps, uvw, model, obs = _setup(npol, nrec)
    md, od = torch.from_numpy(model).cuda(), torch.from_numpy(obs).cuda()
    keep = od.clone()
    m = md.clone().requires_grad_(True)
    loss = AG.chi2(m, plan, od, 0.3)
    assert loss.dtype == torch.float64 and loss.dim() == 0
    (3.0 * loss).backward(retain_graph=True)
    first = m.grad.clone()
    m.grad = None
    (3.0 * loss).backward()
    assert H.rel_l2(m.grad.cpu().numpy(), first.cpu().numpy()) < 1e-6
    assert torch.equal(od, keep)
    m2 = md.clone().requires_grad_(True)
    loss2 = _separate(m2, plan, od, 0.3)
    (3.0 * loss2).backward()
    # the same FP32 residuals, summed in FP64 in another order
    assert abs(loss.item() - loss2.item()) <= 1e-12 * abs(loss2.item())
    assert H.rel_l2(first.cpu().numpy(), m2.grad.cpu().numpy()) < 1e-6
    res = obs - oracle.degrid(geom, taps, uvw, model.astype(np.complex128))[0]
    assert abs(loss.item() - np.sum(np.abs(res) ** 2) / 0.09) <= TOL * abs(loss.item())
    ref, _ = oracle.grid(geom, taps, uvw, -6.0 / 0.09 * res)
    assert H.rel_l2(first.cpu().numpy(), ref) < TOL
    plan.close()


def test_calls_that_keep_the_separate_steps():
    plan, _, _, _, model, obs = _setup(2, 4000)
    md, od = torch.from_numpy(model).cuda(), torch.from_numpy(obs).cuda()
    strided = torch.stack([od, od], -1)[..., 0]
    for o in (od.to(torch.complex128), od.conj().clone().conj(), strided):
        m, m2 = md.clone().requires_grad_(True), md.clone().requires_grad_(True)
        a, b = AG.chi2(m, plan, o, 0.5), _separate(m2, plan, o, 0.5)
        a.backward()
        b.backward()
        assert a.item() == b.item()
        assert H.rel_l2(m.grad.cpu().numpy(), m2.grad.cpu().numpy()) < 1e-6
    og, og2 = od.clone().requires_grad_(True), od.clone().requires_grad_(True)
    AG.chi2(md, plan, og, 0.5).backward()
    _separate(md, plan, og2, 0.5).backward()
    assert torch.equal(og.grad, og2.grad)
    with pytest.raises(RuntimeError):
        AG.chi2(md, plan, od[:-1], 0.5)
    plan.close()
