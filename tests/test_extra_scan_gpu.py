"""GPU parity of the direct-to-LDS block scan with activations and epilogues (fused Swish, accumulated
slices of wide features) at the edges of its 32-row blocks and of its pipeline, against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2405_17381_amd import binding

pytestmark = pytest.mark.gpu
TOL = 2e-2      # bf16, as everywhere: 16-bit operands and results, max |difference| over max |result|


def _close(names, got, ref):
    for nm, x, r in zip(names, got, ref):
        x = x.to(torch.float64).cpu().numpy()
        assert np.isfinite(x).all(), nm
        assert oracle.rel_max_err(x, r) <= TOL, (nm, oracle.rel_max_err(x, r))


LENGTHS = [(1, 0), (31, 0), (32, 0), (33, 0), (65, 0), (97, 64), (129, 64), (200, 128)]
FORMS = [(n, lseg, sw) for n, lseg in LENGTHS for sw in (None, "piece")]
FORMS += [(n, lseg, sw) for n, lseg in ((33, 0), (129, 64)) for sw in ("no_trio", "no_pair")]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,lseg,switch", FORMS)
def test_swish_block_edges(n, lseg, d, switch):
    lam = [1.0, 0.99, 0.6]
    g = torch.Generator().manual_seed(300 + n + d)
    Qp, Kp, V, dO = [torch.randn((2, 3, n, d), generator=g).to(torch.bfloat16) for _ in range(4)]
    V = (V.float() / d).to(torch.bfloat16)
    sw = {"lseg": lseg, "piece": -1}
    if switch == "piece":                       # the same scans in pieces of 32 tokens
        sw = {"piece": 32}
    elif switch:
        sw[switch] = 1
    xs = [x.cuda() for x in (Qp, Kp, V, dO)]
    with binding.debug(**sw):
        O = binding.la_fwd_swish(xs[0], xs[1], xs[2], lam)
        grads = binding.la_bwd_swish(xs[0], xs[1], xs[2], lam, xs[3])
        torch.cuda.synchronize()
    qp, kp, v, do = [x.to(torch.float64).numpy() for x in (Qp, Kp, V, dO)]
    q, k = oracle.swish(qp), oracle.swish(kp)
    dQ, dK, dV = oracle.c_recurrence_bwd(q, k, v, lam, do)
    ref = (oracle.c_recurrence_fwd(q, k, v, lam), dQ * oracle.swish_grad(qp), dK * oracle.swish_grad(kp), dV)
    _close(("O", "dQp", "dKp", "dV"), (O,) + tuple(grads), ref)


@pytest.mark.parametrize("dv,m", [(64, 2), (64, 4), (128, 2), (128, 3)])
@pytest.mark.parametrize("n,lseg", [(1, 0), (32, 0), (33, 0), (97, 64), (200, 128), (300, 64)])
def test_wide_block_edges(n, lseg, dv, m):
    lam = [1.0, 0.97]
    dk = m * dv
    g = torch.Generator().manual_seed(500 + n + dk)
    mk = lambda f, s: (torch.randn((2, 2, n, f), generator=g) * s).to(torch.bfloat16)
    Qw, Kw, V, dO = mk(dk, dk ** -0.5), mk(dk, dk ** -0.5), mk(dv, dv ** -0.5), mk(dv, 1.0)
    xs = [x.cuda() for x in (Qw, Kw, V, dO)]
    with binding.debug(lseg=lseg, wide_slices=1, piece=-1):
        O = binding.la_fwd_wide(xs[0], xs[1], xs[2], lam)
        grads = binding.la_bwd_wide(xs[0], xs[1], xs[2], lam, xs[3])
        torch.cuda.synchronize()
    qw, kw, v, do = [x.to(torch.float64).numpy() for x in (Qw, Kw, V, dO)]
    O_, dQ_, dK_, dV_ = np.zeros_like(v), np.empty_like(qw), np.empty_like(kw), np.zeros_like(v)
    for j in range(m):
        sl = slice(j * dv, (j + 1) * dv)
        q, k = np.ascontiguousarray(qw[..., sl]), np.ascontiguousarray(kw[..., sl])
        O_ += oracle.c_recurrence_fwd(q, k, v, lam)
        dQ_[..., sl], dK_[..., sl], c = oracle.c_recurrence_bwd(q, k, v, lam, do)
        dV_ += c
    _close(("O", "dQw", "dKw", "dV"), (O,) + tuple(grads), (O_, dQ_, dK_, dV_))
    with binding.debug(wide_slices=1, piece=64):        # the same scans in pieces
        O = binding.la_fwd_wide(xs[0], xs[1], xs[2], lam)
        grads = binding.la_bwd_wide(xs[0], xs[1], xs[2], lam, xs[3])
        torch.cuda.synchronize()
    _close(("O", "dQw", "dKw", "dV"), (O,) + tuple(grads), (O_, dQ_, dK_, dV_))
