"""GPU parity of la_fwd_wide's kernel with the non-square state on cut sequences (d_k = 256, d_v = 128,
bf16), against the CPU oracle and the accumulated scans."""
import numpy as np
import pytest
import torch

import oracle
from paper_2405_17381_amd import binding

pytestmark = pytest.mark.gpu
TOL = 2e-2      # bf16: max |difference| over max |result|, as everywhere


@pytest.mark.parametrize("n,lseg", [(449, 64), (512, 64), (1000, 64), (1337, 128), (2049, 256), (4100, 512)])
def test_cut_sequences(n, lseg):
    """Odd and even numbers of plan segments, partial last blocks and segments, heads on both sides of the
    decay cut-off; the scratch the query gives holds the wide states exactly."""
    B, H, dk, dv = 2, 4, 256, 128
    lam = [1.0, 0.999, 0.95, 0.4]
    g = torch.Generator().manual_seed(1100 + n)
    mk = lambda f, s: (torch.randn((B, H, n, f), generator=g) * s).to(torch.bfloat16)
    Qw, Kw, V = mk(dk, dk ** -0.5), mk(dk, dk ** -0.5), mk(dv, dv ** -0.5)
    guard = 4096
    with binding.debug(lseg=lseg):
        assert binding.la_plan(B, H, n, dv, binding.LA_BF16)[2] >= 8
        need = binding.la_workspace_bytes(B, H, n, dv, binding.LA_BF16, False)
        ws = torch.full((need + guard,), 171, dtype=torch.uint8, device="cuda")
        O = binding.la_fwd_wide(Qw.cuda(), Kw.cuda(), V.cuda(), lam, workspace=ws[:need])
        with binding.debug(wide_slices=1):
            S = binding.la_fwd_wide(Qw.cuda(), Kw.cuda(), V.cuda(), lam)
    assert (ws[need:] == 171).all()
    qw, kw, v = [x.to(torch.float64).numpy() for x in (Qw, Kw, V)]
    ref = np.zeros_like(v)
    for j in range(2):
        sl = slice(j * dv, (j + 1) * dv)
        ref += oracle.c_recurrence_fwd(np.ascontiguousarray(qw[..., sl]), np.ascontiguousarray(kw[..., sl]), v, lam)
    O, S = [x.to(torch.float64).cpu().numpy() for x in (O, S)]
    assert oracle.rel_max_err(O, ref) <= TOL
    assert np.linalg.norm(O - ref) <= np.linalg.norm(S - ref)       # no rounding between the halves
