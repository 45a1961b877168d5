"""GPU parity of the fp32 kernels' split arithmetic (products of three-part bf16 splits) at the edges of
its range: magnitudes where a workgroup changes to the fp32 instruction, infinities and NaN, tiny values,
and the accuracy that the split must not lose against plain fp32 arithmetic."""
import numpy as np
import pytest
import torch

import oracle
from paper_2405_17381_amd import binding, synth

pytestmark = pytest.mark.gpu


def _all(xs, lam, **switches):
    with binding.debug(**switches):
        Q, K, V, dO = [x.cuda() for x in xs]
        O = binding.la_fwd(Q, K, V, lam)
        g = binding.la_bwd(Q, K, V, lam, dO)
        torch.cuda.synchronize()
    return [t.to(torch.float64).cpu().numpy() for t in (O,) + tuple(g)]


def _ref(xs, lam):
    q, k, v, g = [x.to(torch.float64).numpy() for x in xs]
    return (oracle.c_recurrence_fwd(q, k, v, lam),) + oracle.c_recurrence_bwd(q, k, v, lam, g)


def _rms(x, r):
    return float(np.linalg.norm(x - r) / np.linalg.norm(r))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lseg", [0, 128])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** 27, 2.0 ** 31, 1e-12])
def test_scales(d, lseg, scale):
    """The method is linear in V and dO: scaling one operand over the bound at which a workgroup leaves the
    split form (2^28) must not change the relative error.  fp32 products and sums of n = 300 terms: 1e-6."""
    lam = [1.0, 0.99, 0.5]
    w = synth.custom(1, 3, 300, d, lam, seed=61 + d, dtype="f32")
    Q, K, V, dO = synth.draw(w)
    xs = (Q, K, V * scale, dO)
    for nm, x, r in zip(("O", "dQ", "dK", "dV"), _all(xs, lam, lseg=lseg), _ref(xs, lam)):
        assert _rms(x, r) <= 1e-6, (nm, _rms(x, r))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 97, 300])
def test_no_less_exact_than_plain_fp32(d, n):
    """Error against 64-bit arithmetic, split form against the literal fp32 kernel."""
    lam = [1.0, 0.9999, 0.9]
    w = synth.custom(2, 3, n, d, lam, seed=71 + n + d, dtype="f32")
    xs = synth.draw(w)
    ref = _ref(xs, lam)
    for nm, x, p, r in zip(("O", "dQ", "dK", "dV"), _all(xs, lam), _all(xs, lam, f32_plain=1), ref):
        # (both sit on the rounding of the result, 2^-25 or 3e-8, when there is little to sum)
        assert _rms(x, r) <= 1.05 * _rms(p, r) + 1e-8, (nm, _rms(x, r), _rms(p, r))


@pytest.mark.parametrize("lseg", [0, 64])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38])
def test_values_out_of_the_split_range(lseg, value):
    """One infinite (NaN, or nearly overflowing) entry of V in the second block.  Everything that depends on
    it is not finite; nothing else is that plain fp32 arithmetic on the same 32-row blocks keeps finite, no
    infinity turns into NaN, and the finite results agree."""
    lam = [1.0, 0.9]
    w = synth.custom(1, 2, 160, 128, lam, seed=81, dtype="f32")
    xs = [x.clone() for x in synth.draw(w)]
    xs[2][0, :, 40, 5] = value
    got, plain = _all(xs, lam, lseg=lseg), _all(xs, lam, lseg=lseg, f32_plain=1)
    if not np.isfinite(value):
        assert not np.isfinite(got[0][:, :, 40:, 5]).any()           # O's column 5 from that row on
        assert not np.isfinite(got[1][:, :, 40:, :]).any()           # dQ from that row on
        assert not np.isfinite(got[2][:, :, 40, :]).any()            # dK of that row
    for nm, x, p in zip(("O", "dQ", "dK", "dV"), got, plain):
        f = np.isfinite(p)
        assert np.isfinite(x[f]).all(), nm
        assert np.isnan(p[np.isnan(x)]).all(), nm
        both = np.isinf(x) & np.isinf(p)
        assert np.array_equal(x[both], p[both]), nm
        assert _rms(x[f], p[f]) <= 1e-6, (nm, _rms(x[f], p[f]))


def test_carried_state_out_of_the_split_range():
    """A carried-in state beyond 2^87 sends the first segment to the fp32 instruction."""
    lam = [1.0, 0.9]
    w = synth.custom(1, 2, 100, 64, lam, seed=91, dtype="f32")
    Q, K, V, _ = [x.cuda() for x in synth.draw(w)]
    kv = torch.full((1, 2, 64, 64), 1e30, device="cuda")
    out = torch.empty_like(kv)
    O = binding.la_fwd_state(Q, K, V, lam, kv_in=kv, kv_out=out)
    with binding.debug(f32_plain=1):
        out2 = torch.empty_like(kv)
        P = binding.la_fwd_state(Q, K, V, lam, kv_in=kv, kv_out=out2)
    for a, b in ((O, P), (out, out2)):
        assert torch.isfinite(a).all()
        assert float((a.double() - b.double()).norm() / b.double().norm()) <= 1e-6
