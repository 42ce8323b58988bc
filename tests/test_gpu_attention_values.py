"""Fused attention of narrow heads (below 128) on values that a stage with
random weights does not meet, against the fp64 oracle."""
import numpy as np
import pytest

import oracle
from synth import gen_params, get_config
from tests.conftest import rel_l2
from tests.gpu_harness import log, run_gpu, takes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


# The grid forms of the fused kernels on 256 compute units: workgroups of 32
# rows, pairs of query blocks, query blocks (causal and bidirectional).
FORMS = {
    "split": dict(heads=4, seq=328, micro_batch=1, causal=True),
    "paired": dict(heads=16, seq=1000, micro_batch=4, causal=True),
    "block": dict(heads=10, seq=1000, micro_batch=4, causal=True),
    "bidirectional": dict(heads=4, seq=1128, micro_batch=4, causal=False),
}


def narrow(form, d):
    f = FORMS[form]
    cfg = get_config("small_bf16").with_(layers=1, hidden=d * f["heads"], ffn=2 * d * f["heads"], n_mb=1, rerouted=(), **f)
    takes(cfg, attention="block" if form == "bidirectional" else form)
    return cfg


@pytest.mark.parametrize("d", [32, 64, 96])
@pytest.mark.parametrize("form", list(FORMS))
def test_common_component_of_values(form, d):
    """Values and keys with a large common component: dP - Dv, the part of dP
    that tells the keys apart, is then far smaller than Dv = rowsum(dO o O), and
    an error of Dv reaches dQ as a multiple of the keys' common component.

    Bound on the error of dQ relative to dQ (rms), with a value's common part 3,
    its varying part v = 0.02 sqrt(h) and the keys' common part 3 v:
    - values round to bf16, which the oracle does not do: spacing 2^-6 at 3, so
      2^-6 / sqrt(12) of v;
    - probabilities round to bf16 (2^-9 / sqrt(3)) before they multiply V, so a
      row of them does not sum to 1 exactly, and dP - Dv keeps that share of the
      values' common part, which sums up over the keys' common part: 3 * 3 / v
      of 2^-9 / sqrt(3);
    - dS rounds to bf16 and sums up over the keys' common part: 3 * 2^-9.
    One and a half times their sum.  (O rounded in Dv: 0.19 to 0.64 in place of
    0.02 to 0.04.)"""
    cfg = narrow(form, d)
    h = cfg.hidden
    v = cfg.w_std * np.sqrt(h)
    bound = 1.5 * (2.0 ** -6 / np.sqrt(12) / v + 9 / v * 2.0 ** -9 / np.sqrt(3) + 3 * 2.0 ** -9)
    log(f"[values] {form} d={d} h={h} s={cfg.seq} b={cfg.micro_batch}: bound {bound:.2e}")
    params = gen_params(cfg)
    params[0][3][h:2 * h] = 3 * v
    params[0][3][2 * h:] = 3
    g = run_gpu(cfg, params=params)
    o = oracle.run_oplist(cfg, params=params)
    e = rel_l2(g.grads[0][2][:, :h], o.grads[0][2][:, :h])
    log(f"[values] {form} d={d}: rel-L2 of the query weights' gradient {e:.2e}")
    assert e < bound, (e, bound)
    for mb in o.y:
        assert rel_l2(g.y[mb], o.y[mb]) < 2e-2 and rel_l2(g.dx[mb], o.dx[mb]) < 2e-2


@pytest.mark.parametrize("scale", [2.0 ** 10, -2.0 ** 52])
@pytest.mark.parametrize("form", list(FORMS))
def test_scores_of_any_size(form, scale):
    """Queries and keys that are one constant each (weights zero, biases exact
    in bf16), so that every key of a row has the same score, 8 scale^2 after the
    scaling at d = 64, and the softmax is uniform whatever that score is.  Scores
    of 8e6, which fp32 holds to one part in 2^24 only, and of -1.6e32, whose
    exponentials have no range: the output, the input gradient and the value
    weights' gradient (dV = P^T dO) stay within the bar of bf16 stages."""
    cfg = narrow(form, 64)
    h = cfg.hidden
    params = gen_params(cfg)
    params[0][2][:, :2 * h] = 0
    params[0][3][:h] = abs(scale)
    params[0][3][h:2 * h] = scale
    log(f"[values] {form} h={h} s={cfg.seq} b={cfg.micro_batch}: queries and keys of {scale:.1e}")
    g = run_gpu(cfg, params=params)
    o = oracle.run_oplist(cfg, params=params)
    e = {"grad": rel_l2(g.grads[0][2][:, 2 * h:], o.grads[0][2][:, 2 * h:])}
    for mb in o.y:
        e["y"], e["dx"] = rel_l2(g.y[mb], o.y[mb]), rel_l2(g.dx[mb], o.dx[mb])
    log(f"[values] {form} {scale:.1e}: rel-L2 of the value weights' gradient, y, dx {e}")
    assert all(v < 2e-2 for v in e.values()), e
