"""The plane transforms up to 32 points against the oracle's far field at
gpu_helpers.BOUNDS: every size, both boundaries and precisions, with numbers
of planes (components x z) that do not divide into the planes of a block, and
batches large enough for the two-wave blocks, their last systems included."""
import numpy as np
import pytest

from gpu_helpers import assert_parity, oracle_cfg
from oracle import pmmm as opm
from paper_1409_5981_amd import inputs

pytestmark = pytest.mark.gpu


def _set(n_cells, p, boundary, n, seed, dtype=np.float32):
    rng = np.random.default_rng(seed)
    x, y, z = (rng.random(n).astype(dtype) for _ in range(3))
    return inputs.ParticleSet(x, y, z, inputs.neutral_pm1(rng, n, dtype), n_cells, p, boundary)


def _np(out):
    import torch
    torch.cuda.synchronize()
    return {"phi": out[0].double().cpu().numpy(),
            "grad": torch.stack(list(out[1:]), 1).double().cpu().numpy()}


# transforms of 4 (periodic only), 8, 16 and 32 points
@pytest.mark.parametrize("prec,dt", [("f32", np.float32), ("f64", np.float64)])
@pytest.mark.parametrize("boundary,n,p,cutoff", [
    ("periodic", 4, 5, 1), ("periodic", 8, 2, 2), ("periodic", 16, 4, 2), ("periodic", 32, 2, 2),
    ("open", 4, 3, 1), ("open", 8, 4, 2), ("open", 16, 6, 2)])
def test_planes_match_oracle(boundary, n, p, cutoff, prec, dt):
    import torch
    from paper_1409_5981_amd._lib import Plan
    print(f"planes {boundary} n={n} p={p} c={cutoff} {prec}", flush=True)
    ps = _set(n, p, boundary, 2000 + 20 * n, n + p, dt)
    plan = Plan(n, p, boundary, box=ps.box, cutoff=cutoff, precision=prec)
    t = [torch.from_numpy(np.ascontiguousarray(a, dtype=dt)).cuda() for a in (ps.x, ps.y, ps.z, ps.q)]
    res = _np(plan.far(*t))
    ref = opm.far_field(ps.pos, ps.q.astype(np.float64), oracle_cfg(ps, cutoff))
    assert_parity(res, ref.phi, ref.grad, prec, f"planes {boundary} n={n} p={p} {prec}")


@pytest.mark.parametrize("boundary,n,p,nsys", [("periodic", 8, 6, 67), ("periodic", 16, 5, 26),
                                               ("open", 16, 6, 11)])
def test_planes_of_large_batches(boundary, n, p, nsys):
    import torch
    from paper_1409_5981_amd._lib import Batch
    print(f"batch {boundary} n={n} p={p} systems={nsys}", flush=True)
    systems = [_set(n, p, boundary, 400 + 2 * i, 50 + i) for i in range(nsys)]
    offs = np.concatenate([[0], np.cumsum([s.n for s in systems])]).astype(np.int64)
    t = [torch.from_numpy(np.concatenate([getattr(s, a) for s in systems]).astype(np.float32)).cuda()
         for a in ("x", "y", "z", "q")]
    batch = Batch([{"n": n, "p": p, "boundary": boundary}] * nsys)
    res = _np(batch.far(offs, *t))
    batch.sync_status()
    for i in (0, nsys // 2, nsys - 1):
        s, a, b = systems[i], offs[i], offs[i + 1]
        ref = opm.far_field(s.pos, s.q.astype(np.float64), oracle_cfg(s))
        assert_parity({"phi": res["phi"][a:b], "grad": res["grad"][a:b]}, ref.phi, ref.grad, "f32",
                      f"system {i} of {nsys}")
