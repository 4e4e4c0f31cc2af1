"""GPU parity of the far field where the binning changes its way: around the
largest call of the two-launch form, around the chunk of the local sort (a
bucket of one, two and many chunks), with few particles on many cells, on
cell counts that are no power of two, and with cells above the dense
threshold reduced by a P2M block or as listed items -- against the oracle at
the bounds of gpu_helpers.BOUNDS, and bitwise equal when called again."""
import numpy as np
import pytest

from gpu_helpers import assert_parity, gpu_far, oracle_cfg
from oracle import pmmm as opm
from paper_1409_5981_amd import inputs

pytestmark = pytest.mark.gpu


def _clustered(n, n_cells, boundary, share, seed, dtype, edge):
    """`share` of the particles in one cell off the mesh's centre, the rest
    uniform, in random order; masses."""
    rng = np.random.default_rng(seed)
    k = int(n * share)
    pos = rng.random((n, 3)) * n_cells
    pos[:k] = n_cells // 3 + rng.random((k, 3))
    pos = (pos[rng.permutation(n)] * edge).astype(dtype)
    top = dtype(n_cells * edge)
    pos = np.where(pos >= top, np.nextafter(top, dtype(0)), pos)
    q = (rng.random(n) / n).astype(dtype)
    return inputs.ParticleSet(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), q, n_cells, 2,
                              boundary, box=float(n_cells * edge))


@pytest.mark.parametrize("n,n_cells,boundary,share,prec", [
    (255, 8, "open", 0.6, "f32"), (256, 8, "periodic", 0.6, "f64"),
    (257, 8, "periodic", 0.9, "f32"), (3000, 6, "periodic", 0.5, "f32"),
    (32768, 16, "periodic", 0.5, "f32"), (32769, 16, "periodic", 0.5, "f32"),
    (32769, 16, "open", 0.0, "f64"), (5000, 32, "open", 0.7, "f32"),
    (40000, 8, "open", 0.95, "f32"), (40000, 8, "open", 0.0, "f64"),
    (33000, 5, "periodic", 0.3, "f32"), (140000, 32, "periodic", 0.2, "f32"),
    (1050000, 16, "open", 0.1, "f32"), (2100000, 32, "open", 0.05, "f32")])
def test_binning_forms(n, n_cells, boundary, share, prec):
    dt = np.float32 if prec == "f32" else np.float64
    ps = _clustered(n, n_cells, boundary, share, 70 + n % 97, dt, 1.0 / 32)
    res, plan = gpu_far(ps, precision=prec)
    ref = opm.far_field(ps.pos, ps.q.astype(np.float64), oracle_cfg(ps))
    assert_parity(res, ref.phi, ref.grad, prec, f"binning {n} on {n_cells}^3 {boundary} {prec}")
    again, _ = gpu_far(ps, precision=prec, plan=plan)
    assert all(np.array_equal(res[k], again[k]) for k in res)


def test_binning_batch_of_small_systems():
    """A batch small enough for the two-launch binning, with an empty system
    and dense cells; then the same batch with larger systems."""
    import torch
    from paper_1409_5981_amd._lib import Batch
    for sizes in ([300, 0, 2500, 77], [300, 9000, 0, 20000]):
        sets = [_clustered(n, 8, "periodic", 0.5, 80 + n, np.float32, 1.0 / 8) for n in sizes]
        batch = Batch([dict(n=8, p=2, boundary="periodic") for _ in sizes])
        off = np.concatenate([[0], np.cumsum(sizes)])
        t = [torch.from_numpy(np.concatenate([getattr(s, a) for s in sets])).cuda() for a in "xyzq"]
        out = batch.far(off, *t)
        torch.cuda.synchronize()
        for i, s in enumerate(sets):
            if s.n == 0:
                continue
            got = [o[off[i]:off[i + 1]].double().cpu().numpy() for o in out]
            ref = opm.far_field(s.pos, s.q.astype(np.float64), oracle_cfg(s))
            assert_parity({"phi": got[0], "grad": np.stack(got[1:], 1)}, ref.phi, ref.grad, "f32",
                          f"batch system of {s.n}")


@pytest.mark.parametrize("n,n_cells,p,boundary,share", [
    (40000, 8, 2, "open", 0.5), (100000, 8, 8, "periodic", 0.3), (140000, 5, 4, "periodic", 0.0)])
def test_fp64_cells_of_several_items(n, n_cells, p, boundary, share):
    """FP64 plans above the whole-cell size: the partial sums of a cell cut
    into items (one of 20000 or 30000 particles, or every cell of about 1100) hold 64
    bits too, so the field keeps the FP64 bounds."""
    ps = _clustered(n, n_cells, boundary, share, 90 + p, np.float64, 1.0 / 32)
    ps.p = p
    res, _ = gpu_far(ps, precision="f64")
    ref = opm.far_field(ps.pos, ps.q, oracle_cfg(ps))
    assert_parity(res, ref.phi, ref.grad, "f64", f"split cells {n} on {n_cells}^3 {boundary} p={p}")


# share x n particles in one bucket of the partition, which holds 8 cells of
# 16^3, 64 of 32^3 and 1024 of 128^3: 33 to 273 chunks (FP64: 50), whose
# histograms every chunk reads itself, and with more than 2^21 particles 282 to
# 560, which find them summed.
@pytest.mark.parametrize("n,n_cells,p,share,prec", [
    (140000, 32, 2, 0.95, "f32"), (290000, 32, 2, 0.91, "f32"), (1200000, 32, 2, 0.93, "f32"),
    (2400000, 32, 2, 0.955, "f32"), (2100000, 16, 2, 0.55, "f32"), (2100000, 128, 1, 0.6, "f32"),
    (215000, 32, 2, 0.95, "f64"), (2100000, 32, 2, 0.9, "f64")])
def test_binning_buckets_of_many_chunks(n, n_cells, p, share, prec):
    print(f"large bucket {n} on {n_cells}^3 p={p} {prec}", flush=True)
    dt = np.float32 if prec == "f32" else np.float64
    rng = np.random.default_rng(n)
    k = int(n * share)
    pos = rng.random((n, 3)) * n_cells
    cells = np.array({16: (8, 1, 1), 32: (32, 2, 1), 128: (128, 8, 1)}[n_cells])
    pos[:k] = np.array([0, 8, 10]) + rng.random((k, 3)) * cells
    pos = (pos[rng.permutation(n)] / n_cells).astype(dt)
    pos = np.where(pos >= dt(1), np.nextafter(dt(1), dt(0)), pos)
    q = (rng.random(n) / n).astype(dt)
    ps = inputs.ParticleSet(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), q, n_cells, p,
                            "periodic")
    res, plan = gpu_far(ps, precision=prec)
    ref = opm.far_field(ps.pos, ps.q.astype(np.float64), oracle_cfg(ps))
    assert_parity(res, ref.phi, ref.grad, prec, f"large bucket {n} on {n_cells}^3 {prec}")
    again, _ = gpu_far(ps, precision=prec, plan=plan)
    assert all(np.array_equal(res[x], again[x]) for x in res)


@pytest.mark.parametrize("n,run,prec", [(20000, 12100, "f32"), (9000, 8990, "f64")])
def test_small_binning_with_a_run_of_one_cell(n, run, prec):
    """The two-launch binning counts runs of one cell by whole waves: a run that
    ends inside a wave, then other cells."""
    dt = np.float32 if prec == "f32" else np.float64
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3)) * 16
    pos[:run] = np.array([5, 9, 3]) + rng.random((run, 3))
    pos = (pos / 16).astype(dt)
    q = (rng.random(n) / n).astype(dt)
    ps = inputs.ParticleSet(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), q, 16, 3, "periodic")
    res, plan = gpu_far(ps, precision=prec)
    ref = opm.far_field(ps.pos, ps.q.astype(np.float64), oracle_cfg(ps))
    assert_parity(res, ref.phi, ref.grad, prec, f"run of {run} in {n} {prec}")


@pytest.mark.parametrize("n,prec", [(20000, "f32"), (30000, "f32"), (30000, "f64")])
def test_p2m_of_a_three_cell_box(n, prec):
    """A box of 3 x 1 x 1 cells at c = 1: crowded cells reduced whole by a
    block, and above 8192 particles a cell as items."""
    dt = np.float32 if prec == "f32" else np.float64
    rng = np.random.default_rng(n)
    pos = (rng.random((n, 3)) * np.array([3, 1, 1]) / 32).astype(dt)
    top = (np.array([3, 1, 1]) / 32).astype(dt)
    pos = np.where(pos >= top, np.nextafter(top, dt(0)), pos)
    q = (rng.random(n) / n).astype(dt)
    ps = inputs.ParticleSet(pos[:, 0].copy(), pos[:, 1].copy(), pos[:, 2].copy(), q, 3, 5, "open",
                            box=3 / 32, shape=(3, 1, 1))
    res, _ = gpu_far(ps, precision=prec, cutoff=1)
    ref = opm.far_field(ps.pos, ps.q.astype(np.float64), oracle_cfg(ps, 1))
    # the middle cell's far field is zero: rounding of the convolution only
    end = (np.floor(ps.x.astype(np.float64) * 32) != 1)
    assert_parity({k: v[end] for k, v in res.items()}, ref.phi[end], ref.grad[end], prec,
                  f"three cells {n} {prec}")
