"""The top-k gate over block counts on both sides of its wave and row-group
edges (64, 256, 512 and 1024 blocks, groups of two and four rows with a
remainder), the per-head and the head-shared form, against the fp64 oracle:
lists bit-exact, ties and non-finite affinities included."""
import numpy as np
import pytest
import torch

from oracle import ssba_oracle as O
from paper_2605_15684_amd.inputs import workload_from

from _parity import gpu_desc, inputs, oracle_kw, to64

pytestmark = pytest.mark.gpu

GRIDS = [(4, 4), (4, 252), (32, 32), (20, 52), (60, 68), (64, 64), (4, 1028), (60, 92), (64, 128), (36, 228),
         (124, 132), (128, 128)]   # 1, 63, 64, 65, 255, 256, 257, 345, 512, 513, 1023, 1024 blocks of 4x4


def _w(grid, **kw):
    tb = grid[0] * grid[1] // 16
    base = dict(batch=1, heads=2, grid_h=grid[0], grid_w=grid[1], head_dim=64, tile=4, keep=max(1, tb // 7),
                shift=(1, 2), n_text=3)
    base.update(kw)
    return workload_from(**base)


def _check(w, q, k):
    from paper_2605_15684_amd import ssba
    qg, kg = q.to("cuda"), k.to("cuda")
    desc = gpu_desc(w, qg)
    index, scratch = ssba.build_index(qg, kg, desc)
    got = index.cpu().numpy()
    ref = O.build_index(to64(q), to64(k), gate=w.gate, keep=w.keep, **oracle_kw(w))
    assert np.array_equal(got, ref)
    return ssba.read_status(desc, scratch)


@pytest.mark.parametrize("gate", ["topk", "topk_shared"])
@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: f"{g[0] * g[1] // 16}")
def test_lists(grid, gate):
    d = 128 if grid[0] in (20, 64, 128) else 64
    w = _w(grid, gate=gate, head_dim=d, dtype="f32" if grid[0] == 60 else "bf16")
    (q, k, _), _ = inputs(w)
    assert _check(w, q, k) == 0


@pytest.mark.parametrize("gate", ["topk", "topk_shared"])
def test_lists_of_many_rows(gate):
    """63 blocks in 34 heads: two rows per workgroup, the last group of one."""
    w = _w((4, 252), gate=gate, batch=2, heads=17)
    (q, k, _), _ = inputs(w)
    assert _check(w, q, k) == 0


@pytest.mark.parametrize("grid", [(20, 52), (60, 92), (36, 228)], ids=["65", "345", "513"])
@pytest.mark.parametrize("keep", [1, 64, 65])
def test_equal_affinities_take_the_lowest_ids(grid, keep):
    """Every key block alike except one that ranks first and one last."""
    w = _w(grid, keep=keep, n_text=0)
    (q, k, _), _ = inputs(w)
    rows = O.frame_tiles(w.grid_h, w.grid_w, w.tile, *w.shift)
    q[:] = 1.0
    k[:] = 0.5
    k[:, :, torch.as_tensor(np.asarray(rows[40]))] = 2.0
    k[:, :, torch.as_tensor(np.asarray(rows[0]))] = -2.0
    assert _check(w, q, k) == 0


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
def test_non_finite_affinities_are_flagged(value):
    from paper_2605_15684_amd import _lib
    w = _w((60, 92), n_text=0)
    (q, k, _), _ = inputs(w)
    k[0, 1, 777, 5] = value
    from paper_2605_15684_amd import ssba
    qg, kg = q.to("cuda"), k.to("cuda")
    desc = gpu_desc(w, qg)
    index, scratch = ssba.build_index(qg, kg, desc)
    assert ssba.read_status(desc, scratch) == _lib.SSBA_ERR_NONFINITE
    ref = O.build_index(to64(q), to64(k), gate=w.gate, keep=w.keep, **oracle_kw(w))
    assert np.array_equal(index.cpu().numpy()[0, 0], ref[0, 0])
