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
@pytest.mark.parametrize("grid,heads,d", [((4, 252), 17, 64), ((4, 252), 9, 128), ((20, 52), 5, 128), ((20, 52), 9, 64),
                                          ((60, 68), 4, 64), ((60, 68), 4, 128)])
def test_lists_of_many_rows(grid, heads, d, gate):
    """Two and four rows per workgroup, the last group short, in 63, 65 and 255
    blocks (test_lists has one row in 65, two in 255)."""
    w = _w(grid, gate=gate, batch=2, heads=heads, head_dim=d)
    (q, k, _), _ = inputs(w)
    assert _check(w, q, k) == 0


@pytest.mark.parametrize("heads,layers", [(2, 3), (5, 6)])
@pytest.mark.parametrize("d", [64, 128])
def test_shared_stack(d, heads, layers):
    """The layer driver's rows, one and two per workgroup (15 blocks: the last group of one)."""
    from paper_2605_15684_amd import ssba
    w = _w((24, 40), gate="topk_shared", tile=8, batch=3 * heads, heads=heads, head_dim=d, n_text=0)
    stack = [inputs(w.with_(seed=s)) for s in range(layers)]
    desc = gpu_desc(w, stack[0][1][0])
    keeps = [1 + 2 * l for l in range(layers)]
    index, _ = ssba.forward_layers([dict(q=q, k=k, v=v, out=torch.empty_like(q), keep=n)
                                    for (_, (q, k, v)), n in zip(stack, keeps)], desc)
    for l, (((q, k, _), _), n) in enumerate(zip(stack, keeps)):
        kw = oracle_kw(w)
        kw["shift"] = w.shift if l % 2 == 0 else (-w.shift[0], -w.shift[1])
        assert np.array_equal(index[l].cpu().numpy(), O.build_index(to64(q), to64(k), gate=w.gate, keep=n, **kw))


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
