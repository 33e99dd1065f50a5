"""The fp32 attention kernel at the edges of its decomposition, against the
fp64 oracle (1e-5 max-abs, as every fp32 parity test): 4x4 block counts that
do not fill a workgroup's four waves, lists longer than 64 blocks, text tails
around its 16-row groups and 16-key runs, dense rows that do not fill a 64-row
group, and tensors that are only 4-byte aligned."""
import numpy as np
import pytest
import torch

from oracle import ssba_oracle as O
from paper_2605_15684_amd.inputs import workload_from

from _parity import F32_TOL, gpu_desc, inputs, oracle_index, oracle_kw, run_gpu, to64

pytestmark = pytest.mark.gpu


def _w(**kw):
    base = dict(batch=1, heads=1, grid_h=16, grid_w=16, head_dim=64, tile=4, keep=3, shift=(2, 2), dtype="f32",
                sigma_img=1.0)
    base.update(kw)
    return workload_from(**base)


CASES = [
    _w(grid_h=4, grid_w=4, keep=1), _w(grid_h=4, grid_w=20, keep=5), _w(grid_h=12, grid_w=12, keep=9, n_text=1),
    _w(heads=8, n_text=15), _w(n_text=16, head_dim=128), _w(n_text=17, keep=16), _w(n_text=65, shift=(-1, 7)),
    _w(grid_h=40, grid_w=36, keep=80, n_text=5),                       # 90 blocks, lists of 80
    _w(grid_h=72, grid_w=72, tile=8, keep=70, shift=(-4, 4)),          # 81 blocks, lists of 70
    _w(grid_h=24, grid_w=40, tile=8, keep=4, n_text=33, shift=(3, 5), batch=2, heads=3),
    _w(grid_h=24, grid_w=8, tile=8, keep=2, n_text=63, head_dim=128),
    _w(grid_h=32, grid_w=48, tile=16, keep=3, n_text=64, shift=(8, -8)),
    _w(grid_h=32, grid_w=16, tile=16, keep=1, head_dim=128, n_text=3),
]


def _ids(w):
    return f"{w.grid_h}x{w.grid_w}-D{w.head_dim}-b{w.tile}-k{w.keep}-t{w.n_text}"


@pytest.mark.parametrize("w", CASES, ids=_ids)
def test_lists(w):
    (q, k, v), (qg, kg, vg) = inputs(w)
    index, out = run_gpu(w, qg, kg, vg)
    assert np.array_equal(index, oracle_index(w, q, k))
    ref = O.attention(to64(q), to64(k), to64(v), index, **oracle_kw(w))
    assert float(np.abs(to64(out) - ref).max()) <= F32_TOL


@pytest.mark.parametrize("w", [_w(grid_h=4, grid_w=4, n_text=1), _w(grid_h=4, grid_w=16, head_dim=128),
                               _w(n_text=1), _w(n_text=63, head_dim=128, heads=8)], ids=_ids)
def test_dense(w):
    (q, k, v), (qg, kg, vg) = inputs(w)
    _, out = run_gpu(w, qg, kg, vg, dense=True)
    idx = O.build_index(to64(q), to64(k), gate="dense", **oracle_kw(w))
    ref = O.attention(to64(q), to64(k), to64(v), idx, **oracle_kw(w))
    assert float(np.abs(to64(out) - ref).max()) <= F32_TOL


@pytest.mark.parametrize("w", [_w(n_text=5), _w(grid_h=24, grid_w=16, tile=8, n_text=7, heads=2),
                               _w(tile=8, head_dim=128, n_text=2)], ids=_ids)
def test_four_byte_alignment(w):
    """Rows of D + 3 floats from an odd element on: the same bits as the aligned tensors."""
    from paper_2605_15684_amd import ssba
    _, gpu = inputs(w)
    row = w.head_dim + 3
    sh = w.seq_len * row + 1
    strides = (w.heads * sh, sh, row, 1)

    def odd(t):
        buf = torch.full((1 + w.batch * w.heads * sh,), float("nan"), device="cuda")
        view = torch.as_strided(buf, t.shape, strides, 1)
        return view.copy_(t)

    qo, ko, vo = (odd(t) for t in gpu)
    out = odd(torch.zeros_like(gpu[0]))
    index, _ = ssba.build_index(qo, ko, gpu_desc(w, qo))
    ssba.forward(qo, ko, vo, index, gpu_desc(w, qo), out=out)
    torch.cuda.synchronize()
    want_index, want = run_gpu(w, *gpu)
    assert np.array_equal(index.cpu().numpy(), want_index)
    assert torch.equal(out, want)


def test_nan_stays_where_it_is():
    """A NaN value row reaches the queries that see its key and no others;
    keys that do not exist (a ragged text tail, an id past the grid) add none."""
    from paper_2605_15684_amd import ssba
    w = _w(grid_h=16, grid_w=16, tile=8, keep=2, n_text=3, shift=(0, 0))
    _, (q, k, v) = inputs(w)
    desc = gpu_desc(w, q)
    index, _ = ssba.build_index(q, k, desc)
    v = v.clone()
    v[0, 0, w.n_text] = float("nan")                      # image token (0, 0): block 0
    v[0, 0, w.seq_len - 1] = float("inf")                 # the last row: block 3
    index[0, 0, 1] = torch.tensor([2, 1, 77, -1, -1], dtype=torch.int32, device="cuda")
    out = ssba.forward(q, k, v, index, desc)
    torch.cuda.synchronize()
    lists = index.cpu().numpy()[0, 0]
    frame = O.frame_tiles(w.grid_h, w.grid_w, w.tile, 0, 0)
    for i in range(w.n_tiles):
        ids = set(lists[i, 1:1 + lists[i, 0]])
        rows = out[0, 0, torch.from_numpy(w.n_text + frame[i]).cuda()]
        assert bool(torch.isfinite(rows).all()) == (not ids & {0, 3})
    assert bool(torch.isnan(out[0, 0, :w.n_text]).all())
