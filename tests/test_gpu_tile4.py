"""bf16 attention in 4x4 blocks (one wave per query block): kept lists that end
at, just before and just after the 64 entries in the lanes, odd and even unit
counts, text tails on both sides of 16 rows, groups of four blocks with a
remainder, both layouts, against the fp64 oracle (2e-2 max-abs, as every bf16
parity test; every row)."""
import numpy as np
import pytest
import torch

from oracle import ssba_oracle as O
from paper_2605_15684_amd.inputs import workload_from

from _parity import BF16_TOL, gpu_desc, growing_inputs, inputs, oracle_index, oracle_kw, to64


def _w(**kw):
    base = dict(batch=1, heads=1, grid_h=36, grid_w=40, head_dim=64, tile=4, keep=9, shift=(2, 2))
    base.update(kw)
    return workload_from(**base)


CASES = [
    _w(grid_h=4, grid_w=4, keep=1), _w(grid_h=4, grid_w=8, keep=1, n_text=1, head_dim=128),
    _w(keep=1), _w(keep=63), _w(keep=64, n_text=15), _w(keep=65, n_text=16), _w(keep=90, n_text=17),
    _w(keep=8, n_text=33, heads=3, batch=2, shift=(-1, 3)), _w(keep=64, n_text=77, head_dim=128),
    _w(grid_h=52, grid_w=44, keep=129, heads=2), _w(grid_h=52, grid_w=44, keep=143, head_dim=128, shift=(3, -2)),
]


def _ids(w):
    return f"{w.grid_h}x{w.grid_w}-B{w.batch}H{w.heads}-D{w.head_dim}-k{w.keep}-t{w.n_text}"


def _forward(w, qg, kg, vg, idx):
    from paper_2605_15684_amd import ssba
    out = ssba.forward(qg, kg, vg, torch.from_numpy(idx).to("cuda"), gpu_desc(w, qg))
    torch.cuda.synchronize()
    return out.float().cpu().double().numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["topk", "uneven", "bthd"])
@pytest.mark.parametrize("w", CASES, ids=_ids)
def test_tile4(w, form):
    (q, k, v), gpu = inputs(w)
    idx = oracle_index(w, q, k)
    if form == "uneven":   # block i keeps the first 1 + 7 i mod keep entries (a softmax over no keys has no reference)
        tb = w.n_tiles
        idx = idx.copy()
        idx.reshape(-1, tb, tb + 1)[:, :, 0] = 1 + 7 * np.arange(tb) % w.keep
    if form == "bthd":     # the [B, T, H, D] layout of a projection's output
        gpu = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in gpu]
    got = _forward(w, *gpu, idx)
    ref = O.attention(to64(q), to64(k), to64(v), idx, **oracle_kw(w))
    assert np.isfinite(got).all()
    assert float(np.abs(got - ref).max()) <= BF16_TOL


@pytest.mark.gpu
@pytest.mark.parametrize("w", [_w(keep=90, n_text=5), _w(keep=90, n_text=40, head_dim=128)], ids=_ids)
def test_scores_that_grow(w):
    """A new maximum in half of the rows after 1, 7, 30 and 64 blocks; a text group's waves end at different ones."""
    (q, k, v), idx, bound = growing_inputs(w, (1, 7, 30, 64))
    got = _forward(w, *(t.to("cuda") for t in (q, k, v)), idx)
    ref = O.attention(to64(q), to64(k), to64(v), idx, **oracle_kw(w))
    assert (np.abs(got - ref) <= bound).all()


@pytest.mark.gpu
def test_masked_keys_add_nothing():
    """Ids past the grid and the rows after a text tail are not seen, whatever they hold."""
    w = _w(keep=66, n_text=3)
    (q, k, v), (qg, kg, vg) = inputs(w)
    idx = oracle_index(w, q, k).copy()
    frame = O.frame_tiles(w.grid_h, w.grid_w, w.tile, *w.shift)
    vg[0, 0, w.n_text:w.n_text + 16] = float("nan")    # the rows that a unit of 16 would run into
    vg[0, 0, w.n_text + int(frame[0][0])] = float("inf")
    bad = {t for t in range(w.n_tiles) if (np.asarray(frame[t]) < 16).any()} | {0}
    ok = [t for t in range(w.n_tiles) if t not in bad]
    idx[0, 0, :, 0] = 66
    idx[0, 0, :, 1:67] = np.resize(np.array(ok), 66)
    idx[0, 0, :, 7] = -3
    idx[0, 0, :, 65] = 5000
    got = _forward(w, qg, kg, vg, idx)
    assert np.isfinite(got[0, 0, w.n_text:]).all()
    want = idx.copy()                                  # the same without the two ids
    want[0, 0, :, 0] = 64
    want[0, 0, :, 1:65] = np.delete(idx[0, 0, :, 1:67], [6, 64], axis=1)
    v2 = vg.cpu().clone()
    v2[~torch.isfinite(v2)] = 0
    ref = O.attention(to64(q), to64(k), to64(v2), want, **oracle_kw(w))
    assert float(np.abs(got[0, 0, w.n_text:] - ref[0, 0, w.n_text:]).max()) <= BF16_TOL
