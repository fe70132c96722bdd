"""pic_sync on sections of every length and alignment: it writes the caller's
cells four slots at a time where a whole aligned group lies in a tile's
section, and one by one at the section's ends.

Sparse plasmas (0 to 9 particles a tile, so sections start at every residue
of 4, some empty, some inside one group) and a dense one, with the caller's
cell array at each 4-byte alignment, its neighbours guarded.  The cells after
a step are the canonical sort of the cells the same step's push left (the
oracle's permutation of the eager twin's), bit for bit."""
import numpy as np
import pytest

import oracle
from _parity import flush

pytestmark = pytest.mark.gpu

DX = DY = 0.1
DT = 0.07


def _load(nx, ny, tile, most, seed):
    rng = np.random.default_rng(seed)
    ix, iy = [], []
    for ty in range(ny // tile):
        for tx in range(nx // tile):
            k = int(rng.integers(0, most + 1))
            ix.append(tx * tile + rng.integers(0, tile, k))
            iy.append(ty * tile + rng.integers(0, tile, k))
    st = {"ix": np.concatenate(ix).astype(np.int32), "iy": np.concatenate(iy).astype(np.int32)}
    n = st["ix"].size
    for f in ("x", "y"):
        st[f] = rng.uniform(0, 0.999, n).astype(np.float32)
    for f in ("ux", "uy", "uz"):
        st[f] = rng.normal(0, 0.8, n).astype(np.float32)
    return st


@pytest.mark.parametrize("tile,most,shift", [(8, 9, 1), (16, 9, 2), (16, 3000, 3), (32, 9, 0), (32, 9000, 1)])
def test_sync_writes_every_cell_and_nothing_else(tile, most, shift):
    import torch
    from paper_2501_14795_amd import Sim, _lib
    from paper_2501_14795_amd.sim import _Buffers
    nx, ny = 3 * tile, 5 * tile
    st = _load(nx, ny, tile, most, tile + most)
    n = st["ix"].size
    eager = Sim(nx, ny, DX, DY, DT, tile, [(-1.0, -0.1, st)])
    buf = _Buffers(nx, ny, DX, DY, DT, tile, [(-1.0, -0.1, st)])
    guarded = torch.full((n + 8,), -7, dtype=torch.int32, device="cuda")
    cell = guarded[4 + shift:4 + shift + n]   # 4-byte aligned, shift mod 4 of 16 bytes
    cell.copy_(buf.particles[0]["cell"])
    buf.bufs.sp[0].cell = cell.data_ptr()
    first = (cell.data_ptr() - guarded.data_ptr()) // 4
    stream = torch.cuda.current_stream().cuda_stream
    torch.cuda.synchronize()
    handle = _lib.pic_init(buf.cfg, buf.bufs, stream)
    for step in range(3):
        eager.push_deposit()
        pushed = eager.state(0)
        eager.sort()
        eager.field_advance()
        off, src = oracle.sort_canonical(nx, ny, tile, pushed["ix"], pushed["iy"])
        _lib.pic_step(handle, stream)
        _lib.pic_sync(handle, stream)
        torch.cuda.synchronize()
        got = guarded.cpu().numpy()
        assert np.array_equal(got[first:first + n], pushed["cell"][src]), step
        assert (np.delete(got, np.arange(first, first + n)) == -7).all(), step
        assert np.array_equal(buf.particles[0]["x"].cpu().numpy(), pushed["x"][src]), step
    assert _lib.pic_check(handle, stream) == 0 and eager.check() == 0
    flush(f"T{tile}, up to {most} particles a tile ({n}), cells at {first % 4} mod 4: equal over 3 steps")
    _lib.pic_destroy(handle)
    eager.close()
