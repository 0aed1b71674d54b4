"""Rows of any length and alignment through the step kernels: 16-byte tiles and
the float tiles after them (csrc/tiles.h).  On the CPU the tiles themselves,
compiled with g++ and walked; on the GPU every entry point at the tiles' edges
against the oracle and, bit for bit, against the same columns on aligned rows."""

import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2211_00889_amd import _lib
from tests._util import TOL, rel_err

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_tiles_cover_every_column_once(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "tile_cover")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-I",
                    os.path.join(ROOT, "paper_2211_00889_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "tile_cover.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout[-2000:]


# (P, ld): one column more and less than a 256-column tile and a 1024-column
# block; the last whole round of 32 neighbouring tiles (8192 columns) and one
# tile more; every remainder mod 4; rows that start on lines, on 16 bytes and on
# single floats.
EDGES = [(1, 1), (255, 255), (256, 257), (257, 288), (1023, 1023), (1024, 1028), (1025, 1025),
         (1027, 1056), (8191, 8191), (8192, 8193), (8193, 8224), (8449, 8449), (8446, 8446),
         (16640, 16644), (33284, 33284),
         # up to 35 rows of these are above and below the 128 MiB that the step reads
         # through the caches (the counts decide)
         (1_000_003, 1_000_003), (1_200_004, 1_200_128)]


@pytest.mark.gpu
@pytest.mark.parametrize("P,ld", EDGES)
def test_every_entry_point_at_the_tiles_edges(P, ld):
    torch = pytest.importorskip("torch")
    n, m, lr, mu = 5, 3, float(np.float32(0.1)), float(np.float32(0.9))
    rng = np.random.default_rng(P + ld)
    X = rng.standard_normal((n, P)).astype(np.float32)
    V = (0.1 * rng.standard_normal((n, P))).astype(np.float32)
    G = (0.03 * rng.standard_normal((n, m, P))).astype(np.float32)
    mask = (np.arange(m)[None, :] < rng.integers(1, m + 1, size=n)[:, None]).astype(np.uint8)
    counts = mask.sum(axis=1).astype(np.int32)
    W = _lib.w_ring(n)
    pad = np.float32(-7.5)

    def rows(a, stride):
        out = np.full(a.shape[:-1] + (stride,), pad, np.float32)
        out[..., :P] = a
        return torch.from_numpy(out).to("cuda:0")

    for order in (_lib.MIX_THEN_STEP, _lib.STEP_THEN_MIX):
        print(f"[case] step P={P} ld={ld} order={order}", flush=True)
        got = []
        for stride in (ld, (P + 127) // 128 * 128):  # the second: aligned rows
            Xd, Vd, Gd = rows(X, stride), rows(V, stride), rows(G, stride)
            _lib.step_strided(Xd, Vd, Gd, P, mask, W, 0.1, 0.9, order)
            torch.cuda.synchronize()
            got.append((Xd.cpu().numpy(), Vd.cpu().numpy()))
            assert (got[-1][0][:, P:] == pad).all() and (got[-1][1][:, P:] == pad).all()
        for a, b in zip(*got):
            assert np.array_equal(a[:, :P], b[:, :P])
        Xo, Vo = oracle.step.step(X, V, G, mask, W.astype(np.float64), lr, mu, order)
        assert rel_err(got[0][0][:, :P], Xo) <= TOL and rel_err(got[0][1][:, :P], Vo) <= TOL

    print(f"[case] server P={P} ld={ld}", flush=True)
    xd, Vd = torch.from_numpy(X[0].copy()).to("cuda:0"), rows(V, ld)
    _lib.step_server(xd, Vd, rows(G, ld), P, mask, 0.1, 0.9)
    torch.cuda.synchronize()
    xo, Vo = oracle.step.parameter_server_step(X[0], V, G, mask, lr, mu)
    assert rel_err(xd.cpu().numpy(), xo) <= TOL and rel_err(Vd.cpu().numpy()[:, :P], Vo) <= TOL

    print(f"[case] unfused P={P}", flush=True)  # contiguous rows
    Gbar = torch.full((n, P), pad, dtype=torch.float32, device="cuda:0")
    Xd, Vd, Yd = rows(X, P), rows(V, P), torch.empty((n, P), dtype=torch.float32, device="cuda:0")
    _lib.accumulate(rows(G, P), mask, Gbar)
    _lib.mix(Xd, W, Yd)
    _lib.update(Yd, Vd, Gbar, counts, m, 0.1, 0.9)
    torch.cuda.synchronize()
    Xo, Vo = oracle.step.step(X, V, G, mask, W.astype(np.float64), lr, mu, _lib.MIX_THEN_STEP)
    assert rel_err(Gbar.cpu().numpy(), oracle.step.accumulate(G, mask)) <= TOL
    assert rel_err(Yd.cpu().numpy(), Xo) <= TOL and rel_err(Vd.cpu().numpy(), Vo) <= TOL
