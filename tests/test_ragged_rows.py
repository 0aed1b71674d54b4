"""Rows of any length and alignment through the step kernels: 16-byte tiles and
the float tiles after them (csrc/tiles.h).  On the CPU the tiles themselves,
compiled with g++ and walked; on the GPU every entry point at the tiles' edges
against the oracle and, bit for bit, against the same columns on aligned rows; and
every form of the fused step (whole rows of four columns or ragged ones, read through
the caches or streamed), bit for bit against the same columns in windows that all
take one form."""

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
         (16640, 16644), (33284, 33284)]


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
        for stride in (ld, (P + 255) // 128 * 128):  # the second: aligned rows, another stride
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


# (n, m, P, ld, whole rows of four columns, for the server too, streamed).  The counts
# follow from the case's seed, and the test checks the form they give: n = 5, m = 3
# moves 25 to 35 rows, the server 17 to 27; n = 9, m = 2 45 to 54 and 29 to 38.
FORMS = [
    (5, 3, 900_003, 900_003, False, False, False),
    (5, 3, 1_400_003, 1_400_003, False, False, True),
    (5, 3, 1_400_002, 1_400_005, False, False, True),
    (5, 3, 1_400_004, 1_400_005, False, False, True),
    (5, 3, 1_400_004, 1_400_004, True, True, True),
    (5, 3, 900_004, 900_004, True, True, False),
    (5, 3, 1_400_004, 1_400_032, True, True, True),
    (9, 2, 800_004, 800_004, False, True, True),
    (9, 2, 600_004, 600_004, False, True, False),
    (16, 24, 450_004, 450_004, False, False, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,m,P,ld,whole,server_whole,streamed", FORMS)
def test_every_form_of_the_step(n, m, P, ld, whole, server_whole, streamed):
    """Columns never interact, so windows of them on line-aligned rows, small enough to
    go through the caches, give the reference for any form.  The forms that the case
    names are checked against csrc/tiles.h and step.hip's rules first."""
    torch = pytest.importorskip("torch")
    rng = np.random.default_rng(P + ld + n)
    mask = (np.arange(m)[None, :] < rng.integers(1, m + 1, size=n)[:, None]).astype(np.uint8)
    rows, c = int(mask.sum()) + 4 * n, int(mask.sum())
    lines, sixteen = P % 4 == 0 and ld % 32 == 0, P % 4 == 0 and ld % 4 == 0
    assert whole == (lines or (sixteen and rows < 36))
    assert server_whole == (lines or (sixteen and c + 2 * n + 2 < 124))
    assert streamed == (4 * P * rows > 128 << 20)
    g = torch.Generator(device="cuda:0").manual_seed(P + n)

    def rnd(*shape):
        return torch.empty(shape, dtype=torch.float32, device="cuda:0").normal_(generator=g)

    X, V, G = rnd(n, ld), rnd(n, ld), rnd(n, m, ld)
    W = _lib.w_ring(n)

    def window(a, c0, c1):  # line-aligned rows of whole lines, whatever lies past the columns
        out = torch.zeros(a.shape[:-1] + ((c1 - c0 + 31) // 32 * 32,), dtype=torch.float32, device="cuda:0")
        out[..., :c1 - c0] = a[..., c0:c1]
        return out

    def run(step, x, v):
        """step(x, v, G, columns) on the whole rows and in windows; both ways' x and v."""
        got = [x.clone(), v.clone()]
        step(*got, G, P)
        want = [x.clone(), v.clone()]
        width = (128 << 20) // (4 * rows) // 32 * 32
        for c0 in range(0, P, width):
            c1 = min(P, c0 + width)
            part = [window(x, c0, c1), window(v, c0, c1)]
            step(*part, window(G, c0, c1), part[0].shape[-1])
            for a, b in zip(want, part):
                a[..., c0:c1] = b[..., :c1 - c0]
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b)  # the columns past P too: never written

    for order in (_lib.MIX_THEN_STEP, _lib.STEP_THEN_MIX):
        print(f"[case] form n={n} m={m} P={P} ld={ld} order={order}", flush=True)
        run(lambda x, v, gg, cols: _lib.step_strided(x, v, gg, cols, mask, W, 0.1, 0.9, order), X, V)
    print(f"[case] form n={n} m={m} P={P} ld={ld} server", flush=True)
    run(lambda x, v, gg, cols: _lib.step_server(x, v, gg, cols, mask, 0.1, 0.9), X[0].clone(), V)
