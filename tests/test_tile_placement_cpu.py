"""Tile placement of the multi-step kernels (host-side checks of the index rules the kernels
use; no GPU).

Two steps per launch with walls through the boundary nodes: in the second step a boundary node
rebuilds its populations by non-equilibrium extrapolation from its neighbours f and ff along the
inward normal (the inward diagonal at a corner), whose own pre-collision populations are pulled
from the first step's results held in LDS for the tile and a one-node halo ring.  The kernel
places the last tile of each row and column against the far wall, x0 = min(t W, nx - W),
y0 = min(t H, ny - H).  The first tests check, for every tile of many lattice shapes, that every
LDS read of that rule stays in the tile's region and lands on a node the first step computed,
and that a tile the kernel treats as interior holds no boundary node in its region.  The last
ones check the region bookkeeping of three steps per launch and that the order in which a launch
visits its tiles (row by row or in vertical strips) covers every tile once.
"""
import numpy as np
import pytest

# two-step tiles: 64 x 8 (FP32, FP16 storage) and 32 x 8 (FP64)
TILES = [(64, 8), (32, 8)]


def _check_lattice(W, H, nx, ny, perx, pery):
    RW, RH = W + 2, H + 2
    ntx, nty = -(-nx // W), -(-ny // H)

    def boundary(X, Y):
        return (not perx and X in (0, nx - 1)) or (not pery and Y in (0, ny - 1))

    for ty in range(nty):
        for tx in range(ntx):
            x0, y0 = min(tx * W, nx - W), min(ty * H, ny - H)
            assert x0 >= 0 and y0 >= 0
            interior = x0 >= 2 and x0 + W + 1 <= nx - 1 and y0 >= 2 and y0 + H + 1 <= ny - 1
            if interior:
                for lx in range(RW):
                    for ly in range(RH):
                        X, Y = x0 - 1 + lx, y0 - 1 + ly
                        assert 0 <= X < nx and 0 <= Y < ny and not boundary(X, Y)
                continue

            def computed(lx, ly):
                # the first step skips region nodes beyond a wall; across a periodic side it
                # computes the wrapped node
                X, Y = x0 - 1 + lx, y0 - 1 + ly
                return (perx or 0 <= X < nx) and (pery or 0 <= Y < ny)

            for t in range(W * H):
                x, y = x0 + t % W, y0 + t // W
                assert x < nx and y < ny
                bx = not perx and x in (0, nx - 1)
                by = not pery and y in (0, ny - 1)
                if not (bx or by):
                    continue
                dx = (1 if x == 0 else -1) if bx else 0
                dy = (1 if y == 0 else -1) if by else 0
                for k in (1, 2):                       # f and ff
                    px, py = x + k * dx, y + k * dy
                    assert 0 <= px < nx and 0 <= py < ny
                    cx, cy = px - x0 + 1, py - y0 + 1
                    for ex in (-1, 0, 1):              # the node and its eight upstream nodes
                        for ey in (-1, 0, 1):
                            lx, ly = cx + ex, cy + ey
                            assert 0 <= lx < RW and 0 <= ly < RH, (W, H, nx, ny, x, y, k)
                            assert computed(lx, ly), (W, H, nx, ny, perx, pery, x, y, lx, ly)


@pytest.mark.parametrize("W,H", TILES)
def test_boundary_rule_reads_stay_in_the_tile_region(W, H):
    sizes_x = list(range(W, W + 9)) + list(range(2 * W - 3, 2 * W + 4)) + [3 * W + 1, 100, 129, 200]
    sizes_y = list(range(H, H + 10)) + [2 * H - 1, 2 * H + 1, 37, 70, 129, 257]
    n = 0
    for nx in sizes_x:
        for ny in sizes_y:
            for perx, pery in ((False, False), (True, False), (False, True)):
                _check_lattice(W, H, nx, ny, perx, pery)
                n += 1
    assert n == len(sizes_x) * len(sizes_y) * 3


def test_a_misplaced_last_tile_is_caught():
    """The same check with the last tile left ragged (x0 = t W) fails on a lattice whose last
    column of tiles is narrower than three nodes."""
    W, H, nx, ny = 64, 8, 66, 16
    ragged_x0 = (nx // W) * W                      # 64: the tile holds columns 64, 65 only
    px = (nx - 1) - 2                              # ff of the right-wall node
    assert px - ragged_x0 + 1 - 1 < 0              # its upstream column falls outside the region
    _check_lattice(W, H, nx, ny, False, False)     # the placement the kernel uses passes


# ---------------------------------------------------------------- three steps per launch
# The three-step kernel keeps a two-node halo: step one computes the (W + 4) x (H + 4) region,
# step two the inner (W + 2) x (H + 2) region in place, step three the tile.  Each region node
# belongs to one thread: its tile node, an inner-ring node (threads [0, N1)) or an outer-ring
# node (threads [N1, N1 + N2)).  The check below walks, for every tile, every node the third
# step stores, the region nodes its pulls read in step two and theirs in step one, and checks
# that each was computed by the previous step and holds a node of the domain (across a periodic
# side: the wrapped one).
def _check_three_step(W, H, nx, ny, perx, pery):
    RW, RH = W + 4, H + 4
    N1 = 2 * (W + 2) + 2 * H
    N2 = 2 * RW + 2 * (H + 2)
    assert N1 + N2 <= W * H
    own = {(t % W + 2, t // W + 2) for t in range(W * H)}
    r1, r2 = set(), set()
    for t in range(N1 + N2):
        if t < N1:
            if t < 2 * (W + 2):
                rx, ry = 1 + t % (W + 2), (1 if t < W + 2 else RH - 2)
            else:
                q = t - 2 * (W + 2)
                rx, ry = (1 if q < H else RW - 2), 2 + q % H
            assert (rx, ry) not in r1
            r1.add((rx, ry))
        else:
            k = t - N1
            if k < 2 * RW:
                rx, ry = k % RW, (0 if k < RW else RH - 1)
            else:
                q = k - 2 * RW
                rx, ry = (0 if q < H + 2 else RW - 1), 1 + q % (H + 2)
            assert (rx, ry) not in r2
            r2.add((rx, ry))
    assert not (own & r1) and not (own & r2) and not (r1 & r2)
    assert own | r1 | r2 == {(x, y) for x in range(RW) for y in range(RH)}
    inner = own | r1
    assert inner == {(x, y) for x in range(1, RW - 1) for y in range(1, RH - 1)}
    ntx, nty = -(-nx // W), -(-ny // H)
    for ty_ in range(nty):
        for tx_ in range(ntx):
            x0, y0 = tx_ * W, ty_ * H
            interior = x0 >= 3 and x0 + W + 2 <= nx - 1 and y0 >= 3 and y0 + H + 2 <= ny - 1
            def locate(lx, ly):
                X, Y = x0 - 2 + lx, y0 - 2 + ly
                if not (0 <= X < nx):
                    if not perx:
                        return None
                    X = X + nx if X < 0 else X - nx
                if not (0 <= Y < ny):
                    if not pery:
                        return None
                    Y = Y + ny if Y < 0 else Y - ny
                return X, Y
            if interior:
                for lx in range(RW):
                    for ly in range(RH):
                        X, Y = x0 - 2 + lx, y0 - 2 + ly
                        assert 1 <= X <= nx - 2 and 1 <= Y <= ny - 2
            def valid(p):
                q = locate(*p)
                return q is not None and 0 <= q[0] < nx and 0 <= q[1] < ny
            step1 = {p for p in own | r1 | r2 if locate(*p) is not None}
            step2 = {p for p in inner if locate(*p) is not None}
            def sources(p):
                X, Y = locate(*p)
                out = []
                for ex in (-1, 0, 1):
                    for ey in (-1, 0, 1):
                        okx = (ex == 0) or perx or (0 <= X - ex < nx)
                        oky = (ey == 0) or pery or (0 <= Y - ey < ny)
                        if okx and oky:
                            out.append((p[0] - ex, p[1] - ey))
                return out
            for p in own:
                X, Y = x0 + p[0] - 2, y0 + p[1] - 2
                if X < nx and Y < ny:
                    for q in sources(p):                 # step three reads step two at q
                        assert q in step2 and valid(q), (p, q)
                        # the wrapped node at q pulls the same neighbours as the real one
                        for r_ in sources(q):            # step two at q reads step one at r_
                            assert r_ in step1 and valid(r_), (p, q, r_)


@pytest.mark.parametrize("W,H", TILES + [(64, 12)])
def test_three_step_rings_cover_the_region_and_feed_every_stored_node(W, H):
    for nx in (3, 5, 65, 70, 129):
        for ny in (3, 5, 9, 37):
            for perx, pery in ((False, False), (True, False), (False, True), (True, True)):
                _check_three_step(W, H, nx, ny, perx, pery)


def _tile_of(b, ntx, nty, sw):
    """The kernels' tile order: row by row (sw = 0, or sw >= ntx), or vertical strips of sw
    tiles, the last one narrower, each walked row by row."""
    if sw <= 0 or sw >= ntx:
        return b % ntx, b // ntx
    st = sw * nty
    s, rem = divmod(b, st)
    ws = min(sw, ntx - s * sw)
    return s * sw + rem % ws, rem // ws


@pytest.mark.parametrize("sw", [0, 1, 2, 3, 4, 5, 8, 16, 64])
def test_tile_order_is_a_permutation(sw):
    """Every tile of the launch grid is visited once, for every strip width and grid shape."""
    for ntx in list(range(1, 40)) + [64, 128, 234]:
        for nty in (1, 2, 5, 8, 33, 256):
            seen = {_tile_of(b, ntx, nty, sw) for b in range(ntx * nty)}
            assert len(seen) == ntx * nty, (ntx, nty)
            assert all(0 <= x < ntx and 0 <= y < nty for x, y in seen), (ntx, nty)
    # within a full strip, consecutive tiles run along a row of the strip, then down
    assert [_tile_of(b, 10, 3, 4) for b in range(6)] == [(0, 0), (1, 0), (2, 0), (3, 0), (0, 1), (1, 1)]
    assert _tile_of(24, 10, 3, 4) == (8, 0) and _tile_of(25, 10, 3, 4) == (9, 0) and _tile_of(26, 10, 3, 4) == (8, 1)


# ------------------------------------------------------------ region launch (small lattices)

def _spread(side, steps, nx, ny, perx, pery, nee):
    """Walks a region launch of `steps` steps on regions of side^2 nodes: which region nodes hold
    right values after each step, LDS reads in the padded plane, every lattice node stored."""
    edge, tile = steps - 1, side - 2 * (steps - 1)
    pad, nodes = side + 1, side * side
    stored = set()
    for by in range(-(-ny // tile)):
        for bx in range(-(-nx // tile)):
            x0, y0 = bx * tile, by * tile
            if nee:
                x0, y0 = min(x0, nx - tile), min(y0, ny - tile)
            at = {}
            for t in range(nodes):
                X, Y = x0 - edge + t % side, y0 - edge + t // side
                if perx:
                    X %= nx
                if pery:
                    Y %= ny
                if 0 <= X < nx and 0 <= Y < ny:
                    at[t] = (X, Y)
            right = set(at)                     # step one pulls from global memory
            for s in range(edge):
                now = set()
                for t, (X, Y) in at.items():
                    r = pad + t
                    w = (not perx and X in (0, nx - 1), not pery and Y in (0, ny - 1))
                    need = []
                    if nee and any(w):
                        dx = (1 if X == 0 else -1) if w[0] else 0
                        dy = (1 if Y == 0 else -1) if w[1] else 0
                        for k in (1, 2):
                            q = min(max(r + k * (dy * side + dx), pad), pad + nodes - 1)
                            for ey in (-1, 0, 1):
                                for ex in (-1, 0, 1):
                                    assert 0 <= q + ey * side + ex < nodes + 2 * pad
                                    need.append((t % side + k * dx + ex, t // side + k * dy + ey))
                    else:
                        for ey in (-1, 0, 1):
                            for ex in (-1, 0, 1):
                                assert 0 <= r + ey * side + ex < nodes + 2 * pad
                                if (perx or 0 <= X + ex < nx) and (pery or 0 <= Y + ey < ny):
                                    need.append((t % side + ex, t // side + ey))
                    if all(0 <= a < side and 0 <= b < side and b * side + a in right for a, b in need):
                        now.add(t)
                # a wave stops when none of its rows is s + 1 nodes deep
                deep = set()
                for v in range(0, nodes, 64):
                    r0, r1 = v // side, (v + 63) // side
                    d = r1 if r1 < side // 2 else side - 1 - r0 if r0 >= side // 2 else side // 2
                    if d > s:
                        deep.update(range(v, v + 64))
                right = now & deep
            for j in range(tile):
                for i in range(tile):
                    if x0 + i < nx and y0 + j < ny:
                        assert (edge + j) * side + edge + i in right, (side, steps, nx, ny, bx, by, i, j)
                        stored.add((x0 + i, y0 + j))
    assert len(stored) == nx * ny


@pytest.mark.parametrize("side,steps", [(16, 1), (16, 3), (16, 4), (16, 5), (16, 6), (22, 2), (22, 4), (22, 5)])
def test_region_launch_stores_right_nodes(side, steps):
    t = side - 2 * (steps - 1)
    for perx, pery in ((False, False), (True, False), (False, True), (True, True)):
        for nx, ny in ((3, 3), (t, t + 1), (2 * t + 1, 7), (side + 3, 2 * t - 1)):
            _spread(side, steps, nx, ny, perx, pery, False)
    for perx, pery in ((False, False), (True, False), (False, True)):
        for nx, ny in ((side, side), (side + 1, side + t - 1), (2 * t + 1 + side, side)):
            _spread(side, steps, nx, ny, perx, pery, True)


def test_region_tile_index_by_multiplication():
    """The kernel divides the tile index by the tiles across with a multiplication by
    ceil(2^32 / ntx)."""
    for ntx in list(range(2, 300)) + [511, 512, 4000]:
        inv = ((1 << 32) + ntx - 1) // ntx
        for b in list(range(0, 40 * ntx, 7)) + [100 * ntx - 1, 100 * ntx]:
            assert (b * inv) >> 32 == b // ntx


# ------------------------------------------------------------ march (large lattices)

E9 = ((0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1))
OPP = (0, 3, 4, 1, 2, 7, 8, 5, 6)


def _collided(q, mix):
    return np.einsum("ij,j...->i...", mix, q)


def _pull(q, nx, ny, perx, pery):
    """Pulls of every node, across a wall the node's own opposite population."""
    out = np.empty_like(q)
    for i, (ex, ey) in enumerate(E9):
        out[i] = np.roll(q[i], (ey, ex), (0, 1))
        x, y = np.arange(nx), np.arange(ny)
        wall = np.zeros((ny, nx), bool)
        if not perx:
            wall |= ((x - ex < 0) | (x - ex >= nx))[None, :]
        if not pery:
            wall |= ((y - ey < 0) | (y - ey >= ny))[:, None]
        out[i][wall] = q[OPP[i]][wall]
    return out


def _march(q, K, W, chunk, perx, pery, mix):
    """The march's bookkeeping with strips of W lanes: what a strip holds of each level, the shifts
    between lanes, ghost columns and ghost rows, chunk ends (nine populations, a linear collision)."""
    ny, nx = q.shape[1:]
    H, V = K - 1, W - 2 * (K - 1)
    pulled, out = _pull(q, nx, ny, perx, pery), np.full_like(q, np.nan)

    def left(v):
        return np.concatenate(([0.0], v[:-1]))

    def right(v):
        return np.concatenate((v[1:], [0.0]))
    for strip in range(-(-nx // V)):
        xv = strip * V - H + np.arange(W)
        x = xv % nx if perx else np.clip(xv, 0, nx - 1)
        gl, gr = (xv == -1) & (not perx), (xv == nx) & (not perx)
        mine = (np.arange(W) >= H) & (np.arange(W) < H + V) & (xv < nx)
        for ya in range(0, ny, chunk):
            yb = min(ya + chunk, ny)

            def first(lv):
                return ya - (K - lv) if pery else max(0, ya - (K - lv))

            def last(lv):
                return yb + (K - lv) if pery else min(ny, yb + (K - lv))
            up0, up1, row = (np.full((H, 3, W), np.nan) for _ in range(3))
            for r in range(first(1), yb + H):
                f = np.full((9, W), np.nan)
                if r < last(1):
                    f = _collided(pulled[:, r % ny, :][:, x], mix)
                for lv in range(1, K):
                    a, rp = lv - 1, r - (lv - 1)
                    if not perx:
                        f = f.copy()
                        l7, l3, l6, r8, r1, r5 = (right(f[7]), right(f[3]), right(up0[a, 2]), left(f[8]), left(f[1]),
                                                  left(up0[a, 1]))
                        up0[a, 1][gl], f[1][gl], f[8][gl] = l7[gl], l3[gl], l6[gl]
                        up0[a, 2][gr], f[3][gr], f[7][gr] = r8[gr], r1[gr], r5[gr]
                    if not pery and rp == 0:
                        up0[a] = f[4], right(f[7]), left(f[8])
                    if not pery and rp == ny:
                        f[4], f[7], f[8] = up0[a, 0], left(up0[a, 1]), right(up0[a, 2])
                    p = np.stack((row[a, 0], left(row[a, 1]), up1[a, 0], right(row[a, 2]), f[4], left(up1[a, 1]),
                                  right(up1[a, 2]), right(f[7]), left(f[8])))
                    up1[a] = up0[a]
                    up0[a], row[a] = f[[2, 5, 6]], f[[0, 1, 3]]
                    f = p
                    rn = rp - 1
                    if first(lv + 1) <= rn < last(lv + 1):
                        f = _collided(f, mix)
                        if lv + 1 == K:
                            out[:, rn, xv[mine]] = f[:, mine]
    return out


@pytest.mark.parametrize("K", [3, 4])
@pytest.mark.parametrize("perx,pery", [(False, False), (True, False), (False, True), (True, True)])
def test_march_moves_what_one_step_moves(K, perx, pery):
    rng = np.random.default_rng(K)
    mix = rng.uniform(-1, 1, (9, 9)) / 3
    for W, nx, ny, chunk in ((12, 6, 9, 4), (12, 13, 11, 3), (12, 18, 8, 8), (16, 31, 17, 5), (16, 40, 21, 10)):
        q = rng.uniform(-1, 1, (9, ny, nx))
        want = q
        for _ in range(K):
            want = _collided(_pull(want, nx, ny, perx, pery), mix)
        got = _march(q, K, W, chunk, perx, pery, mix)
        np.testing.assert_allclose(got, want, rtol=0, atol=1e-13, err_msg=str((W, nx, ny, chunk)))
