"""Drawings whose decisions are ties: right angles, quarter circles, exact
reversals, connectors.  Where the arithmetic of a decision is exact (integer
coordinates, or the same rounding on both sides of a symmetry), the counts are
those of the oracle without a margin."""
import numpy as np

from paper_2405_00127_amd import scenes as S

KAPPA = 0.5522847498307936  # arm of a quarter circle of radius 1


def scale(s):
    return np.array([[s, 0, 0, s, 0, 0]], np.float32)


def rotation(degrees):
    c, s = np.cos(np.radians(degrees)), np.sin(np.radians(degrees))
    return np.array([[c, s, -s, c, 0, 0]], np.float32)


def polygons(join, turn=90, closed=False, xform=None):
    """Polylines of equal sides that turn by the same angle, to and fro (or
    round and round when closed)."""
    b = S.SceneBuilder()
    for k in range(20):
        p, a = np.array([100.0 * (k % 17), 90.0 * (k // 17)]), 0.0
        pts = [p]
        for j in range(40):
            p = p + 30.0 * np.round([np.cos(np.radians(a)), np.sin(np.radians(a))], 15)
            pts.append(p)
            a += turn if closed or j % 2 == 0 else -turn
        b.add_path([S.MOVE] + [S.LINE] * 40 + ([S.CLOSE] if closed else []), np.array(pts), 0, 0)
    return b.build(S.make_styles([6.0], join, S.CAP_ROUND), xform)


def circles(radius, w, corner=0.0, fill=False, xform=None):
    """Circles of four cubics, or (corner > 0) rounded squares."""
    b = S.SceneBuilder()
    for k in range(60):
        r, s = radius * (1 + k % 7), corner
        q = KAPPA * r
        c = np.array([50.0 * (k % 23), 50.0 * (k // 23)])
        verbs, pts = [S.MOVE], [[r + s, 0.0]]
        for quarter in range(4):
            at = [[r + s, s], [r + s, s + q], [q + s, r + s], [s, r + s]]
            if s:
                verbs.append(S.LINE)
                pts.append(at[0])
            verbs.append(S.CUBIC)
            pts += at[1:]
            # the next quarter, turned by a right angle about the middle
            pts = [[y, -x] for x, y in pts]
        pts = np.array(pts) + c
        b.add_path(verbs + [S.CLOSE], pts, 0, 0)
    st = S.make_styles([w], S.JOIN_ROUND, S.CAP_ROUND)
    if fill:
        st["flags"] |= S.STYLE_FILL
    return b.build(st, xform)


def reversals(join, xform=None):
    """Lines that turn back on themselves, onto shorter and longer ones."""
    b = S.SceneBuilder()
    ways = np.array([[30, 0], [0, 30], [3, 4], [5, 12], [7, 1], [1, 1], [13, 29]], float)
    for k in range(200):
        p, d = np.array([40.0 * (k % 17), 40.0 * (k // 17)]), ways[k % 7]
        pts = [p, p + d, p - d * (k % 5), p + 3 * d, p + 3 * d + d[::-1] * [1, -1], p + 3 * d]
        b.add_path([S.MOVE] + [S.LINE] * 5, np.array(pts), 0, 0)
    return b.build(S.make_styles([3.0], join, S.CAP_SQUARE), xform)


def connectors(size, w, xform=None):
    """S and U curves whose middle control vector is perpendicular to both ends."""
    b = S.SceneBuilder()
    for k in range(60):
        z = size * (1 + k % 9)
        h = [0.5, 1.0, 2.0][k % 3] * z
        pts = [[0, 0], [0, z], [h, z], [h, 2 * z], [h, 3 * z],
               [h, 4 * z], [2 * h, 4 * z], [2 * h, 3 * z], [3 * h, 3 * z],
               [4 * h, 3 * z], [3 * h, 4 * z], [4 * h, 4 * z],
               [5 * h, 4 * z], [4 * h, 5 * z], [5 * h, 5 * z]]
        b.add_path([S.MOVE, S.CUBIC, S.LINE, S.CUBIC, S.LINE, S.CUBIC, S.CUBIC],
                   np.array(pts) + [50.0 * (k % 13), 60.0 * (k // 13)], 0, 0)
    return b.build(S.make_styles([w], S.JOIN_ROUND, S.CAP_ROUND), xform)


SYMMETRIC = {
    "right_angles_round": lambda x: polygons(S.JOIN_ROUND, xform=x),
    "right_angles_miter": lambda x: polygons(S.JOIN_MITER, xform=x),
    "squares": lambda x: polygons(S.JOIN_ROUND, closed=True, xform=x),
    "circles_3_1": lambda x: circles(3.0, 1.0, xform=x),
    "circles_10_4": lambda x: circles(10.0, 4.0, xform=x),
    "circles_half_2": lambda x: circles(0.5, 2.0, xform=x),
    "discs": lambda x: circles(4.0, 2.0, fill=True, xform=x),
    "rounded_squares": lambda x: circles(4.0, 2.0, corner=20.0, xform=x),
    "reversals_round": lambda x: reversals(S.JOIN_ROUND, xform=x),
    "reversals_bevel": lambda x: reversals(S.JOIN_BEVEL, xform=x),
}
