"""The broad phase of the obstacle test keeps every disc that the exact FP32
test counts (CPU only): its arithmetic restated in numpy FP32 on boxes of
points from centimetres to kilometres wide, around and far from the start."""
import numpy as np
import pytest

from test_obstacle_fp32_cpu import device_inside, fma32

F = np.float32
WIDEN = F(1.0 + 2.0**-21)


def table(cxw, cyw, r, fx, fy):
    """Centre and squared reach q of a disc in the frame of the start."""
    cx, cy = (F(cxw) - F(fx)).astype(F), (F(cyw) - F(fy)).astype(F)
    c2 = fma32(cx, cx, (cy * cy).astype(F))
    q = fma32((F(1.0000152587890625) * r).astype(F), r, (F(3.0517578125e-05) * c2).astype(F))
    return cx, cy, q


def candidate(px, py, cx, cy, q):
    """Box test of one wave's points against every disc, and the group's box test."""
    xc, yc = px[0], py[0]
    rx, ry = np.abs(px - xc).astype(F).max(), np.abs(py - yc).astype(F).max()
    bx0, bx1 = fma32(-WIDEN, rx, xc), fma32(WIDEN, rx, xc)
    by0, by1 = fma32(-WIDEN, ry, yc), fma32(WIDEN, ry, yc)
    dx = np.maximum(np.maximum((bx0 - cx).astype(F), (cx - bx1).astype(F)), F(0))
    dy = np.maximum(np.maximum((by0 - cy).astype(F), (cy - by1).astype(F)), F(0))
    R = np.sqrt(q).astype(F)
    meets = (((cx - R).astype(F) <= bx1) & ((cx + R).astype(F) >= bx0) & ((cy - R).astype(F) <= by1)
             & ((cy + R).astype(F) >= by0))
    return fma32(dx, dx, (dy * dy).astype(F)) < q, meets


@pytest.mark.parametrize("extent", [0.01, 1.0, 10.0, 300.0, 5000.0])
@pytest.mark.parametrize("far", [0.0, 1.0, 60.0, 1000.0])
def test_no_hit_is_lost(extent, far):
    rng = np.random.default_rng(int(extent * 100 + far))
    hits = edges = 0
    for _ in range(60):
        fx, fy = F(rng.uniform(-50, 50)), F(rng.uniform(-50, 50))
        base = rng.uniform(-far, far, 2)
        n = 64
        # discs around the corners and edges of the box that the points span, so that many are barely touched
        r = rng.uniform(0.05, 1.5, n).astype(F)
        pts = base + rng.uniform(-extent, extent, (384, 2))
        anchor = pts[rng.integers(0, 384, n)]
        anchor[: n // 2] = pts[[pts[:, 0].argmin(), pts[:, 0].argmax(), pts[:, 1].argmin(), pts[:, 1].argmax()]][
            rng.integers(0, 4, n // 2)]
        th = rng.uniform(0, 2 * np.pi, n)
        d = r * (1.0 + rng.choice([0.0, 1e-7, -1e-7, 1e-6, -1e-6, 1e-4, -1e-4], n))
        cxw = (anchor[:, 0] + d * np.cos(th) + fx).astype(F)
        cyw = (anchor[:, 1] + d * np.sin(th) + fy).astype(F)
        px, py = pts[:, 0].astype(F), pts[:, 1].astype(F)
        inside = np.stack([device_inside(px, py, cxw[i], cyw[i], r[i], fx, fy).any() for i in range(n)])
        cx, cy, q = table(cxw, cyw, r, fx, fy)
        cand, meets = candidate(px, py, cx, cy, q)
        assert not (inside & ~cand).any()
        assert not (inside & ~meets).any()
        hits += int(inside.sum())
        edges += int((~inside).sum())
    assert hits > 100  # the discs are placed to be touched
