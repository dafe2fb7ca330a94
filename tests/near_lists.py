"""Meshes and the flagged pairs that both searches (host and device) have to give on them,
pair by pair and in order, by their definition."""
import numpy as np

from paper_2606_13482_amd.inputs import cube_sphere, icosphere


def _turned(V):
    """Away from the axes, so that few distances are equal."""
    a, b = 0.4, 1.1
    Rz = np.array([[np.cos(a), -np.sin(a), 0], [np.sin(a), np.cos(a), 0], [0, 0, 1]])
    Rx = np.array([[1, 0, 0], [0, np.cos(b), -np.sin(b)], [0, np.sin(b), np.cos(b)]])
    return V @ Rz @ Rx


def mesh(name):
    if name == "sphere":             # 5120 triangles: several runs of 64 for each wave
        V, T = icosphere(4)
        return _turned(V), T
    if name == "flat":               # slivers, 1452 triangles
        V, T = cube_sphere(11, "ellipsoid", axes=(1.0, 1.6, 0.02))
        return _turned(V), T
    V, T = icosphere(3)              # edges of some units in the last place, neighbours far apart in the list
    return np.rint(16 * V) + 2.0 ** 52, T[np.random.default_rng(1).permutation(len(T))]


CASES = [("sphere", 2.0), ("sphere", 0.0), ("sphere", 0.3), ("flat", 2.0), ("flat", 0.7), ("far", 0.0), ("far", 1.0)]


def expected(V, T, factor):
    """Pairs p <= q, ascending: a shared vertex, or |c_p - c_q|^2 < (factor max(longest))^2."""
    c = (V[T[:, 0]] + V[T[:, 1]] + V[T[:, 2]]) / 3.0
    L = np.zeros(len(T))
    for i, j in ((1, 0), (2, 0), (2, 1)):
        e = V[T[:, i]] - V[T[:, j]]
        L = np.maximum(L, np.sqrt(e[:, 0] * e[:, 0] + e[:, 1] * e[:, 1] + e[:, 2] * e[:, 2]))
    out = []
    for p in range(len(T)):
        d = c[p] - c[p:]
        dd = d[:, 0] * d[:, 0] + d[:, 1] * d[:, 1] + d[:, 2] * d[:, 2]
        thr = factor * np.maximum(L[p], L[p:])
        hit = (dd < thr * thr) | (T[p:, :, None] == T[p]).any((1, 2))
        q = p + np.flatnonzero(hit)
        out.append(np.stack([np.full(len(q), p), q], 1))
    return np.concatenate(out).astype(np.int32)
