"""Triangles in one axis-aligned plane: their boxes are flat, a box's entry
often lies a rounding beyond the hit inside it, and culling then depends on the
bound at each visit.  A ray's result is still the lone traversal's, bit for
bit, however the rays are spread over lanes, waves and launches."""
import numpy as np
import pytest

from paper_1912_12786_amd import workloads as W
from tests import parity as P

pytestmark = pytest.mark.gpu


def announce(msg):
    print(f"[gpu-case] {msg}", flush=True)


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_1912_12786_amd import rtx
    rtx.load_library()
    return torch, rtx


def decals(n, planes, seed):
    """n overlapping triangles on planes of constant z."""
    g = np.random.default_rng(seed)
    v = np.empty((n, 3, 3), np.float32)
    v[..., :2] = g.uniform(0, 1, (n, 1, 2)) + g.uniform(-0.2, 0.2, (n, 3, 2))
    v[..., 2] = np.float32([0.3, 0.37, 0.5, 0.61])[g.integers(0, planes, n)][:, None]
    return v


def tiles(k):
    """Two walls each way of k x k quads that share their edges."""
    g = np.linspace(0, 1, k + 1, dtype=np.float32)
    out = []
    for i, j in np.ndindex(k, k):
        p = [(g[i], g[j]), (g[i + 1], g[j]), (g[i + 1], g[j + 1]), (g[i], g[j + 1])]
        for w in (0.25, 0.5):
            for t in ((0, 1, 2), (0, 2, 3)):
                out.append([[*p[c], w] for c in t])
                out.append([[w, *p[c]] for c in t])
    return np.array(out, np.float32)


SCENES = {"decals": lambda: decals(600, 1, 1), "layers": lambda: decals(400, 4, 2),
          "tiles": lambda: tiles(12)}
WIDTH = 128


def scene_of(oracle_lib, name, max_leaf=1):
    v = SCENES[name]()
    g = np.random.default_rng(4)
    geom = g.integers(0, 4, size=len(v)).astype(np.uint32)
    tc = g.uniform(0, 1, size=(len(v), 3, 2)).astype(np.float32)
    return v, geom, tc, W.alpha_textures(4, 64, 13), oracle_lib.build_bvh(v, max_leaf=max_leaf)


def rays_of(n):
    """A camera's rays off the planes, and from n = 20,000 on as many rays
    again through the walls' shared edges."""
    cam = W.pinhole_rays(WIDTH, -(-n // WIDTH), np.array([0.5, 0.45, 2.5]), np.full(3, 0.5), 40.0)[:n]
    if n < 20_000:
        return cam
    g = np.random.default_rng(9)
    edge = np.zeros((n, 8), np.float32)
    edge[:, :2] = g.integers(0, 25, (n, 2)) / np.float32(24)
    edge[:, 2] = 2.0
    edge[:, 4:6] = g.integers(-3, 4, (n, 2)) / 8
    edge[:, 6] = -1.0
    edge[:, 7] = np.inf
    return np.concatenate([cam, edge])


def least(torch, rtx):
    class Least(rtx.Workspace):
        def get(self, nbytes):
            self.buf = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
            return self.buf.data_ptr(), nbytes
    return Least("cuda")


def ways(torch, rtx, n):
    """(shape, options) over what a launch's rays may be spread by."""
    options = [{}, {"longest_first": True}, {"waves_per_simd": 1}, {"workspace": least(torch, rtx)}]
    if n % WIDTH == 0:
        options += [{"image_width": WIDTH}, {"image_width": WIDTH, "longest_first": True}]
    for shape in rtx.rt_launch_shapes():
        yield from ((shape, kw) for kw in (options if shape[0] == 64 and shape[2] == 64 else [{}]))


# waves of one ray, part of a wave, waves of 1, 4 and 64 rays, a queue that is drawn from
@pytest.mark.parametrize("n_rays", [1, 40, 5000, 128 * 128, 40_000, 420_000])
@pytest.mark.parametrize("name", list(SCENES))
@pytest.mark.parametrize("kind", ["default", "procedural", "alpha"])
def test_closest_in_one_plane(env, oracle_lib, name, kind, n_rays):
    torch, rtx = env
    v, geom, tc, tex, bvh = scene_of(oracle_lib, name)
    rays_np = rays_of(n_rays)
    idx = np.arange(0, len(rays_np), max(1, len(rays_np) // 40_000))
    rays, at = torch.from_numpy(rays_np).cuda(), torch.from_numpy(idx).cuda()
    okw = dict(geom_ids=geom, texcoords=tc, textures=tex) if kind == "alpha" else {}
    for layout in ("f32", "q8", "f32p", "wide4"):
        sc = rtx.upload_scene(v, geom, tc, tex, layout=layout, max_leaf=1)
        B = oracle_lib.traverse(v, bvh, rays_np[idx], kind, layout=layout, **okw)
        for shape, kw in ways(torch, rtx, len(rays_np)):
            what = f"{name} {kind} {layout} {n_rays} rays {shape} {sorted(kw)}"
            announce(what)
            try:
                got = rtx.trace(sc, rays, kind, shape=shape, **kw)
            except rtx.RtxError as e:
                assert e.status == rtx.RT_ERR_UNSUPPORTED
                continue
            torch.cuda.synchronize()
            P.assert_exact_vs_b(P.hits_to_numpy(got[at]), B, what)


def quads_on_a_grid(n, seed):
    """n corners on a grid of 32 with a quad of one cell across each axis, many
    of them twice: equal distances within a leaf and across leaves."""
    c = np.round(np.random.default_rng(seed).uniform(0, 1, (n, 3)) * 32)
    out = []
    for a in range(3):
        for t in (((0, 0), (1, 0), (1, 1)), ((0, 0), (1, 1), (0, 1))):
            tri = np.repeat(c[:, None], 3, axis=1)
            for k, (x, y) in enumerate(t):
                tri[:, k, (a + 1) % 3] += x
                tri[:, k, (a + 2) % 3] += y
            out.append(tri)
    return (np.stack(out, 1).reshape(-1, 3, 3) / 32).astype(np.float32)


@pytest.mark.parametrize("max_leaf", [1, 2, 4, 7])
@pytest.mark.parametrize("n_rays", [200_000, 20_000])
def test_equal_distances_in_a_leaf(env, oracle_lib, max_leaf, n_rays):
    """Rays from grid points along rational directions through quads on a grid,
    hit after hit at one distance, also in the same leaf."""
    torch, rtx = env
    v = quads_on_a_grid(4000, 8)
    bvh = oracle_lib.build_bvh(v, max_leaf=max_leaf)
    edge = rays_of(n_rays)[n_rays:].copy()
    edge[:, :2] = np.random.default_rng(3).integers(0, 65, (n_rays, 2)) / np.float32(64)
    rays = torch.from_numpy(edge).cuda()
    for layout in ("f32", "q8", "f32p", "wide4"):
        sc = rtx.upload_scene(v, layout=layout, max_leaf=max_leaf)
        B = oracle_lib.traverse(v, bvh, edge, "default", layout=layout)
        for shape, kw in ways(torch, rtx, n_rays):
            what = f"quads on a grid, leaves <= {max_leaf}, {layout} {n_rays} rays {shape} {sorted(kw)}"
            announce(what)
            try:
                got = rtx.trace(sc, rays, shape=shape, **kw)
            except rtx.RtxError as e:
                assert e.status == rtx.RT_ERR_UNSUPPORTED
                continue
            torch.cuda.synchronize()
            P.assert_exact_vs_b(P.hits_to_numpy(got), B, what)


@pytest.mark.parametrize("kind", ["default", "procedural"])
def test_batch_in_one_plane(env, oracle_lib, kind):
    torch, rtx = env
    names, counts = list(SCENES), [3000, 30, 9001]
    built = [scene_of(oracle_lib, n) for n in names]
    rays_np = [rays_of(n) for n in counts]
    rays = torch.from_numpy(np.concatenate(rays_np)).cuda()
    for layout in ("f32", "q8", "f32p", "wide4"):
        scenes = [rtx.upload_scene(b[0], layout=layout, max_leaf=1) for b in built]
        announce(f"batch in one plane {kind} {layout}")
        got = P.hits_to_numpy(rtx.Batch(scenes, counts, kind).trace(rays))
        B = [oracle_lib.traverse(b[0], b[4], r, kind, layout=layout) for b, r in zip(built, rays_np)]
        P.assert_exact_vs_b(got, {k: np.concatenate([x[k] for x in B]) for k in ("t", "u", "v", "prim")},
                            f"batch {kind} {layout}")


@pytest.mark.parametrize("k", [1, 2, 4, 5, 8])
@pytest.mark.parametrize("name", list(SCENES))
@pytest.mark.parametrize("kind", ["default", "procedural", "alpha"])
def test_k_nearest_in_one_plane(env, oracle_lib, name, kind, k):
    torch, rtx = env
    v, geom, tc, tex, bvh = scene_of(oracle_lib, name)
    okw = dict(geom_ids=geom, texcoords=tc, textures=tex) if kind == "alpha" else {}
    for n_rays in (40, 5000, 128 * 128):
        rays_np = rays_of(n_rays)
        rays = torch.from_numpy(rays_np).cuda()
        for layout in ("f32", "q8", "f32p", "wide4"):
            sc = rtx.upload_scene(v, geom, tc, tex, layout=layout, max_leaf=1)
            B = oracle_lib.traverse(v, bvh, rays_np, kind, layout=layout, multi_k=k, **okw)
            for shape, kw in ways(torch, rtx, n_rays):
                what = f"{name} {kind} {layout} k={k} {n_rays} rays {shape} {sorted(kw)}"
                announce(what)
                try:
                    hits, n_hits = rtx.trace(sc, rays, kind, query="multi", k=k, shape=shape, **kw)
                except rtx.RtxError as e:
                    assert e.status == rtx.RT_ERR_UNSUPPORTED
                    continue
                torch.cuda.synchronize()
                assert np.array_equal(n_hits.cpu().numpy().view(np.uint32), B["n_hits"]), what
                h = hits.cpu().numpy()
                assert np.array_equal(h[..., 1].view(np.uint32), B["prim"]), what
                for c, key in ((0, "t"), (2, "u"), (3, "v")):
                    assert np.array_equal(P.bits(h[..., c]), P.bits(B[key])), (what, key)
