"""The traversal stack at its edges: trees that fill the ring exactly, overflow
it by one, and spill deeply, in a workspace of exactly the stated size followed
by guard words; and a two-level scene deep on both levels."""
import numpy as np
import pytest

from tests import parity as P
from tests.golden.load import uniform_alpha_textures
from tests.test_gpu_parity import deep_scene
from tests.test_oracle_instances import world_boxes

pytestmark = pytest.mark.gpu
GUARD = 0x5A
GUARD_BYTES = 4096


def announce(msg):
    print(f"[gpu-case] {msg}", flush=True)


@pytest.fixture(scope="module")
def env():
    import torch
    assert torch.cuda.is_available()
    from paper_1912_12786_amd import rtx
    rtx.load_library()
    return torch, rtx


class GuardedWorkspace:
    """A workspace that is given out at exactly the size asked for, guard bytes
    behind it."""

    def __init__(self, torch):
        self.torch, self.buf, self.n = torch, None, 0

    def get(self, nbytes):
        self.n = nbytes
        self.buf = self.torch.full((nbytes + GUARD_BYTES,), GUARD, dtype=self.torch.uint8,
                                   device="cuda")
        return self.buf.data_ptr(), nbytes

    def intact(self):
        return bool((self.buf[self.n:] == GUARD).all())


def masks(n, seed):
    """Texture ids (one triangle in 25 opaque, the others transparent, so that
    most of the tree is walked), texture coordinates and the two textures."""
    geom = (np.random.default_rng(seed).random(n) < 0.04).astype(np.uint32)
    return geom, np.zeros((n, 3, 2), np.float32), uniform_alpha_textures([0, 255], (2, 2))


def axis_rays(n=200):
    rng = np.random.default_rng(3)
    rays = np.zeros((n, 8), np.float32)
    rays[:, 0] = -1.0
    rays[:, 1:3] = rng.uniform(-0.2, 0.2, size=(n, 2))
    rays[:, 4] = 1.0
    rays[n // 2:, 5:7] = rng.normal(0, 1e-3, size=(n - n // 2, 2))
    rays[:, 7] = np.inf
    return rays


# single-triangle leaves: the rows' trees are 1, 6, 7, 8, 9, 10 and 36 deep
@pytest.mark.parametrize("n", [2, 14, 17, 20, 23, 26, 160])
@pytest.mark.parametrize("query", ["closest", "any", "multi"])
def test_stack_depths(env, oracle_lib, n, query):
    torch, rtx = env
    verts, rays_np = deep_scene(n), axis_rays()
    rays = torch.from_numpy(rays_np).cuda()
    bvh = oracle_lib.build_bvh(verts, max_leaf=1)
    geom, tc, tex = masks(n, 5)
    B = oracle_lib.traverse(verts, bvh, rays_np, "alpha", geom_ids=geom, texcoords=tc, textures=tex,
                            any_hit=query == "any", multi_k=5 if query == "multi" else 0)
    for layout in ("f32", "q8", "f32p", "wide4"):
        sc = rtx.upload_scene(verts, geom, tc, tex, layout=layout, max_leaf=1)
        ref = None
        for shape in rtx.rt_launch_shapes():
            ws = GuardedWorkspace(torch)
            announce(f"stack n={n} depth={sc.info.max_depth} {query} {layout} {shape}")
            try:
                got = rtx.trace(sc, rays, "alpha", query=query, k=5, shape=shape, workspace=ws)
            except rtx.RtxError as e:
                assert e.status == rtx.RT_ERR_UNSUPPORTED
                continue
            torch.cuda.synchronize()
            assert ws.buf is None or ws.intact()
            got = torch.cat([got[0].reshape(-1).view(torch.int32), got[1]]) if query == "multi" \
                else got.view(torch.int32)
            if ref is None:
                ref = got
                if layout == "f32" and query == "closest":
                    P.assert_exact_vs_b(P.hits_to_numpy(got.view(torch.float32)), B, f"stack n={n}")
                elif layout == "f32" and query == "any":
                    assert np.array_equal(P.occluders_to_numpy(got), B["prim"])
                elif layout == "f32":
                    assert np.array_equal(P.occluders_to_numpy(got[-len(rays_np):]), B["n_hits"])
            assert torch.equal(got, ref)


# (top-level rows of instances, triangles of the deepest mesh)
@pytest.mark.parametrize("n_inst,n_tris", [(2, 2), (5, 20), (40, 160)])
@pytest.mark.parametrize("any_hit", [False, True])
def test_two_level_stack(env, oracle_lib, n_inst, n_tris, any_hit):
    torch, rtx = env
    meshes = [deep_scene(n_tris), deep_scene(3)]
    ids = (np.arange(n_inst) % 2).astype(np.uint32)
    # instance q: the mesh shrunk by 1.3^q and moved along x, so that the top
    # level peels off the largest boxes one at a time
    maps = np.zeros((n_inst, 12), np.float32)
    scale = 1.3 ** np.arange(n_inst)
    maps[:, [0, 5, 10]] = scale[:, None]
    maps[:, 3] = -2.0 * np.arange(n_inst)
    lo = np.empty((n_inst, 3), np.float32)
    hi = np.empty((n_inst, 3), np.float32)
    for q in range(n_inst):
        lo[q:q + 1], hi[q:q + 1] = world_boxes(meshes[ids[q]], maps[q:q + 1])
    rays_np = axis_rays()
    announce(f"two-level stack: {n_inst} instances, {n_tris} triangles, any={any_hit}")
    looks = [masks(len(m), 6 + i) for i, m in enumerate(meshes)]
    akw = dict(geom_ids=[g for g, _, _ in looks], texcoords=[t for _, t, _ in looks],
               textures=looks[0][2])
    sc = rtx.InstancedScene(meshes, ids, maps, lo, hi, max_leaf=1, **akw)
    ws = GuardedWorkspace(torch)
    out, inst, cnt = sc.trace(torch.from_numpy(rays_np).cuda(), "alpha", any_hit=any_hit,
                              count=True, workspace=ws)
    torch.cuda.synchronize()
    assert ws.buf is None or ws.intact()
    bvhs = [oracle_lib.build_bvh(m, max_leaf=1) for m in meshes]
    B = oracle_lib.traverse_instanced(meshes, bvhs, ids, maps, oracle_lib.build_tlas(lo, hi),
                                      rays_np, "alpha", any_hit=any_hit, **akw)
    assert np.array_equal(inst.cpu().numpy().view(np.uint32), B["inst"])
    P.assert_counters_vs_b(cnt, B, "two-level stack")
    if any_hit:
        assert np.array_equal(P.occluders_to_numpy(out), B["prim"])
    else:
        P.assert_exact_vs_b(P.hits_to_numpy(out), B, "two-level stack")
