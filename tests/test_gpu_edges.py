"""Kernels at the sizes where they can go wrong: the edges of their tiles, the
smallest inputs, and the class counts at which their layout changes."""
import dataclasses

import numpy as np
import pytest

import oracle
import scenes
from gpu_cases import cuda, gpu_map_of, oracle_map_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [2, 20, 32, 33, 64, 65, 128, 129, 255])
def test_readout_of_any_number_of_voxels(K):
    # a workgroup serves 64, 32, 16 or 8 voxels by class count and writes their
    # rows together; every subset of the outputs has the same values
    sc = scenes.random_points_scene(seed=K, n=400, K=K, extent=0.8)
    om, gm = oracle_map_of(sc, scsm=True), gpu_map_of(sc, model="scsm")
    rng = np.random.default_rng(K)
    q = rng.integers(-9, 9, size=(131, 3)).astype(np.int32)
    ref = oracle.readout(om.lookup(q), free_class=0)
    a_ref = om.lookup(q)
    for M in (1, 7, 8, 9, 63, 64, 65, 131):
        print(f"[case] readout K={K} M={M}", flush=True)
        out = {k: v.cpu().numpy() for k, v in gm.query(cuda(q[:M])).items()}
        assert np.array_equal(out["alpha"], (a_ref[:M]).astype(np.float32))
        np.testing.assert_allclose(out["mean"], ref["mean"][:M], rtol=1e-6)
        np.testing.assert_allclose(out["var"], ref["var"][:M], rtol=1e-6)
        np.testing.assert_allclose(out["p_occ"], ref["p_occ"][:M], rtol=1e-6, atol=1e-7)
        assert np.array_equal(out["label"], ref["label"][:M])
        for k in out:
            one = gm.query(cuda(q[:M]), **{n: n == k for n in out})
            assert list(one) == [k] and np.array_equal(one[k].cpu().numpy(), out[k])


@pytest.mark.parametrize("n", [1, 127, 129, 700_000])
def test_unit_sizes_chosen_per_insert(n):
    # no free samples: n rows, all of one class in a few blocks, so that a unit's
    # rows (128 at least, 192 for the largest) decide how many units there are
    sc = scenes.random_points_scene(seed=3, n=n, K=2, extent=0.35, centre=(0.4, 0.4, 0.4), l=0.15)
    sc.scans[0].label[:] = 1
    print(f"[case] unit size n={n}", flush=True)
    om, gm = oracle_map_of(sc), gpu_map_of(sc)
    st = gm.stats()
    chunk = 192 if n == 700_000 else 128
    assert st["n_units"] >= -(-n // chunk) and st["n_units"] <= n // chunk + st["n_point_blocks"]
    ijk, a_ref, _, _ = om.export()
    a = gm.query(cuda(ijk.astype(np.int32)))["alpha"].cpu().numpy()
    assert np.max(np.abs(a - a_ref) / a_ref) <= 1e-5


@pytest.mark.parametrize("n", [1, 2, 1_023, 1_025, 65_536, 65_537, 262_144, 262_145])
@pytest.mark.parametrize("extent,res", [(2.0, 0.1), (700.0, 0.3)])
def test_sorted_cells_at_tile_edges(n, extent, res):
    # the radix sort's tiles (1,024 elements up to 2^18, 4,096 beyond), its passes
    # without a scan of the counts (up to 64 tiles), 32- and 64-bit keys
    from paper_1909_04631_amd import bucket_cells
    rng = np.random.default_rng(n)
    xyz = rng.uniform(-extent, extent, size=(n, 3)).astype(np.float32)
    if extent > 100:
        xyz[:, 2] *= 0.05
    print(f"[case] cells n={n} extent={extent}", flush=True)
    keys, start, count, order = [t.cpu().numpy() for t in bucket_cells(cuda(xyz), res, 4)]
    ref = oracle.pack_keys(oracle.voxel_coords(xyz, np.float32(res)))
    uk, inv, cnt = np.unique(ref, return_inverse=True, return_counts=True)
    by_key = np.argsort(keys.view(np.uint64))
    assert np.array_equal(keys.view(np.uint64)[by_key], uk)
    assert np.array_equal(count[by_key], cnt)
    # the rows of a cell in input order: a stable sort by key gives the same order
    want = np.argsort(inv, kind="stable")
    first = np.concatenate([[0], np.cumsum(cnt)])
    got = np.concatenate([order[s:s + c] for s, c in zip(start[by_key], count[by_key])])
    assert np.array_equal(got, want) and first[-1] == n


@pytest.mark.parametrize("B,K,n", [(1, 3, 5), (2, 2, 1), (2, 2, 33), (4, 20, 1_025), (8, 5, 64),
                                   (32, 2, 3)])
@pytest.mark.parametrize("spread", ["near", "far"])
def test_import_export_round_trip(B, K, n, spread):
    # blocks in random order come back in ascending key order, near ones sorted by
    # keys relative to their box, far ones (a box of more than 32 bits) by full
    # keys; arrays that are 4-byte aligned only take scalar accesses
    import torch
    from paper_1909_04631_amd import SemanticMap, SmkiError
    rng = np.random.default_rng(B * 100 + n)
    lim = (1 << 20) // B
    half = 12 if spread == "near" else lim
    ijk = np.unique(rng.integers(-half, half, size=(4 * n + 8, 3)), axis=0)
    ijk = ijk[rng.permutation(ijk.shape[0])[:n]].astype(np.int32)
    if spread == "far":
        ijk[0], ijk[-1] = -lim, lim - 1
    n = ijk.shape[0]
    alpha = rng.uniform(0.5, 2.0, size=(n, K, B, B, B)).astype(np.float32)
    alpha[rng.random((n, K)) < 0.5] = np.float32(1e-3)     # classes without evidence
    print(f"[case] import/export B={B} K={K} n={n} {spread}", flush=True)
    order = np.lexsort((ijk[:, 2], ijk[:, 1], ijk[:, 0]))
    for shift in (0, 1):
        m = SemanticMap(0.1, B, 0.2, 0.1, K, 1e-3, model="scsm")
        buf = torch.empty(alpha.size + shift, dtype=torch.float32, device="cuda")
        a = buf[shift:].view(alpha.shape)
        a.copy_(cuda(alpha))
        m.import_(cuda(ijk), a)
        assert m.num_blocks() == n
        got_ijk, got = m.export()
        assert np.array_equal(got_ijk.cpu().numpy(), ijk[order])
        assert np.array_equal(got.cpu().numpy(), alpha[order])
        # the same into an array of the caller's that is not 16-byte aligned
        import ctypes
        from paper_1909_04631_amd import _lib
        out = torch.empty(alpha.size + 1, dtype=torch.float32, device="cuda")[1:]
        k = ctypes.c_int64()
        assert _lib.lib().smki_export(m._h, n, ctypes.byref(k), None,
                                      ctypes.c_void_p(out.data_ptr())) == 0
        assert np.array_equal(out.cpu().numpy(), alpha[order].reshape(-1))
        # voxels of the first block by query
        v = ijk[0] * B + rng.integers(0, B, size=(7, 3))
        q = m.query(cuda(v.astype(np.int32)))["alpha"].cpu().numpy()
        l = v - ijk[0] * B
        assert np.array_equal(q, alpha[0][:, l[:, 0], l[:, 1], l[:, 2]].T)
        if n > 1:   # a duplicate anywhere, and a block out of range, leave the map as it was
            for bad, status in ((np.concatenate([ijk[1:], ijk[-1:]]), -5),
                                (np.concatenate([ijk[1:], [[lim, 0, 0]]]).astype(np.int32), -6)):
                with pytest.raises(SmkiError) as e:
                    m.import_(cuda(bad), cuda(alpha))
                assert e.value.status == status
            assert np.array_equal(m.export()[1].cpu().numpy(), alpha[order])


def test_export_after_inserts_and_a_reset():
    # the box that the export's keys are relative to follows inserts, resets and
    # imports: blocks in ascending order each time, equal to the map's voxels
    sc = scenes.make_config(0)
    p, s = sc.params, sc.scans[0]
    far = s.xyz + np.float32(150.0)
    gm = gpu_map_of(sc)
    for step in ("one scan", "a far scan added", "reset, then the far scan"):
        print(f"[case] export after {step}", flush=True)
        if step.startswith("reset"):
            gm.reset()
        if "far" in step:
            gm.insert_scan(cuda(far), cuda(s.label), s.origin + np.float32(150.0), p.free_step)
        ijk, alpha = [t.cpu().numpy() for t in gm.export()]
        assert np.array_equal(np.lexsort((ijk[:, 2], ijk[:, 1], ijk[:, 0])), np.arange(ijk.shape[0]))
        assert np.unique(ijk, axis=0).shape[0] == ijk.shape[0] == gm.num_blocks()
        for b in range(0, ijk.shape[0], 17):
            v = ijk[b] * gm.B + np.array([[0, 1, 2], [gm.B - 1, 0, gm.B - 1]])
            q = gm.query(cuda(v.astype(np.int32)))["alpha"].cpu().numpy()
            l = v - ijk[b] * gm.B
            assert np.array_equal(q, alpha[b][:, l[:, 0], l[:, 1], l[:, 2]].T)


@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("n", [1, 64, 65, 4_000])
def test_counting_model_runs_across_wavefronts(n, soft):
    # every hit in one of three voxels: runs of equal keys that start before a
    # wavefront's rows and end inside, or span several wavefronts
    import torch
    from paper_1909_04631_amd import SemanticMap
    rng = np.random.default_rng(n)
    cell = np.sort(rng.choice(3, size=n, p=[0.9, 0.05, 0.05]))
    xyz = (0.05 + 0.1 * np.array([[0, 0, 0], [0, 0, 1], [9, 3, 2]])[cell]).astype(np.float32)
    lab = rng.integers(0, 3, size=n).astype(np.int32)
    w = rng.uniform(0.0, 1.0, size=(n, 3)).astype(np.float32)
    w[rng.random((n, 3)) < 0.3] = 0.0
    print(f"[case] counting runs n={n} soft={soft}", flush=True)
    m = SemanticMap(0.1, 8, 0.3, 0.1, 3, 1e-3, model="scsm")
    if soft:
        m.insert_scan_soft(cuda(xyz), cuda(w), (0, 0, 0), 0.0)
        add = np.stack([np.bincount(cell, weights=w[:, k].astype(np.float64), minlength=3)
                        for k in range(3)], 1)
    else:
        m.insert_scan(cuda(xyz), cuda(lab), (0, 0, 0), 0.0)
        add = np.stack([np.bincount(cell[lab == k], minlength=3) for k in range(3)], 1)
    torch.cuda.synchronize()
    q = np.array([[0, 0, 0], [0, 0, 1], [9, 3, 2]], np.int32)
    a = m.query(cuda(q))["alpha"].cpu().numpy()
    want = np.float32(1e-3) + add.astype(np.float32)
    assert np.array_equal(a, want.astype(np.float32))


@pytest.mark.parametrize("B,K", [(4, 5), (8, 70)])
def test_replay_with_more_targets_than_its_grid(B, K):
    # captured on hits that fill a few blocks (the window is widened by two of
    # them), replayed on hits all over the window: many more target blocks than
    # the launches start workgroups for, then on the first hits again (the slot
    # table is back as it was), and after a replay that fails
    import torch
    from paper_1909_04631_amd import SemanticMap, SmkiError
    rng = np.random.default_rng(B)
    n = 700
    near = rng.uniform(0.0, 0.5, size=(n, 3)).astype(np.float32)
    near[0], near[1] = -6.0, 6.0
    wide = rng.uniform(-5.9, 5.9, size=(n, 3)).astype(np.float32)
    out = wide.copy()
    out[5] = 400.0
    lab = rng.integers(0, K, size=n).astype(np.int32)
    origins = [(0.0, 0.0, 0.0)]
    m = SemanticMap(0.1, B, 0.2, 0.1, K, 1e-3, initial_blocks=1 << 15)
    xyz, y = cuda(wide), cuda(lab)
    m.insert_scan(xyz, y, origins[0], 0.0)     # (room in the map for the wide hits)
    m.reset()
    xyz.copy_(cuda(near))
    g = m.batch_capture(xyz, y, [0, n], origins, 0.0, margin=1.0)
    q = cuda(np.floor(np.concatenate([near, wide]) / np.float32(0.1)).astype(np.int32))
    fresh = SemanticMap(0.1, B, 0.2, 0.1, K, 1e-3, initial_blocks=1 << 15)
    for name, data in (("wide", wide), ("near", near), ("out", out), ("wide", wide)):
        print(f"[case] replay {name} B={B} K={K}", flush=True)
        m.reset()
        xyz.copy_(cuda(data))
        g.replay([0, n], origins)
        if name == "out":
            with pytest.raises(SmkiError):
                m.sync()
            assert m.num_blocks() == 0
            continue
        m.sync()
        st = m.stats()
        fresh.reset()
        fresh.insert_scan(cuda(data), y, origins[0], 0.0)
        ref = fresh.stats()
        assert all(st[k] == ref[k] for k in ("n_updated_voxels", "n_pairs", "n_new_blocks",
                                             "n_new_class_blocks", "n_target_blocks"))
        assert torch.equal(m.query(q)["alpha"], fresh.query(q)["alpha"])
    g.close()


@pytest.mark.parametrize("soft", [False, True])
@pytest.mark.parametrize("lv", [0.3, 0.6, 0.8, 0.95, 1.2, 1.45, 1.5, 1.57, 1.65])
def test_small_stencils_around_unit_edges(lv, soft):
    # stencils of 1 to 33 voxels around a cell (lanes over rows), and the first
    # larger one; units of 64 rows and of 96 (a batch and a half)
    import torch
    from paper_1909_04631_amd import SemanticMap
    K, res = 3, 0.2
    l = float(np.float32(lv) * np.float32(res))
    rng = np.random.default_rng(int(100 * lv))
    n = 1_500
    xyz = rng.uniform(-1.0, 1.0, size=(n, 3)).astype(np.float32)
    xyz[: n // 2] = np.float32(0.1) + rng.normal(0, 0.03, size=(n // 2, 3)).astype(np.float32)
    xyz[:40] = np.float32(0.2) * np.round(xyz[:40] / np.float32(0.2))   # on voxel faces
    lab = rng.integers(0, K, size=n).astype(np.int32)
    w = rng.uniform(0.0, 1.0, size=(n, K)).astype(np.float32)
    w[rng.random((n, K)) < 0.4] = 0.0
    om = oracle.OracleMap(K, float(np.float32(res)), 8, l, 0.5, float(np.float32(1e-3)))
    if soft:
        om.insert_scan_soft(xyz, w, (0, 0, 0), 0.0)
    else:
        om.insert_scan(xyz, lab, (0, 0, 0), 0.0)
    ijk, a_ref, nv, nb = om.export()
    for B, budget in ((2, 64), (4, 64), (8, 96), (16, 96)):
        print(f"[case] small stencil l/res={lv} B={B} soft={soft}", flush=True)
        m = SemanticMap(res, B, l, 0.5, K, 1e-3, unit_budget=budget)
        if soft:
            m.insert_scan_soft(cuda(xyz), cuda(w), (0, 0, 0), 0.0)
        else:
            m.insert_scan(cuda(xyz), cuda(lab), (0, 0, 0), 0.0)
        a = m.query(cuda(ijk.astype(np.int32)))["alpha"].cpu().numpy()
        assert np.max(np.abs(a - a_ref) / a_ref) <= 1e-5
        st = m.stats()
        assert abs(st["n_pairs"] - int(nv.sum())) <= int(nb.sum())
        torch.cuda.synchronize()


@pytest.mark.parametrize("lv", [0.9, 1.9, 2.9, 3.9])
@pytest.mark.parametrize("K,budget", [(3, 0), (70, 64)])
def test_merge_of_small_blocks(lv, K, budget):
    # blocks of 4^3, reach 1 to 4: classes beyond one wavefront, slots of one unit,
    # of several and of more than 64, rows at the window's corners, a second insert
    # on top of the first, its replay, and 64-bit offsets of partial sums
    from paper_1909_04631_amd import SemanticMap
    res = 0.2
    l = float(np.float32(lv) * np.float32(res))
    rng = np.random.default_rng(int(10 * lv) + K)
    n = 9_000
    xyz = rng.uniform(-3.0, 3.0, size=(n, 3)).astype(np.float32)
    xyz[: n // 2] = np.float32(0.5) + rng.uniform(0, 0.2, size=(n // 2, 3)).astype(np.float32)
    lab = rng.integers(0, K, size=n).astype(np.int32)
    lab[: n // 2] = K - 1
    om = oracle.OracleMap(K, float(np.float32(res)), 4, l, 0.5, float(np.float32(1e-3)))
    gm, rm, wm, wr = [SemanticMap(res, 4, l, 0.5, K, 1e-3, unit_budget=budget,
                                  initial_blocks=1 << 14, wide_offsets=w)
                      for w in (False, False, True, True)]
    for step, rows in enumerate((slice(0, n), slice(0, n, 3))):
        print(f"[case] merge B=4 l/res={lv} K={K} budget={budget} insert {step}", flush=True)
        x, y = np.ascontiguousarray(xyz[rows]), np.ascontiguousarray(lab[rows])
        om.insert_scan(x, y, (0, 0, 0), 0.0)
        gm.insert_scan(cuda(x), cuda(y), (0, 0, 0), 0.0)
        ijk, a_ref, _, _ = om.export()
        q = cuda(ijk.astype(np.int32))
        a = gm.query(q)["alpha"].cpu().numpy()
        assert np.max(np.abs(a - a_ref) / a_ref) <= 1e-5
        # 64-bit offsets of partial sums, and the replays, give the same bits
        wm.insert_scan(cuda(x), cuda(y), (0, 0, 0), 0.0)
        assert np.array_equal(wm.query(q)["alpha"].cpu().numpy(), a)
        for m in (rm, wr):
            g = m.batch_capture(cuda(x), cuda(y), [0, x.shape[0]], [(0.0, 0.0, 0.0)], 0.0)
            m.reset()      # (the capture inserts once)
            if step == 1:
                m.insert_scan(cuda(xyz), cuda(lab), (0, 0, 0), 0.0)
            g.replay([0, x.shape[0]], [(0.0, 0.0, 0.0)])
            m.sync()
            assert np.array_equal(m.query(q)["alpha"].cpu().numpy(), a)
            g.close()
    if budget:
        assert gm.stats()["n_units"] > 1_500 // budget
