"""Edges of the kernels' size classes and dispatch rules, with inputs made for
them: per-tile sort sizes on few and on many tiles, footprints that only a caller's
own arrays can hold (indefinite conics, opacities above the cap), slot lists of
every length class, predicate bytes at odd sizes and addresses."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    return torch


@pytest.fixture(scope="module")
def gs():
    from paper_2607_19893_amd import gsmi
    return gsmi


def host_u32(t, k=None):
    a = t.detach().cpu().numpy().view(np.uint32).reshape(-1)
    return a if k is None else a[:k]


SORT_SIZES = [1, 63, 64, 65, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4096, 4097]


# 256 and 512 tiles (at most two per compute unit), 528 and 1200 (more), 7500 (a block's
# counters cover the range of its own tiles) and 37,500 (several passes over them); every
# depth of a tile another, runs of 2 to 9 equal ones, and one of 100 in the longer tiles
@pytest.mark.parametrize("ties", ["none", "short", "long"])
@pytest.mark.parametrize("width,height", [(256, 256), (512, 256), (528, 256), (640, 480), (1600, 1200), (4000, 2400)])
def test_bin_sort_sizes(width, height, ties, torch_gpu, gs):
    torch = torch_gpu
    rng = np.random.default_rng(width)
    TX, TY = (width + 15) // 16, (height + 15) // 16
    T = TX * TY
    special = rng.choice(T, len(SORT_SIZES), replace=False)
    other = np.setdiff1d(np.arange(T), special)
    tile = np.concatenate([np.full(k, t) for t, k in zip(special, SORT_SIZES)] + [rng.choice(other, 3000)]).astype(np.int64)
    rng.shuffle(tile)
    n = tile.size
    # a primitive covers its tile, every seventh two beside each other where neither is special
    x0, y0 = tile % TX, tile // TX
    wide = (np.arange(n) % 7 == 0) & (x0 + 1 < TX) & ~np.isin(tile, special) & ~np.isin(tile + 1, special)
    assert wide.sum() > 50
    rect = np.stack([x0, y0, x0 + 1 + wide, y0 + 1], 1).astype(np.int16)
    depth = (1.0 + rng.permutation(n) * 2.0 ** -14).astype(np.float32)
    assert np.unique(depth).size == n
    for t in special:
        at = np.flatnonzero(tile == t)
        if ties == "short":
            k = 0
            while k < at.size:
                run = int(rng.integers(2, 10))
                depth[at[k:k + run]] = depth[at[k]]
                k += 3 * run
        elif ties == "long" and at.size > 120:
            depth[rng.choice(at, 100, replace=False)] = np.float32(1.5)
    assert np.array_equal(np.bincount(np.concatenate([tile, tile[wide] + 1]), minlength=T)[special], SORT_SIZES)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    u32 = lambda k: torch.zeros(max(1, k), dtype=torch.int32, device="cuda")  # noqa: E731
    f = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
    keep = dict(radius=u32(n), tiles=dev((1 + wide).astype(np.int32)), rect=dev(rect), depth=dev(depth), mean2d=f(n, 2),
                conic_opacity=f(n, 4), rgb=f(n, 3), clamp=torch.zeros(n, dtype=torch.uint8, device="cuda"))
    proj = gs.make_proj(**keep)
    M = int((1 + wide).sum())
    cap = M + 5
    vals, emit, ranges, order, off = u32(cap), u32(cap), u32(2 * T), u32(T), u32(n)
    cnt, status = u32(2), u32(4)
    ws = torch.zeros(gs.gs_workspace_bytes(gs.GS_WS_BIN_SORT, n, cap, width, height), dtype=torch.uint8, device="cuda")
    gs.gs_bin_sort(proj, n, dev(np.arange(n, dtype=np.int32)), dev(np.array([n], np.int32)), width, height, cap, vals,
                   ranges, off, emit, None, cnt[:1], status, ws, tile_order=order)
    torch.cuda.synchronize()
    assert host_u32(status)[0] == 0 and host_u32(cnt)[0] == M
    ids = np.concatenate([np.arange(n), np.flatnonzero(wide)])
    tiles = np.concatenate([tile, tile[wide] + 1])
    ref = np.lexsort((ids, depth[ids].view(np.uint32), tiles))
    np.testing.assert_array_equal(host_u32(vals, M), ids[ref])
    count = np.bincount(tiles, minlength=T)
    start = np.cumsum(count) - count
    np.testing.assert_array_equal(host_u32(ranges).reshape(T, 2)[count > 0], np.stack([start, start + count], 1)[count > 0])
    # each sorted pair names the emission position of its (primitive, tile)
    first = np.cumsum(1 + wide) - (1 + wide)
    np.testing.assert_array_equal(host_u32(emit, M), (first[ids] + (tiles != tile[ids]))[ref])


# ids without tiles: none, every third, all but one in a hundred (a block of 2048 pairs
# then spans more ranks than it has pairs)
@pytest.mark.parametrize("empty", [0.0, 0.34, 0.99])
def test_bin_sort_rectangles(empty, torch_gpu, gs):
    """Rectangles of 1 to 6000 tiles, beginning and ending anywhere in a thread's eight
    pairs and a block's 2048."""
    torch = torch_gpu
    width, height = 1600, 1216
    TX, TY = 100, 76
    T = TX * TY
    rng = np.random.default_rng(int(empty * 100))
    n = 60000 if empty > 0.9 else 3000
    w, h = rng.integers(1, 6, n), rng.integers(1, 6, n)
    big = rng.choice(n, n // 100, replace=False)
    w[big], h[big] = rng.integers(1, TX + 1, big.size), rng.integers(1, 61, big.size)
    w[big[0]], h[big[0]] = TX, 60
    x0, y0 = rng.integers(0, TX - w + 1), rng.integers(0, TY - h + 1)
    tiles = np.where(rng.uniform(size=n) < empty, 0, w * h)
    tiles[big[0]] = TX * 60
    rect = np.stack([x0, y0, x0 + w, y0 + h], 1).astype(np.int16)
    depth = rng.uniform(1.0, 9.0, n).astype(np.float32)
    listed = rng.permutation(n).astype(np.int32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    u32 = lambda k: torch.zeros(max(1, k), dtype=torch.int32, device="cuda")  # noqa: E731
    f = lambda *s: torch.zeros(*s, device="cuda")  # noqa: E731
    keep = dict(radius=u32(n), tiles=dev(tiles.astype(np.int32)), rect=dev(rect), depth=dev(depth), mean2d=f(n, 2),
                conic_opacity=f(n, 4), rgb=f(n, 3), clamp=torch.zeros(n, dtype=torch.uint8, device="cuda"))
    M = int(tiles.sum())
    cap = M + 7
    vals, emit, ranges, order, off = u32(cap), u32(cap), u32(2 * T), u32(T), u32(n)
    cnt, status = u32(2), u32(4)
    ws = torch.zeros(gs.gs_workspace_bytes(gs.GS_WS_BIN_SORT, n, cap, width, height), dtype=torch.uint8, device="cuda")
    gs.gs_bin_sort(gs.make_proj(**keep), n, dev(listed), dev(np.array([n], np.int32)), width, height, cap, vals, ranges,
                   off, emit, None, cnt[:1], status, ws, tile_order=order)
    torch.cuda.synchronize()
    assert host_u32(status)[0] == 0 and host_u32(cnt)[0] == M
    ids = np.repeat(listed, tiles[listed])
    local = np.arange(M) - np.repeat(np.cumsum(tiles[listed]) - tiles[listed], tiles[listed])
    tile = (y0[ids] + local // w[ids]) * TX + x0[ids] + local % w[ids]
    ref = np.lexsort((ids, depth[ids].view(np.uint32), tile))
    np.testing.assert_array_equal(host_u32(vals, M), ids[ref])
    np.testing.assert_array_equal(host_u32(emit, M), ref)
    count = np.bincount(tile, minlength=T)
    start = np.cumsum(count) - count
    np.testing.assert_array_equal(host_u32(ranges).reshape(T, 2)[count > 0], np.stack([start, start + count], 1)[count > 0])


def reference(u, con, op, rgb, order, W, H, dL):
    """Image, final T, and the gradients of (u, v, A, B, C, opacity, rgb) in 64 bits, every
    pixel blending all pairs in order; with each pixel's distance to its nearest decision."""
    import torch
    q = torch.tensor(np.concatenate([u, con, op[:, None], rgb], 1)[order], dtype=torch.float64, requires_grad=True)
    ys, xs = np.mgrid[0:H, 0:W]
    px = torch.tensor(xs.reshape(-1) + 0.5, dtype=torch.float64)[:, None]
    py = torch.tensor(ys.reshape(-1) + 0.5, dtype=torch.float64)[:, None]
    dx, dy = q[:, 0] - px, q[:, 1] - py
    sig = 0.5 * (q[:, 2] * dx * dx + q[:, 4] * dy * dy) + q[:, 3] * dx * dy
    raw = q[:, 5] * torch.exp(-sig)
    al = torch.clamp(raw, max=float(np.float32(0.99)))
    with torch.no_grad():
        ok = (sig >= 0) & (al >= float(np.float32(1 / 255)))
        T = torch.cumprod(1 - al * ok, 1)
        take = ok & (T >= float(np.float32(1e-4)))
        near = torch.minimum((al * 255 - 1).abs().amin(1), torch.where(ok, (T / 1e-4 - 1).abs(), 1.0).amin(1))
        near = torch.minimum(near, (raw / 0.99 - 1).abs().amin(1))
        near = torch.minimum(near, torch.where(raw.detach() * 255 > 0.9, sig.abs() * 1e3 + (sig == 0), 1.0).amin(1))
    al = al * take
    Tk = torch.cumprod(torch.cat([torch.ones(al.shape[0], 1, dtype=torch.float64), 1 - al[:, :-1]], 1), 1)
    img = ((al * Tk)[:, :, None] * q[:, 6:9]).sum(1)
    (img * torch.tensor(dL.reshape(3, -1).T.astype(np.float64))).sum().backward()
    g = np.zeros((len(order), 9))
    g[order] = q.grad.numpy()
    last = np.where(take.any(1), take.shape[1] - torch.flip(take, [1]).int().argmax(1).numpy(), 0)
    return img.detach().numpy().T.reshape(3, H, W), (Tk[:, -1] * (1 - al[:, -1])).detach().numpy().reshape(H, W), g, \
        near.numpy().reshape(H, W), last.reshape(H, W)


# one pair; the edges of a backward batch (64) and of a forward batch (256), several batches
@pytest.mark.parametrize("n,width,height", [(1, 16, 16), (64, 37, 29), (65, 37, 29), (257, 24, 41), (700, 21, 18)])
def test_raster_special_pairs(n, width, height, torch_gpu):
    """Every pair in every tile's list, among them indefinite conics, opacities above the
    0.99 cap and below 1/255, and thin footprints centred far outside the image."""
    from paper_2607_19893_amd import scenes
    from paper_2607_19893_amd.pipeline import ViewTrainer
    torch = torch_gpu
    rng = np.random.default_rng(1000 + n)
    sc = scenes.tiny(n=n).scene
    cam = scenes.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), (0.0, -1.0, 0.0), width, height, 60.0)
    tx, ty = (width + 15) // 16, (height + 15) // 16
    tr = ViewTrainer(sc, capacity=n * tx * ty + 64, max_width=width, max_height=height, with_replica=False)
    uv = rng.uniform(-6, 1, (n, 2)) + rng.random((n, 2)) * [width + 10, height + 10]
    s1, s2 = np.exp(rng.uniform(-0.5, 2.5, n)), np.exp(rng.uniform(-0.5, 2.5, n))
    th = rng.uniform(0, np.pi, n)
    op = rng.uniform(0.02, 0.35, n)
    kind = np.arange(n) % 11 if n > 1 else np.array([0])
    op[kind == 3] = rng.uniform(0.991, 1.0, (kind == 3).sum())
    op[kind == 5] = rng.uniform(0.0, 0.0039, (kind == 5).sum())
    far = kind == 7                                     # thin, 150..300 px long, centred off the image
    s1[far], s2[far] = rng.uniform(60, 120, far.sum()), 0.6
    uv[far] += np.stack([np.cos(th[far]), np.sin(th[far])], 1) * rng.uniform(80, 150, far.sum())[:, None]
    c, s = np.cos(th), np.sin(th)
    A, B, C = (c / s1) ** 2 + (s / s2) ** 2, c * s * (s1 ** -2 - s2 ** -2), (s / s1) ** 2 + (c / s2) ** 2
    bad = kind == 9                                     # indefinite: sigma < 0 in a double wedge
    B[bad] = np.sqrt(A[bad] * C[bad]) * rng.uniform(1.05, 2.0, bad.sum())
    u32f = lambda a: np.ascontiguousarray(a, np.float32)  # noqa: E731
    uv, con, op = u32f(uv), u32f(np.stack([A, B, C], 1)), u32f(op)
    rgb = u32f(rng.random((n, 3)))
    depth = u32f(rng.permutation(n) + 1.0)
    dL = u32f(rng.uniform(-1, 1, (3, height, width)))
    order = np.argsort(depth)
    img, fT, _, near, last = reference(uv, con, op, rgb, order, width, height, dL)
    sure = near > 2e-5              # fp32 alpha and T of these few hundred pairs lie closer than that to the 64-bit ones
    assert sure.mean() > 0.97
    dL *= sure                      # an undecided pixel passes on no gradient
    g = reference(uv, con, op, rgb, order, width, height, dL)[2]
    tr.project(cam)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tr.tiles.copy_(dev(np.full(n, tx * ty, np.int32)))
    tr.rect.copy_(dev(np.tile(np.array([0, 0, tx, ty], np.int16), (n, 1))))
    tr.depth.copy_(dev(depth))
    tr.mean2d.copy_(dev(uv))
    tr.conic.copy_(dev(np.concatenate([con, op[:, None]], 1)))
    tr.rgb.copy_(dev(rgb))
    tr.clamp.zero_()
    tr.visible()
    tr.bin_sort()
    tr.raster_fwd(active=True)
    tr.set_dL(dL)
    tr.raster_bwd(grad2d=True)
    torch.cuda.synchronize()
    assert tr.host_status()[0] == 0
    hw = width * height
    got = tr.img.view(-1)[:3 * hw].cpu().numpy().reshape(3, height, width)
    # T after k pairs carries 2k roundings of 2^-24: 700 pairs, 8.4e-5
    assert np.abs(got - img)[:, sure].max() <= 1e-4
    assert np.abs(tr.final_T.view(-1)[:hw].cpu().numpy().reshape(height, width) - fT)[sure].max() <= 1e-4
    np.testing.assert_array_equal(host_u32(tr.n_contrib, hw).reshape(height, width)[sure], last[sure])
    g2 = tr.grad2d.cpu().numpy()[:n].astype(np.float64)
    # a term passes through T's 2n roundings forward and as many back; sums cancel to a
    # column's rms at most
    bound = (4 * n + 200) * 2.0 ** -24 * (np.abs(g) + np.sqrt((g ** 2).mean(0)))
    assert (np.abs(g2 - g) <= bound + 1e-9).all(), np.abs((g2 - g) / (bound + 1e-12)).max(0)


# lists of every length class of the slot sums, on few and on many visible rows
@pytest.mark.parametrize("V", [5, 700, (1 << 17), (1 << 17) + 77])
def test_slot_sums(V, torch_gpu):
    from paper_2607_19893_amd import scenes
    from paper_2607_19893_amd.pipeline import ViewTrainer
    torch = torch_gpu
    rng = np.random.default_rng(V)
    nt = rng.integers(1, 5, V)
    special = [1, 7, 8, 9, 39, 40, 41, 64, 255, 256, 257, 1000]
    at = rng.choice(V, min(V, 5 * len(special)), replace=False)
    nt[at] = np.resize(special, at.size)
    M = int(nt.sum())
    sc = scenes.tiny(n=V).scene
    cam = scenes.tiny(n=10).cameras[0]
    tr = ViewTrainer(sc, capacity=M, max_width=cam.width, max_height=cam.height, with_replica=False)
    tr.project(cam)
    off = np.cumsum(nt) - nt
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tr.vis_idx.copy_(dev(np.arange(V, dtype=np.int32)))
    tr.counts[0:1].copy_(dev(np.array([V], np.int32)))
    tr.tiles.copy_(dev(nt.astype(np.int32)))
    tr.pair_offset.copy_(dev(off.astype(np.int32)))
    tr.conic.copy_(dev(np.tile(np.array([1, 0, 1, 1], np.float32), (V, 1))))
    slots = rng.standard_normal((M, 12)).astype(np.float32)      # nine sums and padding per pair
    # whole numbers in lists of more than 40 slots: four of them add up below 2^24, exactly in
    # 32 bits, and all of a list's do not
    long_slots = np.repeat(nt > 40, nt)
    slots[long_slots] = rng.integers(1 << 20, 1 << 22, (long_slots.sum(), 12))
    tr.ws_bwd.view(torch.float32)[:M * 12].copy_(dev(slots.reshape(-1)))
    tr.raster_bwd_project(grad2d=True)
    torch.cuda.synchronize()
    s = np.add.reduceat(slots[:, :9].astype(np.float64), off, 0)
    mag = np.add.reduceat(np.abs(slots[:, :9]).astype(np.float64), off, 0)
    scale = np.array([1, 1, 0.5, 1, 0.5, -1, 1, 1, 1])
    err = np.abs(tr.grad2d.cpu().numpy()[:V] - s * scale)
    # at most 4 + 8 + 6 additions in a row per value, each 2^-24 of the summed magnitudes
    assert (err <= 20 * 2.0 ** -24 * mag * np.abs(scale) + 1e-12).all()
    # lists of more than 40 slots: four of a lane's in 32 bits, which is exact here, the rest in
    # 64 bits, rounded once
    many = nt > 40
    assert (err <= 1.001 * 2.0 ** -24 * np.abs(s * scale) + 1e-12)[many].all()


@pytest.mark.parametrize("n", [1, 31, 32, 33, 8191, 8193, 100003])
@pytest.mark.parametrize("shift", [0, 1, 16])
def test_scope_from_bytes(n, shift, torch_gpu, gs):
    torch = torch_gpu
    rng = np.random.default_rng(n + shift)
    a = np.where(rng.random(n) < 0.3, rng.choice([1, 2, 127, 128, 255], n), 0).astype(np.uint8)
    buf = torch.full((n + shift + 64,), 255, dtype=torch.uint8, device="cuda")
    buf[shift:shift + n] = torch.from_numpy(a).cuda()
    words = gs.scope_words(n)
    sc = torch.full((words + 1,), -1, dtype=torch.int32, device="cuda")
    gs.gs_scope_from_pred(gs.GS_PRED_U8_NONZERO, buf[shift:shift + n], n, 0, sc)
    bits = np.zeros(words * 32, np.uint8)
    bits[:n] = a != 0
    ref = np.packbits(bits, bitorder="little").view(np.uint32)
    np.testing.assert_array_equal(host_u32(sc, words), ref)
    assert host_u32(sc)[words] == 0xFFFFFFFF
    b = (rng.random(n) < 0.2).astype(np.uint8)
    buf[shift:shift + n] = torch.from_numpy(b).cuda()
    gs.gs_scope_from_pred(gs.GS_PRED_U8_NONZERO, buf[shift:shift + n], n, 1, sc)
    bits[:n] |= b
    np.testing.assert_array_equal(host_u32(sc, words), np.packbits(bits, bitorder="little").view(np.uint32))


# 32,768 blocks of 8192 ids are summed by the scatter itself, one more by a pass of its own
@pytest.mark.parametrize("n", [4096 * 8192 + 5, 32768 * 8192, 32768 * 8192 + 5])
def test_hazard_lists_over_many_blocks(n, torch_gpu, gs):
    torch = torch_gpu
    rng = np.random.default_rng(3)
    sets = [np.unique(np.concatenate([rng.integers(0, n, 20000), [0, n - 1]])) for _ in range(2)]
    RA, WB = sets
    WA = np.unique(np.concatenate([RA[::2], rng.integers(0, n, 500)]))
    RB = np.unique(np.concatenate([WB, RA[::3], WA[::5]]))

    def scope(ids):
        w = np.zeros(gs.scope_words(n), np.uint32)
        np.bitwise_or.at(w, ids >> 5, np.uint32(1) << (ids & 31).astype(np.uint32))
        return torch.from_numpy(w.view(np.int32)).cuda()

    s = [scope(x) for x in (RA, WA, RB, WB)]
    out = [torch.zeros(gs.scope_words(n), dtype=torch.int32, device="cuda") for _ in range(3)]
    ids = [torch.zeros(60000, dtype=torch.int32, device="cuda") for _ in range(3)]
    counts = torch.zeros(4, dtype=torch.int32, device="cuda")
    # a workspace at any word's address will do
    ws = torch.zeros(gs.gs_workspace_bytes(gs.GS_WS_SCOPE, n) + 4, dtype=torch.uint8, device="cuda")[4:]
    gs.gs_scope_conflicts(*s, n, *out, *ids, counts, ws)
    ref = [np.intersect1d(WB, WA), np.intersect1d(np.setdiff1d(RB, WB), WA),
           np.setdiff1d(np.intersect1d(WB, RA), WA)]
    np.testing.assert_array_equal(host_u32(counts), [r.size for r in ref] + [RB.size])
    for t, r in zip(ids, ref):
        np.testing.assert_array_equal(host_u32(t, r.size), r)


def blend_arrays(torch, uv, con, op, rgb, depth, width, height, dL):
    """The forward's and the backward's outputs of a caller's own projection arrays, every
    pair in every tile's list."""
    from paper_2607_19893_amd import scenes
    from paper_2607_19893_amd.pipeline import ViewTrainer
    n = len(op)
    cam = scenes.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), (0.0, -1.0, 0.0), width, height, 60.0)
    tx, ty = (width + 15) // 16, (height + 15) // 16
    tr = ViewTrainer(scenes.tiny(n=n).scene, capacity=n * tx * ty + 64, max_width=width, max_height=height,
                     with_replica=False)
    tr.project(cam)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    tr.tiles.copy_(dev(np.full(n, tx * ty, np.int32)))
    tr.rect.copy_(dev(np.tile(np.array([0, 0, tx, ty], np.int16), (n, 1))))
    tr.depth.copy_(dev(depth))
    tr.mean2d.copy_(dev(uv))
    tr.conic.copy_(dev(np.concatenate([con, op[:, None]], 1)))
    tr.rgb.copy_(dev(rgb))
    tr.clamp.zero_()
    tr.visible()
    tr.bin_sort()
    tr.active.zero_()
    tr.raster_fwd(active=True)
    tr.set_dL(dL)
    tr.raster_bwd(grad2d=True)
    torch.cuda.synchronize()
    assert tr.host_status()[0] == 0
    hw = width * height
    return dict(img=tr.img.view(-1)[:3 * hw].cpu().numpy().reshape(3, height, width),
                final_T=tr.final_T.view(-1)[:hw].cpu().numpy(), n_contrib=host_u32(tr.n_contrib, hw),
                active=tr.active.cpu().numpy()[:n], grad2d=tr.grad2d.cpu().numpy()[:n],
                grad_rows=tr.grad_rows.cpu().numpy()[:n])


def ordinary_pairs(rng, n, width, height):
    """Centres, conics, opacities, colours of n definite footprints over the image."""
    f32 = lambda a: np.ascontiguousarray(a, np.float32)  # noqa: E731
    uv = rng.uniform(-6, 6, (n, 2)) + rng.random((n, 2)) * [width, height]
    s1, s2 = np.exp(rng.uniform(-0.5, 2.5, n)), np.exp(rng.uniform(-0.5, 2.5, n))
    c, s = np.cos(th := rng.uniform(0, np.pi, n)), np.sin(th)
    con = np.stack([(c / s1) ** 2 + (s / s2) ** 2, c * s * (s1 ** -2 - s2 ** -2), (s / s1) ** 2 + (c / s2) ** 2], 1)
    return f32(uv), f32(con), f32(rng.uniform(0.02, 0.3, n)), f32(rng.random((n, 3)))


@pytest.mark.parametrize("n", [3, 400])
def test_raster_far_centres(n, torch_gpu):
    """Pairs whose sigma over the whole image is past every cut-off, up to the end of the
    fp32 range and at infinite centres and conics, leave everything as if they had no
    opacity, and get no gradient themselves."""
    width, height = 37, 29
    rng = np.random.default_rng(n)
    uv, con, op, rgb = ordinary_pairs(rng, n, width, height)
    inf, big = np.inf, np.float32(3.4e38)
    far = [(u, v, A, B, C) for u, v in ((1e20, 3), (5, -1e20), (-2e19, 2e19), (inf, 4), (7, -inf), (inf, inf),
                                        (big, -big), (1e12, 1e12), (-3e4, 3e4), (9, 5e3))
           for A, B, C in ((1, 0, 1), (1, 0.5, 1), (3.3, -3.2, 3.3), (0.3, 0, 3.0))]
    far += [(8, 8, *abc) for abc in ((inf, 0, 1), (1, inf, 1), (1, 0, inf), (big, 0, big), (inf, inf, inf),
                                     (-inf, 0, 1), (0, 0, inf), (1, -inf, 1))]
    far = np.array(far, np.float32)
    far[(far[:, :2] == 8).all(1), :2] = [8.25, 8.25]      # (big, 0, big): off every pixel centre
    k = len(far)
    fop = np.resize(np.array([0.5, 0.99, 0.999, 0.05], np.float32), k)
    at = rng.permutation(n + k)                             # far pairs anywhere in the depth order
    join = lambda a, b: np.ascontiguousarray(np.concatenate([a, b])[at], np.float32)  # noqa: E731
    depth = np.arange(1, n + k + 1, dtype=np.float32)
    arrays = (join(uv, far[:, :2]), join(con, far[:, 2:]))
    col = join(rgb, rng.random((k, 3)))
    dL = rng.uniform(-1, 1, (3, height, width)).astype(np.float32)
    got = blend_arrays(torch_gpu, *arrays, join(op, fop), col, depth, width, height, dL)
    ref = blend_arrays(torch_gpu, *arrays, join(op, np.zeros(k)), col, depth, width, height, dL)
    is_far = at >= n
    assert np.isfinite(ref["img"]).all() and (ref["n_contrib"] > 0).any()
    for name in ("img", "final_T", "n_contrib", "active"):
        np.testing.assert_array_equal(got[name], ref[name], err_msg=name)
    np.testing.assert_array_equal(got["grad2d"][~is_far], ref["grad2d"][~is_far])
    np.testing.assert_array_equal(got["grad_rows"][~is_far], ref["grad_rows"][~is_far])
    finite = is_far & np.isfinite(arrays[0]).all(1) & np.isfinite(arrays[1]).all(1)
    assert (got["grad2d"][finite] == 0).all()


def test_raster_distant_needles(torch_gpu):
    """Footprints a pixel wide whose centres lie 1500 to 3000 px off the image along their
    axis: the terms of sigma are 1e6 and more, sigma itself a few."""
    width, height, n = 40, 33, 300
    rng = np.random.default_rng(5)
    uv, con, op, rgb = ordinary_pairs(rng, n, width, height)
    th = rng.uniform(0, np.pi, n)
    c, s = np.cos(th), np.sin(th)
    s1, s2 = rng.uniform(900, 1200, n), 0.6
    con = np.stack([(c / s1) ** 2 + (s / s2) ** 2, c * s * (s1 ** -2 - s2 ** -2), (s / s1) ** 2 + (c / s2) ** 2], 1)
    con = con.astype(np.float32)
    d = rng.uniform(1500, 3000, n) * rng.choice([-1, 1], n)
    uv = (uv + np.stack([c, s], 1) * d[:, None]).astype(np.float32)
    op[:] = rng.uniform(0.3, 0.985, n)
    keep = con[:, 0].astype(np.float64) * con[:, 2] > con[:, 1].astype(np.float64) ** 2
    uv, con, op, rgb = (a[keep] for a in (uv, con, op, rgb))
    n = len(op)
    assert n > 250
    depth = rng.permutation(n).astype(np.float32) + 1
    order = np.argsort(depth)
    dL = rng.uniform(-1, 1, (3, height, width)).astype(np.float32)
    img, fT, _, near, last = reference(uv, con, op, rgb, order, width, height, dL)
    sure = near > 2e-5
    dL *= sure
    g = reference(uv, con, op, rgb, order, width, height, dL)[2]
    got = blend_arrays(torch_gpu, uv, con, op, rgb, depth, width, height, dL)
    assert sure.mean() > 0.97 and (last > 0).mean() > 0.5
    # T after k pairs carries 2k roundings of 2^-24: 300 pairs, 3.6e-5
    assert np.abs(got["img"] - img)[:, sure].max() <= 1e-4
    np.testing.assert_array_equal(got["n_contrib"].reshape(height, width)[sure], last[sure])
    bound = (4 * n + 200) * 2.0 ** -24 * (np.abs(g) + np.sqrt((g ** 2).mean(0)))
    # (u, v)'s are differences of moments some thousand times their size
    assert (np.abs(got["grad2d"] - g) <= bound + 1e-9)[:, 2:].all(), np.abs((got["grad2d"] - g) / bound).max(0)


def test_raster_colours_not_finite(torch_gpu):
    """An infinite or NaN colour reaches the pixels that include its pair, and the gradients
    of the pairs that share such a pixel, and nothing else."""
    width, height, n = 61, 45, 330
    rng = np.random.default_rng(8)
    uv, con, op, rgb = ordinary_pairs(rng, n, width, height)
    con *= np.float32(4.0)                                  # footprints of a few pixels
    depth = rng.permutation(n).astype(np.float32) + 1
    dL = rng.uniform(0.1, 1, (3, height, width)).astype(np.float32)
    bad = rng.choice(n, 4, replace=False)
    op[bad] = 0.3
    run = lambda c, d: blend_arrays(torch_gpu, uv, con, op, c, depth, width, height, d)  # noqa: E731
    black, white, col = rgb.copy(), rgb.copy(), rgb.copy()
    black[bad], white[bad] = 0, 1
    col[bad] = np.array([[np.inf, 0, 0], [0, np.nan, 0], [0, 0, -np.inf], [np.inf, np.nan, 1]], np.float32)
    ref, got = run(black, dL), run(col, dL)
    hit = (run(white, dL)["img"] != ref["img"]).any(0)      # pixels that include one of the four
    assert 10 < hit.sum() < 0.3 * hit.size
    for name in ("final_T", "n_contrib", "active"):
        np.testing.assert_array_equal(got[name], ref[name], err_msg=name)
    np.testing.assert_array_equal(got["img"][:, ~hit], ref["img"][:, ~hit])
    assert not np.isfinite(got["img"][:, hit]).all(0).any()
    clear = (run(black, dL * hit)["grad2d"] == 0).all(1)    # pairs that no such pixel includes
    clear[bad] = False
    assert clear.sum() > 50
    np.testing.assert_array_equal(got["grad2d"][clear], ref["grad2d"][clear])


def test_raster_bwd_opacity_at_the_cap(torch_gpu):
    """o e^-sigma equal to the 0.99 cap of alpha stops the gradients of opacity and sigma."""
    uv = np.array([[5.5, 9.5]], np.float32)
    con, op = np.array([[1, 0, 1]], np.float32), np.array([0.99], np.float32)
    dL = np.zeros((3, 16, 16), np.float32)
    dL[:, 9, 5] = 1.0
    got = blend_arrays(torch_gpu, uv, con, op, np.full((1, 3), 0.5, np.float32), np.ones(1, np.float32), 16, 16, dL)
    np.testing.assert_array_equal(got["grad2d"][0, :6], 0)
    np.testing.assert_array_equal(got["grad2d"][0, 6:], np.float32(0.99))


def test_raster_bwd_small_offsets(torch_gpu):
    """Centres 2e-4 to 5e-3 px off a pixel centre, one included pixel each: the moments keep
    the offsets' own precision, not that of their distance to a strip or a tile."""
    width, height = 48, 40
    rng = np.random.default_rng(4)
    px, py = [a.reshape(-1) for a in np.meshgrid(np.arange(0, width, 3), np.arange(0, height))]
    n = px.size
    off = rng.uniform(2e-4, 5e-3, (n, 2)) * rng.choice([-1, 1], (n, 2))
    uv = (np.stack([px, py], 1) + 0.5 + off).astype(np.float32)
    con = np.tile(np.array([4000, 900, 4800], np.float32), (n, 1))
    op = rng.uniform(0.1, 0.9, n).astype(np.float32)
    rgb = rng.uniform(0.2, 1, (n, 3)).astype(np.float32)
    dL = rng.uniform(0.2, 1, (3, height, width)).astype(np.float32)
    got = blend_arrays(torch_gpu, uv, con, op, rgb, rng.permutation(n).astype(np.float32) + 1, width, height, dL)
    d = uv.astype(np.float64) - np.stack([px, py], 1) - 0.5
    A, B, C = con.astype(np.float64).T
    sigma = 0.5 * (A * d[:, 0] ** 2 + C * d[:, 1] ** 2) + B * d[:, 0] * d[:, 1]
    ds = -(dL[:, py, px].T.astype(np.float64) * rgb).sum(1) * op * np.exp(-sigma)
    x, y = d.T
    ref = ds[:, None] * np.stack([A * x + B * y, B * x + C * y, x * x / 2, x * y, y * y / 2], 1)
    mag = np.abs(ds)[:, None] * np.stack([abs(A * x) + abs(B * y), abs(B * x) + abs(C * y), x * x / 2, abs(x * y),
                                          y * y / 2], 1)
    # alpha, T and dL/dalpha carry about ten roundings, the offsets and products four more
    assert (np.abs(got["grad2d"][:, :5] - ref) <= 24 * 2.0 ** -24 * mag).all(), \
        (np.abs(got["grad2d"][:, :5] - ref) / mag).max(0) * 2 ** 24
