"""Kernels at the edges of their tiles, splits and dispatch rules, against fp64 on the CPU."""
from __future__ import annotations

import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import gpu_util
    assert torch.cuda.is_available()
    return gpu_util


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


@pytest.mark.parametrize("n,splits", [(1, 0), (17, 1), (64, 0), (65, 0), (1000, 1), (4096, 0), (4097, 0), (9001, 0)])
def test_channel_exponents_over_sample_sizes(G, n, splits):
    """e_c = round(log2 rms_c - o) over every step-th row, step = ceil(n / 4096): one workgroup's share and several, with
    the work space of the smallest split count, and rows that are not next to each other (token-major views)."""
    L = G.L
    g = np.random.default_rng(n)
    hkv = 2
    mag = 2.0 ** g.uniform(-4.0, 4.0, size=(hkv, 128))
    K = W.round_to_bf16((g.standard_normal((1, hkv, n, 128)) * mag[None, :, None, :]).astype(np.float32))
    cfg = L.make_config(batch=1, n_q_heads=hkv, n_kv_heads=hkv, capacity=n, group_size=1, attn_splits=splits)
    h = L.lvr_create(cfg)
    try:
        Kd = G.to_device(K, "bf16").transpose(1, 2).contiguous().transpose(1, 2)
        L.lvr_build(h, Kd, Kd)
        e = L.lvr_export_channel_scales(h, cfg)[0].astype(np.float64)
    finally:
        L.lvr_destroy(h)
    step = (n + 4095) // 4096
    for kv in range(hkv):
        lg = 0.5 * np.log2((K[0, kv, ::step].astype(np.float64) ** 2).mean(axis=0))
        o = math.atan2(np.sin(2 * np.pi * lg).sum(), np.cos(2 * np.pi * lg).sum()) / (2 * np.pi)
        want = np.clip(np.rint(lg - o), -8, 8)
        # the offset is defined up to whole numbers; a channel within fp32's error of a rounding boundary may go either way
        shift = np.rint(np.median(e[kv] - want))
        sure = np.abs((lg - o) - np.floor(lg - o) - 0.5) > 1e-3
        assert np.array_equal(e[kv][sure], np.clip(want + shift, -8, 8)[sure]), (n, kv)


@pytest.mark.parametrize("batch,hkv,n", [(4, 8, 4096), (33, 1, 4096), (5, 8, 3009), (16, 8, 1025), (32, 8, 4097), (70, 8, 1100)])
def test_channel_exponents_of_many_heads(G, batch, hkv, n):
    """Where there are many (sequence, KV head) a workgroup adds up more rows, whole rounds of 64 and what is left of them: the exponents
    of every sequence are those of an index that holds it alone (other sums of the same squares, so a channel at a rounding boundary aside)."""
    L = G.L
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    mag = 2.0 ** (8.0 * torch.rand((batch, hkv, 1, 128), generator=g, device="cuda") - 4.0)
    K = (torch.randn((batch, hkv, n, 128), generator=g, device="cuda") * mag).to(torch.bfloat16)

    def exponents(rows):
        cfg = L.make_config(batch=rows.shape[0], n_q_heads=hkv, n_kv_heads=hkv, capacity=n, group_size=1)
        h = L.lvr_create(cfg)
        try:
            for _ in range(2):   # the second finds the tickets where the first left them
                L.lvr_build(h, rows, rows)
            return L.lvr_export_channel_scales(h, cfg).astype(np.int64)
        finally:
            L.lvr_destroy(h)

    got = exponents(K)
    lg = 0.5 * torch.log2(K[:, :, ::(n + 4095) // 4096].double().square().mean(dim=2)).cpu().numpy()
    for b in range(0, batch, 3):
        alone = exponents(K[b:b + 1].contiguous())[0]
        o = np.arctan2(np.sin(2 * np.pi * lg[b]).sum(-1), np.cos(2 * np.pi * lg[b]).sum(-1))[:, None] / (2 * np.pi)
        sure = np.abs((lg[b] - o) - np.floor(lg[b] - o) - 0.5) > 1e-3
        assert sure.mean() > 0.9 and np.array_equal(got[b][sure], alone[sure]), b


@pytest.mark.parametrize("batch,n", [(1, 65), (3, 4096), (1, 20000)])
def test_channel_exponents_of_builds_in_a_row(G, batch, n):
    """The last workgroup to end forms the exponents: a build after a build on the same index (tickets back at zero), with channels of
    other sizes, gives those of an index of its own."""
    L = G.L
    g = np.random.default_rng(n)
    cfg = L.make_config(batch=batch, n_q_heads=4, n_kv_heads=2, capacity=n, group_size=1)
    data = [G.to_device(W.round_to_bf16((g.standard_normal((batch, 2, n, 128)) * 2.0 ** g.uniform(-4, 4, size=(batch, 2, 1, 128))).astype(np.float32)), "bf16")
            for _ in range(3)]
    one = L.lvr_create(cfg)
    try:
        for Kd in data:
            L.lvr_build(one, Kd, Kd)
            fresh = L.lvr_create(cfg)
            try:
                L.lvr_build(fresh, Kd, Kd)
                want = L.lvr_export_channel_scales(fresh, cfg)
            finally:
                L.lvr_destroy(fresh)
            assert np.array_equal(L.lvr_export_channel_scales(one, cfg), want) and np.ptp(want) >= 4
    finally:
        L.lvr_destroy(one)


@pytest.mark.parametrize("r,S,groups", [(1, 4, 1), (1, 1, 65), (2, 2, 63), (4, 4, 64), (4, 1, 129), (8, 2, 65), (16, 4, 17)])
def test_6_bit_balls_enclose_their_members_tightly(G, r, S, groups):
    """Every group size and block count of the 6-bit build at the edges of its 64-group tiles, from a strided source with a
    tail of ungrouped keys, and once more for a chunk grouped out of the arena: the key rows come back unchanged, a member
    lies within the stored radius of the stored centre in the rescaled space, and the radius is at most the largest
    distance plus what rounding up adds (2^-12 of distance and centre norm, then up to bf16: 2^-7)."""
    L = G.L
    g = np.random.default_rng(groups * 100 + r)
    hkv, chunk = 2, 64
    n = groups * r + (r - 1)
    mag = 2.0 ** g.uniform(-3.0, 3.0, size=(hkv, 128))
    K = W.round_to_bf16((g.standard_normal((1, hkv, n + chunk, 128)) * mag[None, :, None, :]).astype(np.float32))
    cfg = L.make_config(batch=1, n_q_heads=hkv, n_kv_heads=hkv, capacity=n + chunk, group_size=r, n_subspaces=S, buffer_size=chunk)
    h = L.lvr_create(cfg)
    try:
        Kd = G.to_device(K, "bf16")
        first = Kd[:, :, :n].transpose(1, 2).contiguous().transpose(1, 2)
        L.lvr_build(h, first, first)
        L.lvr_append(h, Kd[:, :, n:].contiguous(), Kd[:, :, n:].contiguous())
        centres, radii, _, keys = L.lvr_export_index(h, cfg)
        fac = 2.0 ** L.lvr_export_channel_scales(h, cfg)[0].astype(np.float64)
        n_indexed = L.lvr_length(h)[1]
    finally:
        L.lvr_destroy(h)
    assert n_indexed == (n // r) * r + (chunk // r) * r
    assert np.array_equal(keys, W.f32_to_bf16_bits(K).reshape(keys.shape))
    ng = n_indexed // r
    for kv in range(hkv):
        x = K[0, kv, :n_indexed].astype(np.float64).reshape(ng, r, 128) / fac[kv]
        c = (centres[0, kv].astype(np.uint32) << 16).view(np.float32).astype(np.float64) / fac[kv]
        d = np.sqrt(((x - c[:, None, :]) ** 2).reshape(ng, r, S, 128 // S).sum(-1)).max(1)
        cn = np.sqrt((c ** 2).reshape(ng, S, 128 // S).sum(-1))
        rho = radii[0, kv].astype(np.float64)
        assert (d <= rho).all()
        assert (rho <= (d * (1 + 2.0 ** -11) + cn * 2.0 ** -11) * (1 + 2.0 ** -7)).all()


@pytest.mark.parametrize("dtype,R,n,tree", [("bf16", 256, 3000, False), ("bf16", 17, 3000, False), ("bf16", 256, 100, False),
                                            ("f32", 255, 700, False), ("f32", 1, 64, False), ("bf16", 100, 1024, True)])
def test_threshold_ranks(G, dtype, R, n, tree):
    """Order statistics of the reservoir's scores against fp64: reservoirs of every fill, slots that are not a multiple of a
    lane quarter, equal scores (half the keys are repeated), and rows moved by the tree."""
    L = G.L
    g = np.random.default_rng(R + n)
    hkv, hq = 2, 8
    K = g.standard_normal((1, hkv, n, 128)).astype(np.float32)
    K[:, :, n // 2:] = K[:, :, :n - n // 2]
    K = W.round_to_bf16(K) if dtype == "bf16" else K
    q = g.standard_normal((1, hq, 128)).astype(np.float32)
    kw = dict(grouping=L.LVR_GROUP_TREE) if tree else {}
    with G.Index(K, K, dtype, hq, capacity=n, reservoir_size=R, seed=5, **kw) as ix:
        res = ix.reservoir()
        for mode, param in (("sample-max", 0.0), ("sample-topk", 1.0), ("sample-topk", 7.0), ("budget", 0.02), ("budget", 1.0)):
            tau = ix.threshold(q, mode, param)
            for h in range(hq):
                pos = res[0, h // 4]
                pos = pos[pos >= 0]
                m = pos.size
                s = np.sort(K[0, h // 4, pos].astype(np.float64) @ q[0, h].astype(np.float64))[::-1]
                k = 1 if mode == "sample-max" else (int(param) if mode == "sample-topk" else math.ceil(float(np.float32(param)) * m))
                want = s[min(max(k, 1), m) - 1]
                # an fp32 dot product of 128 terms: 128 * 2^-24 of the sum of magnitudes, which is below 200 here
                assert abs(tau[0, h] - want) <= 200 * 128 * 2.0 ** -24, (mode, param, h)


def check_median_splits(x, got, r):
    """`got` [entries]: the positions a tree of groups of r put in its slots; x [entries][128] fp64, multiples of 0.5 or arbitrary.
    Walks the tree down the given order: a node's entries have to be split at the median of (coordinate, position) on an axis of
    the largest variance, and the last split's order is the slots' order.  Which axis is taken is free among those whose
    variances are within rounding of the largest (exact integers where the values are multiples of 0.5)."""
    halves = np.rint(2.0 * x)
    exact = np.array_equal(halves, 2.0 * x)
    size = r
    while size < len(got):
        size *= 2

    def axes(ent):
        if exact:   # n * sum(v^2) - sum(v)^2: below 2^63 for 32768 entries of magnitude below 90
            v = halves[ent].astype(np.int64)
            var = len(ent) * (v * v).sum(axis=0) - v.sum(axis=0) ** 2
            return np.nonzero(var >= var.max() - var.max() * 1e-13)[0]   # fp64 sums of such values are exact, the quotient is rounded
        with np.errstate(invalid="ignore"):
            v = x[ent] - x[ent].mean(axis=0)
            var = (v * v).mean(axis=0)
        var = np.where(np.isfinite(var), var, 0.0)   # a node is not split on a coordinate that is no number in one of its keys
        return np.nonzero(var >= var.max() * (1 - 1e-10))[0]

    def walk(ent, at, m):   # ent: real entries of a node of m padded ones, ascending; its slots start at `at`
        if len(ent) == 0:
            return
        mine = got[at:at + len(ent)]
        if m == r:
            assert np.array_equal(mine, ent), f"slots {at}..: a group that was never split is out of order"
            return
        orders = [ent[np.lexsort((ent, x[ent, c]))] for c in axes(ent)]
        if m == 2 * r:
            assert any(np.array_equal(mine, o) for o in orders), f"slots {at}..: not the order of the last split"
            return
        left = np.sort(mine[:m // 2])
        fits = [o for o in orders if np.array_equal(left, np.sort(o[:m // 2]))]
        assert fits, f"slots {at}..: {len(ent)} entries are not split at their median"
        walk(left, at, m // 2)
        walk(np.sort(mine[m // 2:]), at + m // 2, m // 2)

    assert np.array_equal(np.sort(got), np.arange(len(got)))
    walk(np.arange(len(got)), 0, size)


@pytest.mark.parametrize("dtype,r,n,ties", [("bf16", 4, 1024, False), ("bf16", 4, 2048, True), ("bf16", 2, 3000, False), ("bf16", 1, 4096, True),
                                            ("f32", 4, 5000, False), ("f32", 16, 16384, True), ("bf16", 8, 32768, True),
                                            ("bf16", 4, 40000, False)])
def test_tree_order_is_the_recursive_median_split(G, dtype, r, n, ties):
    """The stored order against a recursive median split in fp64 on the CPU: inputs one workgroup orders, nodes whose codes are
    fetched by the split and by a launch of their own, padded sizes, and coordinates with few distinct values (where
    only the positions decide between equal entries)."""
    L = G.L
    g = np.random.default_rng(n + r)
    K = (g.standard_normal((1, 2, n, 128)) * np.exp(0.3 * g.standard_normal((1, 2, 1, 128)))).astype(np.float32)
    if ties:
        K = np.rint(2.0 * K) / 2.0
    K = W.round_to_bf16(K) if dtype == "bf16" else K.astype(np.float32)
    cfg = L.make_config(batch=1, n_q_heads=2, n_kv_heads=2, kv_dtype=L.LVR_BF16 if dtype == "bf16" else L.LVR_F32, capacity=n,
                        group_size=r, grouping=L.LVR_GROUP_TREE)
    h = L.lvr_create(cfg)
    try:
        Kd = G.to_device(K, dtype)
        L.lvr_build(h, Kd, Kd)
        slot_pos = L.lvr_export_index(h, cfg)[2]
    finally:
        L.lvr_destroy(h)
    grouped = n // r * r
    for kv in range(2):
        assert np.array_equal(slot_pos[0, kv, grouped:], np.arange(grouped, n))
        check_median_splits(K[0, kv, :grouped].astype(np.float64), slot_pos[0, kv, :grouped], r)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("r,n,kind", [(1, 2, "normal"), (1, 33, "normal"), (2, 7, "few"), (4, 17, "normal"), (16, 32, "few"), (8, 64, "normal"),
                                      (4, 65, "few"), (2, 130, "equal"), (4, 257, "normal"), (16, 512, "outlier"), (4, 513, "normal"),
                                      (4, 900, "few"), (8, 1025, "outlier"), (2, 2049, "few"), (4, 4097, "normal"), (4, 8193, "mean"),
                                      (8, 16500, "few"), (4, 33000, "few")])
def test_tree_order_at_the_edges_of_its_launches(G, dtype, r, n, kind):
    """Sizes around every size of a node that changes hands (one wave, one workgroup, codes fetched by the split, by a launch of
    their own, more than one workgroup's registers hold), as a build from token-major keys and as a buffer chunk of the same keys:
    the order is the recursive median split, the arena holds the keys in that order, and the right half's sums, which are
    differences, stand up to a few large keys and to a common offset."""
    L = G.L
    g = np.random.default_rng(n * 17 + r)
    K = g.standard_normal((1, 2, n, 128))
    if kind == "few":
        K = np.rint(K)
    elif kind == "equal":
        K[:] = K[:, :, :1]
    elif kind == "outlier":
        K[:, :, :: max(n // 3, 1), :5] *= 1000.0
    elif kind == "mean":
        K += 300.0
    K = W.round_to_bf16(K.astype(np.float32)) if dtype == "bf16" else K.astype(np.float32)
    chunk = n // (16 * r) * 16 * r if n <= 4097 else 0   # a buffer the keys fill at once
    cfg = L.make_config(batch=1, n_q_heads=2, n_kv_heads=2, kv_dtype=L.LVR_BF16 if dtype == "bf16" else L.LVR_F32, capacity=n + chunk,
                        group_size=r, grouping=L.LVR_GROUP_TREE, buffer_size=chunk if chunk else 16 * r)
    grouped = n // r * r
    h = L.lvr_create(cfg)
    try:
        Kd = G.to_device(K, dtype)
        Kt = Kd.transpose(1, 2).contiguous().transpose(1, 2)
        L.lvr_build(h, Kt, Kt)
        _, _, slot_pos, keys = L.lvr_export_index(h, cfg)
        if chunk:   # nothing indexed, then one chunk
            L.lvr_build(h, Kd[:, :, :0], Kd[:, :, :0])
            L.lvr_append(h, Kd[:, :, :chunk].contiguous(), Kd[:, :, :chunk].contiguous())
            assert L.lvr_length(h) == (chunk, chunk)
            chunk_pos = L.lvr_export_index(h, cfg)[2]
    finally:
        L.lvr_destroy(h)
    bits = (K.view(np.uint32) >> 16).astype(np.uint16) if dtype == "bf16" else K
    for kv in range(2):
        assert np.array_equal(slot_pos[0, kv, grouped:], np.arange(grouped, n))
        assert np.array_equal(keys[0, kv], bits[0, kv][slot_pos[0, kv]])
        check_median_splits(K[0, kv, :grouped].astype(np.float64), slot_pos[0, kv, :grouped], r)
        if chunk:
            check_median_splits(K[0, kv, :chunk].astype(np.float64), chunk_pos[0, kv], r)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("far", [-1e6, -1e8, 1e8, -1e30, -np.inf, np.inf, np.nan])
@pytest.mark.parametrize("r,n,at", [(2, 12, 3), (4, 60, 0), (2, 250, 100), (4, 512, 0), (4, 1000, 700), (4, 2048, 0), (4, 6000, 5000), (8, 20000, 0),
                                    (8, 36000, 7)])
def test_a_key_far_off_does_not_blur_the_splits_of_the_others(G, dtype, far, r, n, at):
    """One key, the first of the cache or another, is far off in the widest channel (or no number there), its neighbour in the next one, the other
    way: a node's rows' squares reach neither the sums of the nodes beside it, which are differences, nor (fp32) the value that
    all coordinates are taken relative to, so that every node of the others is still split on its own widest axis.  As a build and as a
    buffer chunk."""
    L = G.L
    g = np.random.default_rng(n + at)
    K = g.standard_normal((1, 2, n, 128))
    K[..., :2] *= 3.0
    other = -far if far == far else far
    K[:, 0, at, 0] = far
    K[:, 1, at, 1] = other
    K[:, :, (at + 1) % n, 1] = other
    K = W.round_to_bf16(K.astype(np.float32)) if dtype == "bf16" else K.astype(np.float32)
    chunk = n // (16 * r) * 16 * r if n <= 2048 else 0
    cfg = L.make_config(batch=1, n_q_heads=2, n_kv_heads=2, kv_dtype=L.LVR_BF16 if dtype == "bf16" else L.LVR_F32, capacity=n + chunk,
                        group_size=r, grouping=L.LVR_GROUP_TREE, buffer_size=chunk if chunk else 16 * r)
    h = L.lvr_create(cfg)
    try:
        Kd = G.to_device(K, dtype)
        L.lvr_build(h, Kd, Kd)
        orders = [L.lvr_export_index(h, cfg)[2][..., :n // r * r]]
        if chunk:
            L.lvr_build(h, Kd[:, :, :0], Kd[:, :, :0])
            L.lvr_append(h, Kd[:, :, :chunk].contiguous(), Kd[:, :, :chunk].contiguous())
            orders.append(L.lvr_export_index(h, cfg)[2][..., :chunk])
    finally:
        L.lvr_destroy(h)
    for order in orders:
        for kv in range(2):
            check_median_splits(K[0, kv, :order.shape[-1]].astype(np.float64), order[0, kv], r)


@pytest.mark.parametrize("hq,hkv,n,r,S,tail,kw", [
    (1, 1, 64, 4, 4, 0, {}), (1, 1, 4096, 4, 4, 0, {}), (2, 1, 1000, 2, 1, 3, {}), (8, 2, 4095, 4, 16, 131, {}),
    (8, 1, 8192, 1, 2, 255, dict(query_workgroups=16)), (4, 4, 5000, 16, 8, 17, dict(buffer_size=32)),
    (8, 2, 2048, 4, 4, 40, dict(tree=True)), (4, 1, 3, 4, 4, 5, {}), (4, 2, 700, 4, 4, 100, dict(dense_buffer=True)),
    (4, 2, 700, 4, 4, 300, dict(concurrent=True)), (320, 40, 700, 2, 4, 5, {}), (800, 800, 40, 1, 1, 3, {}),
    (8, 2, 2050, 4, 4, 40, dict(offload=True)), (4, 4, 3000, 2, 1, 0, dict(offload=True, tree=True)), (120, 120, 50, 1, 4, 7, dict(offload=True))])
def test_fp32_one_launch_query_is_the_two_launch_one(G, oracle, hq, hkv, n, r, S, tail, kw):
    """The fused fp32 query against the separate bound test and filter (LVR_SEPARATE_KERNELS): the same sets and counts for
    every head count, block count, group size, segment remainder, buffer content and option, with thresholds that keep
    few keys, everything and nothing, room for fewer entries than there are, and an append that rides in the launch; as many
    (sequence, KV head) pairs as give each a few segments, and more than fit the device at once; rows in host memory; the
    attention over the lists against the oracle."""
    L = G.L
    g = np.random.default_rng(n + hq)
    K = g.standard_normal((1, hkv, n + tail + 2, 128)).astype(np.float32)
    V = g.standard_normal((1, hkv, n + tail + 2, 128)).astype(np.float32)
    q = g.standard_normal((1, hq, 128)).astype(np.float32)
    flags = (L.LVR_ATTEND_BUFFER_DENSE if kw.get("dense_buffer") else 0) | (L.LVR_CONCURRENT_UPDATE if kw.get("concurrent") else 0)
    flags |= L.LVR_KV_IN_HOST_MEMORY if kw.get("offload") else 0
    opt = {k: v for k, v in kw.items() if k in ("query_workgroups", "buffer_size")}
    if kw.get("tree"):
        opt["grouping"] = L.LVR_GROUP_TREE
    total = n + tail
    scores = np.stack([np.sort(K[0, h * hkv // hq, :total] @ q[0, h])[::-1] for h in range(hq)])
    few = max(1, total // 50)
    taus = [0.5 * (scores[:, few - 1] + scores[:, few])[None] if total > few else scores[:, :1].T - 1.0,
            np.full((1, hq), -np.inf), np.full((1, hq), 1e9)]
    got = {}
    for name, extra in (("fused", 0), ("separate", L.LVR_SEPARATE_KERNELS)):
        with G.Index(K[:, :, :n], V[:, :, :n], "f32", hq, capacity=n + tail + 2, group_size=r, n_subspaces=S, flags=flags | extra, **opt) as ix:
            if tail:
                ix.append(K[:, :, n:total], V[:, :, n:total])
            res = []
            for tau in taus:
                tau = tau.astype(np.float32)
                for cap in (total, max(1, few // 2)):
                    idx, cnt, out = ix.query(q, tau, cap=cap, fused=True)
                    ix.stats(raise_on_overflow=False)
                    if cap == total and not kw.get("dense_buffer"):
                        G.check_step(oracle, ix, q, tau, idx, cnt, out, tag=f"f32 {name}")
                    res.append((cnt, [np.sort(idx[0, h, :min(cnt[0, h], cap)]) if cap == total else None for h in range(hq)],
                                out if cap == total else None))
            # two more tokens, the first appended by the step itself
            kn, vn = G.to_device(K[:, :, total:total + 1], "f32"), G.to_device(V[:, :, total:total + 1], "f32")
            qd, td = torch.from_numpy(q).cuda(), torch.from_numpy(taus[0].astype(np.float32)).cuda()
            idx = torch.zeros((1, hq, total + 2), dtype=torch.int32, device="cuda")
            cnt = torch.zeros((1, hq), dtype=torch.int32, device="cuda")
            out = torch.zeros((1, hq, 128), device="cuda")
            L.lvr_append_decode_step(ix.h, kn, vn, qd, td, out, idx, cnt)
            torch.cuda.synchronize()
            res.append((cnt.cpu().numpy(), [np.sort(idx[0, h, :int(cnt[0, h])].cpu().numpy()) for h in range(hq)], out.cpu().numpy()))
            got[name] = res
    for (c1, s1, o1), (c2, s2, o2) in zip(got["fused"], got["separate"]):
        assert np.array_equal(c1, c2)
        for a, b in zip(s1, s2):
            assert a is None or np.array_equal(a, b)
        if o1 is not None:
            # weights of logits of magnitude below 60, each good to 128 * 2^-24 of the sum of its terms' magnitudes
            assert np.abs(o1 - o2).max() <= 1e-4


@pytest.mark.parametrize("index_dtype", ["auto", "same"])
@pytest.mark.parametrize("hq,hkv,n,r,tail", [
    (32, 32, 2000, 1, 3), (8, 8, 9001, 1, 0), (64, 8, 20000, 1, 5), (8, 8, 34001, 1, 7), (8, 8, 50007, 1, 1),
    (16, 16, 34003, 4, 0), (16, 16, 50001, 4, 2), (8, 2, 40001, 1, 0), (24, 12, 12288, 2, 9),
    (64, 8, 16390, 2, 7), (64, 8, 33001, 4, 3)])
def test_segments_chosen_by_the_launch(G, oracle, hq, hkv, n, r, tail, index_dtype):
    """The tiles per wave that a launch picks by itself, powers of two, other even counts and (eight heads, groups of several
    keys) odd ones, with and without the buffer's workgroups, four and eight heads per pass: the oracle's sets and outputs."""
    L = G.L
    g = np.random.default_rng(n + hkv)
    # bf16 values, as the cache holds them (a value off the grid is half an ulp, 2^-9 = 2.0e-3, from what is attended)
    K, V = (torch.from_numpy(g.standard_normal((1, hkv, n + tail, 128)).astype(np.float32)).bfloat16().float().numpy()
            for _ in range(2))
    q = g.standard_normal((1, hq, 128)).astype(np.float32)
    dt = {"auto": L.LVR_INDEX_AUTO, "same": L.LVR_INDEX_SAME}[index_dtype]
    with G.Index(K[:, :, :n], V[:, :, :n], "bf16", hq, capacity=n + tail, group_size=r, buffer_size=64, index_dtype=dt) as ix:
        if tail:
            ix.append(K[:, :, n:], V[:, :, n:])
        for frac in (0.004, 0.05):
            tau = G.oracle_taus(oracle, ix, q, frac=frac)
            idx, cnt, out = ix.query(q, tau, fused=True)
            G.check_step(oracle, ix, q, tau, idx, cnt, out, tag=f"segments n={n} r={r} hkv={hkv} {index_dtype}")


@pytest.mark.parametrize("dtype,batch,hq,hkv,n,splits", [
    ("f32", 1, 4, 2, 3000, -1), ("f32", 1, 4, 2, 3000, 64), ("f32", 9, 32, 8, 300, 0), ("bf16", 1, 4, 2, 3000, -1),
    ("bf16", 1, 4, 2, 3000, 64), ("bf16", 9, 32, 8, 300, 0), ("bf16", 1, 2, 1, 65600, 0)])
def test_carried_scores_are_not_rounded_at_the_size_of_the_logit(G, dtype, batch, hq, hkv, n, splits):
    """Every attention form over carried scores, on integers: each score is 2^20 plus a small exact integer, so the difference
    of two scores is exact and a softmax weight is off by the roundings of that difference times the scale alone.  (Scaled
    first, a logit of 2^17 base-2 units is rounded by up to 2^-7, a weight by half a percent.)"""
    g = np.random.default_rng(n + hq)
    K = g.integers(-4, 5, size=(batch, hkv, n, 128)).astype(np.float32)
    V = W.round_to_bf16(g.uniform(-1.0, 1.0, size=(batch, hkv, n, 128)).astype(np.float32))
    q = g.integers(-4, 5, size=(batch, hq, 128)).astype(np.float32)
    K[..., 0] = q[..., 0] = 1024.0
    with G.Index(K, V, dtype, hq, capacity=n, group_size=4, attn_splits=splits) as ix:
        _, cnt, out = ix.query(q, np.full((batch, hq), -np.inf, dtype=np.float32), fused=True)
    assert (cnt == n).all()
    for b in range(batch):
        for h in range(hq):
            kv = h * hkv // hq
            s = K[b, kv].astype(np.float64) @ q[b, h].astype(np.float64)
            p = np.exp((s - s.max()) / math.sqrt(128))
            want = (p / p.sum()) @ V[b, kv].astype(np.float64)
            # weights above 2^-30 of the largest: 30 ln 2 * 3 * 2^-24 (scale, difference, product) plus two ulps of the
            # exponential; values below 1; the fp32 sums add at most 2^-24 for each of the lists' rounds
            assert np.abs(out[b, h] - want).max() <= 2e-5, (b, h, np.abs(out[b, h] - want).max())


@pytest.mark.parametrize("dtype,n,one_launch", [("f32", 65536, True), ("f32", 65537, False), ("bf16", 65537, True), ("bf16", 262145, False)])
def test_attention_form_of_a_decode_step(G, oracle, dtype, n, one_launch):
    """The context length up to which a head's list is attended in one launch, on both sides of it, against the oracle: 65536
    keys of fp32, 262144 of bf16 (whose rows are half as wide and, beyond 65536, gathered by two workgroups per head)."""
    L = G.L
    g = np.random.default_rng(n)
    K = W.round_to_bf16(g.standard_normal((1, 1, n, 128)).astype(np.float32))
    q = g.standard_normal((1, 2, 128)).astype(np.float32)
    with G.Index(K, K, dtype, 2, capacity=n, group_size=1) as ix:
        L.lvr_profile_enable(ix.h, 64)
        tau = G.oracle_taus(oracle, ix, q, frac=0.02)
        idx, cnt, out = ix.query(q, tau, fused=True)
        launches = L.lvr_profile_read(ix.h)
        G.check_step(oracle, ix, q, tau, idx, cnt, out, tag=f"{dtype} n={n}")
    assert launches["attn_partial"][1] == 1 and launches["attn_combine"][1] == (0 if one_launch else 1)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("batch,hq,hkv,splits", [(1, 4, 1, 64), (1, 16, 2, 256), (1, 32, 8, 64), (1, 64, 8, 9), (3, 32, 8, 64), (1, 8, 4, 1)])
def test_attention_of_lists_by_several_workgroups(G, dtype, batch, hq, hkv, splits):
    """List lengths around the entries of a wave, of a workgroup and of all of a head's workgroups, whose last to end merges the
    others: a length per head, three calls in a row (tickets back at zero, the last one from a graph replayed twice), and the query
    that hands its counts over followed by the attention over its lists.  Entries lost or taken twice are counted: with q = 0 and rows of V
    that are a one in the coordinate position % 128, the output times the list's length is how often each remainder is listed."""
    L = G.L
    g = np.random.default_rng(hq + splits)
    n = 4200
    lens = [0, 1, 15, 16, 17, 63, 64, 65, 128, 129, 255, 256, 257, 511, 513, 1024, 1025, 2049, 4096, 4200]
    K = W.round_to_bf16(g.standard_normal((batch, hkv, n, 128)).astype(np.float32))
    V = W.round_to_bf16(g.standard_normal((batch, hkv, n, 128)).astype(np.float32))
    q = g.standard_normal((batch, hq, 128)).astype(np.float32)
    ones = np.tile(np.eye(128, dtype=np.float32)[np.arange(n) % 128], (batch, hkv, 1, 1))
    with G.Index(K, V, dtype, hq, capacity=n, group_size=4, attn_splits=splits) as ix, \
            G.Index(K, ones, dtype, hq, capacity=n, group_size=4, attn_splits=splits) as counting:
        qd = torch.from_numpy(q).cuda()
        stream = torch.cuda.Stream()
        for call in range(3):
            cap = n if call != 1 else 2048   # room for more entries, and for as many as take fewer workgroups
            cnt = np.array([[lens[(7 * h + 3 * b + call) % len(lens)] for h in range(hq)] for b in range(batch)], dtype=np.int32)
            idx = np.stack([[g.permutation(n)[:cap] for _ in range(hq)] for _ in range(batch)]).astype(np.int32)
            idx_d, cnt_d, out = torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda(), torch.full((batch, hq, 128), np.nan, device="cuda")
            torch.cuda.synchronize()
            if call < 2:
                L.lvr_sparse_attention(ix.h, qd, idx_d, cnt_d, out)
            else:
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=stream):
                    L.lvr_sparse_attention(ix.h, qd, idx_d, cnt_d, out, stream)
                for _ in range(2):
                    out.fill_(float("nan"))
                    graph.replay()
            times = torch.full_like(out, np.nan)
            L.lvr_sparse_attention(counting.h, torch.zeros_like(qd), idx_d, cnt_d, times)
            torch.cuda.synchronize()
            got, times = out.cpu().numpy(), times.cpu().numpy()
            for b in range(batch):
                for h in range(hq):
                    l = idx[b, h, :cnt[b, h]]
                    # weights are ones, their sums whole numbers; one quotient is rounded, by 2^-24 of at most 33
                    assert np.abs(times[b, h] * len(l) - np.bincount(l % 128, minlength=128)).max() <= 1e-4, (call, b, h, len(l))
                    s = K[b, h * hkv // hq][l].astype(np.float64) @ q[b, h].astype(np.float64) / math.sqrt(128)
                    p = np.exp(s - s.max()) if len(l) else s
                    want = (p / max(p.sum(), 1e-300)) @ V[b, h * hkv // hq][l].astype(np.float64)
                    # logits below 6: d + 1 products and 7 levels of fp32 sums (2^-24 * 6 * 136), the exponential's and the sums' few ulps
                    # of weights that add up to one, values below 5
                    assert np.abs(got[b, h] - want).max() <= 3e-4, (call, b, h, len(l), np.abs(got[b, h] - want).max())
        tau = np.sort(np.einsum("bhd,bhnd->bhn", q, np.repeat(K, hq // hkv, axis=1)), axis=-1)
        tau = np.stack([[0.5 * (tau[b, h, -m] + tau[b, h, -m - 1]) for h, m in enumerate(np.resize([3, 60, 70, 300], hq))] for b in range(batch)])
        for _ in range(2):
            idx, cnt, out = ix.query(q, tau.astype(np.float32))
            s = np.einsum("bhd,bhnd->bhn", q.astype(np.float64), np.repeat(K, hq // hkv, axis=1).astype(np.float64))
            slack = 1e-4 * np.abs(tau)
            assert ((s >= tau[..., None]).sum(-1) <= cnt).all() and (cnt <= (s >= (tau - slack)[..., None]).sum(-1)).all()
            assert ix.stats()["keys_emitted"] == int(cnt.sum()) and np.isfinite(out).all()


@pytest.mark.parametrize("hq,hkv,splits,factor", [(1, 1, 256, 7.0), (1, 1, 64, 7.0), (32, 8, 64, 28.0)])
def test_long_lists_are_shared_by_more_workgroups(G, hq, hkv, splits, factor):
    """fp32 lists of 30000 entries against lists of 300 in room for as many, by the clock: one head 25 against 6 us (69 by 16
    workgroups), 32 heads 150 against 7 (223 by 8 workgroups each)."""
    L = G.L
    n = 65536
    K = torch.randn((1, hkv, n, 128), device="cuda")
    q, out = torch.randn((1, hq, 128), device="cuda"), torch.empty((1, hq, 128), device="cuda")
    idx = torch.rand((hq, n), device="cuda").topk(30000, dim=1).indices.sort(dim=1).values.to(torch.int32).reshape(1, hq, -1).contiguous()
    cfg = L.make_config(batch=1, n_q_heads=hq, n_kv_heads=hkv, kv_dtype=L.LVR_F32, capacity=n, group_size=4, attn_splits=splits)
    h = L.lvr_create(cfg)
    try:
        L.lvr_build(h, K, K)
        took = []
        for entries in (300, 30000):
            count = torch.full((1, hq), entries, dtype=torch.int32, device="cuda")
            stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
            L.lvr_sparse_attention(h, q, idx, count, out)
            torch.cuda.synchronize()
            with torch.cuda.graph(graph, stream=stream):
                for _ in range(20):
                    L.lvr_sparse_attention(h, q, idx, count, out, stream)
            took.append(math.inf)
            for _ in range(10):
                start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                start.record()
                graph.replay()
                end.record()
                torch.cuda.synchronize()
                took[-1] = min(took[-1], start.elapsed_time(end))
    finally:
        L.lvr_destroy(h)
    assert took[1] < factor * took[0], took


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("batch,hq,hkv,n,r", [(9, 32, 8, 1000, 4), (33, 8, 8, 96, 1)])
def test_more_heads_than_compute_units(G, oracle, dtype, batch, hq, hkv, n, r):
    """Decode steps of more than 256 query heads, whose lists are attended by eight waves each: lists of one entry, of less and
    more than a round of 512 entries, and none, against the oracle."""
    g = np.random.default_rng(n)
    K, V = (W.round_to_bf16(g.standard_normal((batch, hkv, n, 128)).astype(np.float32)) for _ in range(2))
    q = g.standard_normal((batch, hq, 128)).astype(np.float32)
    with G.Index(K, V, dtype, hq, capacity=n, group_size=r) as ix:
        taus = [G.oracle_taus(oracle, ix, q, k_count=1), G.oracle_taus(oracle, ix, q, frac=0.1), np.full((batch, hq), -np.inf, np.float32)]
        taus.append(taus[1].copy())
        taus[3][:, ::2] = 1e9
        for tau in taus:
            idx, cnt, out = ix.query(q, tau, fused=True)
            G.check_step(oracle, ix, q, tau, idx, cnt, out, tag=f"{dtype} {batch} x {hq} heads")
        assert (cnt[:, ::2] == 0).all() and (out[:, ::2] == 0).all()


@pytest.mark.parametrize("dtype,n", [("bf16", 98303), ("bf16", 98307), ("f32", 49151), ("f32", 49155), ("f32", 5)])
def test_rows_of_a_build_and_an_append_arrive(G, dtype, n):
    """Value rows copied by a build on both sides of the size (48 MiB) from which they are streamed, out of a token-major view,
    with rows behind the last whole group, and by an append: the attention over a list of one position is that row."""
    L = G.L
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    more, hkv, hq = 300, 2, 8
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    K, V = (torch.randn((1, n + more, hkv, 128), generator=g, device="cuda").to(dt).transpose(1, 2) for _ in range(2))
    cfg = L.make_config(batch=1, n_q_heads=hq, n_kv_heads=hkv, kv_dtype=L.LVR_BF16 if dtype == "bf16" else L.LVR_F32, capacity=n + more,
                        group_size=4, index_dtype=L.LVR_INDEX_SAME)
    h = L.lvr_create(cfg)
    try:
        L.lvr_build(h, K[:, :, :n], V[:, :, :n])
        L.lvr_append(h, K[:, :, n:].contiguous(), V[:, :, n:].contiguous())
        keys = L.lvr_export_index(h, cfg)[3]
        q = torch.randn((1, hq, 128), generator=g, device="cuda")
        count = torch.ones((1, hq), dtype=torch.int32, device="cuda")
        out = torch.empty((1, hq, 128), device="cuda")
        edges = torch.tensor([0, n - 1, n - 2, n, n + more - 1, n // 2, n + 1, n // 4 * 4 - 1], device="cuda")
        for picks in [edges] + [torch.randint(0, n + more, (hq,), generator=g, device="cuda") for _ in range(8)]:
            L.lvr_sparse_attention(h, q, picks.to(torch.int32).reshape(1, hq, 1).contiguous(), count, out)
            want = V[0, torch.arange(hq, device="cuda") * hkv // hq, picks].float()
            assert torch.equal(out[0], want), (out[0] != want).any(dim=1)
    finally:
        L.lvr_destroy(h)
    bits = keys.view(np.int16) if dtype == "bf16" else keys.view(np.int32)
    assert np.array_equal(bits, K.contiguous().view(torch.int16 if dtype == "bf16" else torch.int32).cpu().numpy().reshape(bits.shape))


@pytest.mark.parametrize("R,n", [(256, 5000), (255, 255), (65, 900), (64, 900), (2, 2), (1, 1)])
def test_threshold_gap_and_mean(G, R, n):
    """The rules that look at all scores, on integers (exact scores, many equal gaps of which the first counts), for
    reservoirs that end within, at and just behind a wave."""
    g = np.random.default_rng(R)
    K = np.zeros((1, 2, n, 128), dtype=np.float32)
    K[..., 0] = g.integers(-100, 100, size=(1, 2, n)) * 3
    K[..., 1] = g.integers(0, 2, size=(1, 2, n))
    q = np.zeros((1, 4, 128), dtype=np.float32)
    q[0, :, 0] = [1, -2, 5, 0]
    q[0, :, 1] = [1, 1, 0, 0]
    with G.Index(K, K, "f32", 4, capacity=n, reservoir_size=R, seed=3) as ix:
        res = ix.reservoir()
        gap, mean = ix.threshold(q, "sample-gap"), ix.threshold(q, "sample-mean-max")
    for h in range(4):
        pos = res[0, h // 2]
        s = np.sort(K[0, h // 2, pos[pos >= 0]].astype(np.float64) @ q[0, h].astype(np.float64))[::-1]
        d = s[:-1] - s[1:]
        assert gap[0, h] == (s[int(np.argmax(d))] if d.size else s[0]), h
        assert mean[0, h] == np.float32(0.5 * (s[0] + s.sum() / s.size)), h


def test_marshalled_and_plain_arguments_are_the_same_call(G, oracle):
    """Every entry point of a decode loop with tensors, with arguments marshalled once, and with both; on a stream given as an object,
    as a handle and not at all; wrong types and strides are refused either way."""
    L = G.L
    g = np.random.default_rng(5)
    n = 700
    K = W.round_to_bf16(g.standard_normal((1, 2, n, 128)).astype(np.float32))
    q = g.standard_normal((1, 8, 128)).astype(np.float32)
    with G.Index(K, K, "bf16", 8, capacity=n + 8, group_size=1) as ix:
        tau = torch.from_numpy(G.oracle_taus(oracle, ix, q, frac=0.05).astype(np.float32)).cuda()
        qd = torch.from_numpy(q).cuda()
        out, idx, cnt = torch.empty(1, 8, 128, device="cuda"), torch.zeros(1, 8, n + 8, dtype=torch.int32, device="cuda"), torch.zeros(1, 8, dtype=torch.int32, device="cuda")
        k = G.to_device(K[:, :, :1].copy(), "bf16")
        other = torch.cuda.Stream()
        A = L.tensor_arg
        wraps = (lambda t: t, A, lambda t: A(t) if t.dtype == torch.int32 else t, lambda t: A(t) if t.dtype == torch.int32 else t)
        results = []
        for form, w in enumerate(wraps):
            st = (None, L.stream_arg(), other, torch.cuda.current_stream())[form]
            out.fill_(float("nan"))
            torch.cuda.synchronize()
            L.lvr_query(ix.h, w(qd), w(tau), w(idx), w(cnt), st)
            L.lvr_sparse_attention(ix.h, w(qd), w(idx), w(cnt), w(out), st)
            torch.cuda.synchronize()
            listed = out.clone()
            L.lvr_sparse_attention_static(ix.Kd, ix.Vd, w(qd), w(idx), w(cnt), w(out), 0.0, st)
            torch.cuda.synchronize()
            static = out.clone()
            L.lvr_decode_step(ix.h, w(qd), w(tau), w(out), w(idx), w(cnt), st)
            torch.cuda.synchronize()
            step = out.clone()
            L.lvr_dense_attention(ix.h, w(qd), w(out), st)
            torch.cuda.synchronize()
            results.append((listed, static, step, out.clone(), cnt.clone()))
        for r in results[1:]:
            for a, b in zip(results[0], r):
                assert torch.allclose(a.float(), b.float(), rtol=0, atol=1e-5)   # lists come in another order
        L.lvr_append_decode_step(ix.h, A(k), k, A(qd), tau, out, A(idx), cnt)
        torch.cuda.synchronize()
        assert L.lvr_length(ix.h)[0] == n + 1
        import paper_2605_06763_amd.binding as binding
        calls = binding._call   # the compiled calls take all of these themselves: None would send them to ctypes
        assert calls is not None
        for form, w in enumerate(wraps[:3]):
            arg = L.stream_arg()
            assert calls.query(ix.h, w(qd), w(tau), w(idx), w(cnt), arg) == L.LVR_OK
            assert calls.sparse_attention(ix.h, w(qd), w(idx), w(cnt), w(out), arg) == L.LVR_OK
            assert calls.sparse_attention_static(ix.Kd, ix.Vd, w(qd), w(idx), w(cnt), w(out), 0.0, arg) == L.LVR_OK
            assert calls.decode_step(ix.h, w(qd), w(tau), w(out), w(idx), w(cnt), arg) == L.LVR_OK
            assert calls.dense_attention(ix.h, w(qd), w(out), arg) == L.LVR_OK
            assert calls.append_decode_step(ix.h, w(k), k, w(qd), w(tau), w(out), w(idx), w(cnt), arg) == L.LVR_OK
            torch.cuda.synchronize()
            assert L.lvr_length(ix.h)[0] == n + form + 2
        for bad in (qd.double(), qd.transpose(1, 2), qd.cpu()):
            with pytest.raises(ValueError):
                L.lvr_decode_step(ix.h, bad, tau, out, idx, cnt)
        with pytest.raises(ValueError):
            L.lvr_query(ix.h, A(qd), A(tau), A(tau), cnt)
