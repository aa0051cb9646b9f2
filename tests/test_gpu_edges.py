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
