"""Property tests of the projection calls on the GPU over random shapes
(hypothesis, derandomized so every run draws the same examples): the o_proj
with residual and RMSNorm, and the attention prelude with and without Q/K
norm, bias and partial or interleaved rotation, at batches up to 64 (any
multiple of 16 rows) and from 65 to 256 (multiples of 128).  The fixed-shape
tests hold every form of the planner; these mix sizes between them.  Each
output is held to one bf16 spacing of the fp64 oracle, as in those tests."""
import numpy as np
import pytest
from hypothesis import HealthCheck, given, settings
from hypothesis import strategies as st

import workloads as W
from test_gpu_oproj import check_ulps as check_oproj
from test_gpu_oproj import ref as ref_oproj
from test_gpu_oproj import run as run_oproj
from test_gpu_prelude import check_ulps as check_prelude
from test_gpu_prelude import host, ref_prelude, run_prelude
from _gpu import log

pytestmark = pytest.mark.gpu

SETTINGS = dict(deadline=None, derandomize=True, database=None,
                suppress_health_check=[HealthCheck.too_slow, HealthCheck.function_scoped_fixture])


@settings(max_examples=30, **SETTINGS)
@given(batch=st.integers(1, 64), k_tiles=st.integers(1, 128), h_tiles=st.integers(1, 256),
       seed=st.integers(0, 2 ** 16))
def test_oproj_random_shapes(gpu_lib, batch, k_tiles, h_tiles, seed):
    k, h = 32 * k_tiles, 16 * h_tiles
    log(f"o_proj property case B={batch} K={k} H={h} seed={seed}")
    w = W.build_oproj(batch, k, h, seed=seed)
    z, hn = run_oproj(gpu_lib, w)
    rz, rh = ref_oproj(w)
    check_oproj(z, rz, "z")
    check_oproj(hn, rh, "h")


@settings(max_examples=15, **SETTINGS)
@given(batch=st.integers(65, 256), k_tiles=st.integers(1, 96), groups=st.integers(1, 24), seed=st.integers(0, 2 ** 16))
def test_oproj_random_shapes_above_64(gpu_lib, batch, k_tiles, groups, seed):
    k, h = 32 * k_tiles, 128 * groups
    log(f"o_proj property case B={batch} K={k} H={h} seed={seed}")
    w = W.build_oproj(batch, k, h, seed=seed)
    z, hn = run_oproj(gpu_lib, w)
    rz, rh = ref_oproj(w)
    check_oproj(z, rz, "z")
    check_oproj(hn, rh, "h")


@st.composite
def prelude_shapes(draw, batches=(1, 64)):
    d = draw(st.sampled_from([64, 128, 256]))
    hkv = draw(st.sampled_from([1, 2, 4, 8]))
    hq = hkv * draw(st.sampled_from([1, 2, 4, 8]))
    batch = draw(st.integers(*batches))
    if batch > 64 and (hq + 2 * hkv) * d % 128:  # one kv head of 64 and an odd number of query heads
        hq += hkv
    hidden = 32 * draw(st.integers(2, 96))
    rot = draw(st.sampled_from(["full", "half", "none"]))
    opt = dict(qk_norm=draw(st.booleans()), bias=draw(st.booleans()), interleaved=draw(st.booleans()),
               rotary_dim={"full": None, "half": d // 2, "none": 0}[rot])
    return batch, hidden, hq, hkv, d, opt, draw(st.integers(0, 2 ** 16))


@settings(max_examples=30, **SETTINGS)
@given(prelude_shapes())
def test_prelude_random_shapes(gpu_lib, shape):
    batch, hidden, hq, hkv, d, opt, seed = shape
    log(f"prelude property case B={batch} H={hidden} {hq}:{hkv} D={d} {opt} seed={seed}")
    lens = np.random.default_rng(seed).integers(0, 100000, size=batch)
    w = W.build_prelude(batch, hidden, hq, hkv, d, seed=seed, lengths=lens, theta=1.0e6, **opt)
    got = run_prelude(gpu_lib, w)
    for name, g, r in zip("qkv", got, ref_prelude(w)):
        check_prelude(host(g), r, name)


@settings(max_examples=15, **SETTINGS)
@given(prelude_shapes(batches=(65, 256)))
def test_prelude_random_shapes_above_64(gpu_lib, shape):
    batch, hidden, hq, hkv, d, opt, seed = shape
    log(f"prelude property case B={batch} H={hidden} {hq}:{hkv} D={d} {opt} seed={seed}")
    lens = np.random.default_rng(seed).integers(0, 100000, size=batch)
    w = W.build_prelude(batch, hidden, hq, hkv, d, seed=seed, lengths=lens, theta=1.0e6, **opt)
    got = run_prelude(gpu_lib, w)
    for name, g, r in zip("qkv", got, ref_prelude(w)):
        check_prelude(host(g), r, name)
