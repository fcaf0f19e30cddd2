"""Every launch shape the tuner may pick (include/razer_tune.h), forced one at a time through
razer_tune_force, against the CPU oracle: the choice of a shape must never change a result beyond fp32
summation order.  Ragged N, ragged K, single and grouped launches, 16- and 64-element blocks."""
import numpy as np
import pytest
import torch

import paper_2501_04052_amd as razer
from paper_2501_04052_amd import binding, synth
from gpu_util import TOL, bf16_bits_to_dev, dev_to_bf16_bits, launched_kernels, max_rel_err

pytestmark = pytest.mark.gpu
W = 0
SV = (5.0, 8.0)


def _rand_weights(n, k, seed, block=16):
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8)
    scales = rng.integers(0, 256, size=(n, k // block), dtype=np.uint8)
    wq = (codes, scales, np.float32(2.0 ** -9))
    return wq, razer.RazerTensor.from_host(*wq, W, SV)


def _check(oracle, family, shape, m, ns, k, block=16, seed=0):
    print("tuning family", family, "shape", shape, "m", m, "ns", ns, "k", k, "block", block, flush=True)
    a = synth.activation(m, k, seed=9700 + m + k)
    a_dev = bf16_bits_to_dev(a)
    ws = [_rand_weights(n, k, 9800 + seed + i + n, block) for i, n in enumerate(ns)]
    razer.razer_tune_force(family, shape)
    try:
        src, got_shape = razer.razer_tune_lookup(family, m, sum(ns), k)
        assert src == 1 and got_shape[:len(shape)] == tuple(shape)
        if len(ns) == 1:
            ys = [razer.razer_linear(ws[0][1], a_dev)]
        else:
            ys = razer.razer_linear_grouped([w[1] for w in ws], a_dev)
        torch.cuda.synchronize()
    finally:
        razer.razer_tune_force(family, None)
    for (wq, _), y in zip(ws, ys):
        y64, _ = oracle.linear(wq, a_bf16=a)
        err = max_rel_err(dev_to_bf16_bits(y), y64)
        assert err <= TOL, (family, shape, err)


# groups of 16 rows per workgroup and waves (6 groups: up to 32 rows, else the heuristic; 16 waves: one group, up to 8 rows, 9..16
# rows of 4096 elements and more, above 32 rows of 10240 and more)
SMALL_BATCH_SHAPES = [(2, 1, 8), (2, 1, 16), (2, 2, 8), (2, 3, 8), (2, 4, 8), (2, 6, 8), (2, 2)]


@pytest.mark.parametrize("shape", SMALL_BATCH_SHAPES)
@pytest.mark.parametrize("m,ns,k,block", [(5, (1000,), 4160, 16), (16, (328, 200), 4160, 16), (9, (72,), 512, 64),
                                          (16, (100, 36, 4), 34944, 16), (12, (40, 24), 2048 + 128, 128),
                                          (33, (200, 72), 2048 + 64, 64), (64, (300,), 1152, 128), (40, (68, 36), 96, 32)])
def test_small_batch_shapes(oracle, shape, m, ns, k, block):
    _check(oracle, binding.TUNE_SMALL_BATCH, shape, m, ns, k, block)


@pytest.mark.parametrize("shape", [(1, 1, 2), (1, 2, 8), (0, 4, 4), (0, 8, 1)])
def test_small_batch_shapes_on_record_only_size_the_workspace(oracle, shape):
    """Shapes of the kernels that the small-batch kernel replaced: they are accepted, and the call runs as ever."""
    _check(oracle, binding.TUNE_SMALL_BATCH, shape, 20, (200,), 1024)
    _check(oracle, binding.TUNE_SMALL_BATCH, shape, 16, (64, 64), 4096)


@pytest.mark.parametrize("shape", [(2, 1), (2, 2), (4, 1), (8, 1)])
@pytest.mark.parametrize("m,ns,k,block", [(1, (333,), 4096 + 32, 16), (1, (100, 57, 8), 11008, 16), (1, (41,), 28672, 16),
                                          (1, (50,), 4096, 64), (3, (20,), 32768 + 2048, 16)])
def test_gemv_shapes(oracle, shape, m, ns, k, block):
    _check(oracle, binding.TUNE_GEMV, shape, m, ns, k, block)


@pytest.mark.parametrize("shape", [(4,), (8,)])
@pytest.mark.parametrize("m,ns,k,block", [(2, (97, 40), 4096, 16), (3, (333,), 4096 + 32, 16), (4, (100, 57), 11008, 16),
                                          (4, (70,), 16384, 16), (3, (120, 36), 4096 + 128, 64), (4, (50,), 11008 + 64, 32),
                                          (2, (33,), 8192, 128)])
def test_gemv_quad_shapes(oracle, shape, m, ns, k, block):
    _check(oracle, binding.TUNE_GEMV_QUAD, shape, m, ns, k, block)


@pytest.mark.parametrize("shape", [(1,), (3,), (16,)])
@pytest.mark.parametrize("m,ns,k", [(40, (300,), 2048 + 32), (100, (256, 132), 4096), (128, (200,), 1024)])
def test_gemm_slice_counts(oracle, shape, m, ns, k):
    _check(oracle, binding.TUNE_GEMM_SLICES, shape, m, ns, k)


@pytest.mark.parametrize("m,ns,k,block", [(8, (2100,), 1056, 16), (16, (4000,), 4096 + 64, 16), (12, (1400, 1400, 1396), 2048, 16),
                                          (5, (4100,), 11008, 16), (16, (8200,), 8192, 64)])
def test_untabled_small_batch_one_round_of_workgroups(oracle, m, ns, k, block):
    """Up to 16 activation rows, no table entry, and a number of 16-row groups that some G <= 4 turns into one
    round of workgroups: no workspace is asked for, results as the oracle's."""
    print("one-round heuristic m", m, "ns", ns, "k", k, "block", block, flush=True)
    assert razer.razer_tune_lookup(binding.TUNE_SMALL_BATCH, m, sum(ns), k)[0] == 0       # the heuristic applies
    if len(ns) == 1:
        assert razer.razer_workspace_bytes(binding.OP_LINEAR, ns[0], k, m) == 0
    else:                                       # (the grouped query also covers the fallback to one call per matrix)
        assert razer.razer_workspace_bytes_grouped(list(ns), k, m) == max(razer.razer_workspace_bytes(binding.OP_LINEAR, n, k, m) for n in ns)
    a = synth.activation(m, k, seed=9900 + m + k)
    a_dev = bf16_bits_to_dev(a)
    ws = [_rand_weights(n, k, 9950 + i + n, block) for i, n in enumerate(ns)]
    if len(ns) == 1:
        ys = [razer.razer_linear(ws[0][1], a_dev)]
    else:
        ys = razer.razer_linear_grouped([w[1] for w in ws], a_dev)
    torch.cuda.synchronize()
    for (wq, _), y in zip(ws, ys):
        y64, _ = oracle.linear(wq, a_bf16=a)
        assert max_rel_err(dev_to_bf16_bits(y), y64) <= TOL


@pytest.mark.parametrize("m,family,shape,kernel", [
    (8, None, None, "ring_kernel<2, 1, false, 0, 16,"), (8, binding.TUNE_SMALL_BATCH, (2, 1, 8), "ring_kernel<2, 1, false, 0, 8,"),
    (8, binding.TUNE_SMALL_BATCH, (2, 1, 16), "ring_kernel<2, 1, false, 0, 16,"), (8, binding.TUNE_SMALL_BATCH, (2, 1), "ring_kernel<2, 1, false, 0, 8,"),
    (8, binding.TUNE_SMALL_BATCH, (-1,), "ring_kernel<2, 1, false, 0, 16,"), (8, binding.TUNE_SMALL_BATCH, (2, 3, 16), "ring_kernel<2, 3, false, 0, 8,"),
    (4, binding.TUNE_SMALL_BATCH, (2, 3, 8), "ring_kernel<1, 1, false, 0, 16,"), (4, binding.TUNE_GEMV_QUAD, (8,), "gemv_quad_kernel"),
    (4, binding.TUNE_GEMV_QUAD, (-1,), "ring_kernel<1, 1, false, 0, 16,"), (64, binding.TUNE_GEMM_SLICES, (4,), "gemm_rb_kernel<4, 2, 1, 2,"),
    (64, binding.TUNE_GEMM_SLICES, (-1,), "ring_kernel<16, 1, false, 0, 8,"), (300, binding.TUNE_GEMM_SLICES, (4,), "gemm_pp_kernel")])
def test_a_forced_shape_launches_what_its_entry_would(m, family, shape, kernel):
    """A shape is timed by forcing it and used through the table: the same kernel, waves included.  -1 is the call as it
    runs with nothing forced, whichever kernel serves it."""
    n, k = 700, 4096
    _, wt = _rand_weights(n, k, 9990)
    a = bf16_bits_to_dev(synth.activation(m, k, seed=9991))
    if family is not None:
        razer.razer_tune_force(family, shape)
    try:
        razer.razer_linear(wt, a)
        names = launched_kernels(lambda: razer.razer_linear(wt, a))
        src = None if family is None else razer.razer_tune_lookup(family, m, n, k)[0]
    finally:
        razer.razer_tune_force(-1, None)
    assert src in (None, 0 if shape == (-1,) else 1)
    assert any(kernel in x for x in names), names


@pytest.mark.parametrize("m,ns,k,kernel", [
    # 33..64 rows, one group of rows per workgroup: both sides of the length of K
    (64, (2600,), 12288, "ring_kernel"), (64, (2600,), 12320, "gemm_rb_kernel"), (64, (4096,), 14336, "ring_kernel"), (48, (2600,), 16384, "gemm_rb_kernel"),
    (37, (4096,), 20480, "gemm_rb_kernel"), (37, (2600,), 16192, "ring_kernel"),
    # above 64 rows
    (128, (100,), 24576, "gemm_rb_kernel"), (65, (300,), 20480, "gemm_rb_kernel"), (128, (3000,), 28672, "gemm_rb_kernel"), (128, (1000,), 8192, "ring_kernel"),
    (1445, (720,), 15104, "gemm_"), (438, (10352,), 1216, "gemm_"), (2015, (220, 24), 28160, "gemm_"), (1454, (326,), 24960, "gemm_"),
    (512, (4096,), 4096, "ring_kernel"), (700, (300,), 4096, "ring_kernel"), (320, (5120, 5120), 5120, "ring_kernel"), (256, (1000,), 28672, "ring_kernel"),
    (1024, (1536, 1536, 1536), 1536, "ring_kernel"), (2048, (4096,), 4096, "gemm_"),
    (380, (2865,), 8832, "ring_kernel"), (1250, (899,), 6720, "ring_kernel"), (1390, (5539,), 1536, "ring_kernel"), (1514, (130,), 21696, "gemm_"), (1163, (5258,), 1088, "gemm_")])
def test_the_faster_kernel_is_chosen(m, ns, k, kernel):
    """Long rows of few weights are for the GEMM, which cuts K across workgroups; each call here is 5 % or more faster on
    the kernel named, or lies right at the line."""
    ws = [_rand_weights(n, k, 9996)[1] for n in ns]
    a = bf16_bits_to_dev(synth.activation(m, k, seed=9997))
    names = launched_kernels(lambda: razer.razer_linear(ws[0], a) if len(ws) == 1 else razer.razer_linear_grouped(ws, a))
    assert all(kernel in x or "slice_reduce" in x for x in names) and names, names
