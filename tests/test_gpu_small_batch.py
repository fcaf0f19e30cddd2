"""The small-batch kernel (5..64 activation rows, 2..4 with long rows, runs of 64 in small products) where its tiles,
steps and copies end: remainders of 16 rows and of 128 elements, K shorter than one step, every number of staged
activation rows, every number of row groups per workgroup, matrices of a group that share a workgroup, each weight format -- against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_2501_04052_amd as razer
from paper_2501_04052_amd import binding, synth
from gpu_util import TOL, bf16_bits_to_dev, dev_to_bf16_bits, launched_kernels, max_rel_err

pytestmark = pytest.mark.gpu
SV = (5.0, 8.0)


def _weights(n, k, seed, fmt, block):
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8)
    if fmt == razer.WEIGHT_F16:
        scales = rng.integers(0, 1 << 16, size=(n, k // 128)).astype(np.uint16)
    else:
        scales = rng.integers(0, 256, size=(n, k // block), dtype=np.uint8)
    wq = (codes, scales, np.float32(2.0 ** -9))
    return wq, razer.RazerTensor.from_host(*wq, fmt, SV)


def _run(oracle, ns, k, m, fmt, block, groups=None):
    print("small batch ns", ns, "k", k, "m", m, "format", fmt, "block", block, "groups", groups, flush=True)
    a = synth.activation(m, k, seed=4400 + m + k)
    a_dev = bf16_bits_to_dev(a)
    ws = [_weights(n, k, 4500 + i + n, fmt, block) for i, n in enumerate(ns)]
    if groups:
        razer.razer_tune_force(binding.TUNE_SMALL_BATCH, (2, groups))
    try:
        ys = [razer.razer_linear(ws[0][1], a_dev)] if len(ns) == 1 else razer.razer_linear_grouped([w[1] for w in ws], a_dev)
        torch.cuda.synchronize()
    finally:
        razer.razer_tune_force(binding.TUNE_SMALL_BATCH, None)
    for (wq, _), y in zip(ws, ys):
        y64, _ = oracle.linear(wq, a_bf16=a)
        assert max_rel_err(dev_to_bf16_bits(y), y64) <= TOL


@pytest.mark.parametrize("m", [5, 8, 9, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("ns,k,fmt,block", [((37,), 32, razer.WEIGHT, 16), ((16, 4, 100), 4096 + 96, razer.WEIGHT, 16),
                                            ((50,), 1152, razer.WEIGHT, 64), ((36, 20), 1280, razer.WEIGHT_F16, 128)])
def test_edges(oracle, m, ns, k, fmt, block):
    _run(oracle, ns, k, m, fmt, block)


@pytest.mark.parametrize("groups", [1, 2, 3, 4, 6])
@pytest.mark.parametrize("m,fmt,block", [(8, razer.WEIGHT, 16), (16, razer.WEIGHT, 32), (32, razer.WEIGHT, 16), (64, razer.WEIGHT, 16),
                                         (32, razer.WEIGHT_F16, 128), (64, razer.WEIGHT_F16, 128)])
def test_groups_per_workgroup(oracle, groups, m, fmt, block):
    _run(oracle, (68, 33 * 4, 12), 2176, m, fmt, block, groups)


@pytest.mark.parametrize("m", [2, 3, 4])
@pytest.mark.parametrize("ns,k,fmt,block", [((37,), 8192 + 32, razer.WEIGHT, 16), ((2100, 2100, 4), 6144, razer.WEIGHT, 16),
                                            ((50, 3), 8192 + 64, razer.WEIGHT, 64), ((36, 20), 8192 + 128, razer.WEIGHT_F16, 128)])
def test_few_rows_with_long_k(oracle, m, ns, k, fmt, block):
    _run(oracle, ns, k, m, fmt, block)


@pytest.mark.parametrize("m", [65, 128, 129, 321])
@pytest.mark.parametrize("ns,k,fmt,block", [((37,), 32, razer.WEIGHT, 16), ((16, 4, 100), 1024 + 96, razer.WEIGHT, 16),
                                            ((50,), 1152, razer.WEIGHT, 64), ((36, 20), 1280, razer.WEIGHT_F16, 128)])
def test_runs_of_activation_rows(oracle, m, ns, k, fmt, block):
    _run(oracle, ns, k, m, fmt, block)


@pytest.mark.parametrize("m,n,k,fmt,block", [(9, 37, 4096 + 96, razer.WEIGHT, 16), (16, 70, 4096, razer.WEIGHT, 64), (16, 20, 4224, razer.WEIGHT_F16, 128),
                                             (40, 37, 10240 + 96, razer.WEIGHT, 16), (64, 20, 10240, razer.WEIGHT_F16, 128), (33, 16485, 160, razer.WEIGHT, 16), (64, 16485, 192, razer.WEIGHT, 32), (64, 16485, 128, razer.WEIGHT_F16, 128),
                                             (9, 37, 6784 + 64, razer.WEIGHT, 16), (16, 700, 4800, razer.WEIGHT, 64), (16, 20, 10624, razer.WEIGHT_F16, 128)])
def test_number_of_waves(oracle, m, n, k, fmt, block):
    """16 waves with one group per workgroup and rows long enough; fewer where K has fewer steps than waves."""
    _run(oracle, (n,), k, m, fmt, block)


@pytest.mark.parametrize("m,k,fmt,block", [(33, 1184, razer.WEIGHT, 16), (64, 1280 + 96, razer.WEIGHT, 32), (64, 1280, razer.WEIGHT_F16, 128), (130, 1152, razer.WEIGHT, 16)])
def test_four_waves_where_workgroups_outnumber_compute_units(oracle, m, k, fmt, block):
    """Nine steps of K and more, so that every wave takes a second one; the order of the sum is another than that of the
    eight waves which a forced shape asks for."""
    n = 16485
    print("four waves", m, k, fmt, block, flush=True)
    a = synth.activation(m, k, seed=4600 + m)
    a_dev = bf16_bits_to_dev(a)
    wq, wt = _weights(n, k, 4601 + k, fmt, block)
    got = []
    names = launched_kernels(lambda: got.append(razer.razer_linear(wt, a_dev)))
    groups = [int(x.split("ring_kernel<")[1].split(",")[1]) for x in names if "ring_kernel<16," in x]
    assert len(groups) == 1 == len(names), names
    assert -(-n // 16 // groups[0]) * -(-m // 64) > 256                # workgroups
    razer.razer_tune_force(binding.TUNE_SMALL_BATCH, (2, groups[0], 8))
    try:
        eight = dev_to_bf16_bits(razer.razer_linear(wt, a_dev))
    finally:
        razer.razer_tune_force(binding.TUNE_SMALL_BATCH, None)
    got = dev_to_bf16_bits(got[0])
    cols = np.unique(np.r_[0, n - 1, n - 17, np.random.default_rng(46).choice(n, size=200, replace=False)])
    y64, _ = oracle.linear((wq[0][cols], wq[1][cols], wq[2]), a_bf16=a)
    for y in (got, eight):
        assert max_rel_err(y[:, cols], y64) <= TOL
    assert (got != eight).any()


@pytest.mark.parametrize("m,n,k,block,groups,halves", [(130, 37, 9312, 16, None, 1), (130, 37, 9312, 32, None, 1), (130, 37, 4128, 16, None, 2), (64, 3077, 224, 16, None, 1),
                                                       (64, 37, 4128, 16, 2, 1), (50, 37, 8224, 32, 2, 1), (64, 37, 3360, 16, 2, 2), (64, 37, 4160, 16, 2, 2),
                                                       (16, 37, 6688, 16, None, 1), (12, 37, 6688, 32, None, 2), (12, 37, 4128, 32, None, 1)])
def test_steps_of_rows_that_start_inside_a_line(oracle, m, n, k, block, groups, halves):
    """K of an odd number of 32-element runs: whole steps where many rows are read, halves elsewhere."""
    a = bf16_bits_to_dev(synth.activation(m, k, seed=4800))
    wt = _weights(n, k, 4801, razer.WEIGHT, block)[1]
    if groups:
        razer.razer_tune_force(binding.TUNE_SMALL_BATCH, (2, groups))
    try:
        names = launched_kernels(lambda: razer.razer_linear(wt, a))
    finally:
        razer.razer_tune_force(binding.TUNE_SMALL_BATCH, None)
    if m > 16:
        assert any("ring_kernel<16," in x and ", %d, 8, false>" % (0 if halves == 2 else 2) in x for x in names), names
    else:                                                             # (16 waves with halves, 8 with whole steps)
        assert any("ring_kernel<4," in x and ", %d, false>" % (8 * halves) in x for x in names), names
    _run(oracle, (n,), k, m, razer.WEIGHT, block, groups)


@pytest.mark.parametrize("m,n,k,fmt,waves", [(16, 4096, 4096, razer.WEIGHT, 8), (9, 704, 4608, razer.WEIGHT, 8), (9, 704, 4736, razer.WEIGHT, 16), (12, 300, 6656, razer.WEIGHT, 8),
                                             (12, 300, 6784, razer.WEIGHT, 16), (16, 300, 10496, razer.WEIGHT_F16, 8), (16, 300, 10624, razer.WEIGHT_F16, 16)])
def test_sixteen_waves_where_rows_are_long(m, n, k, fmt, waves):
    """9..16 rows, both sides of the lengths from which 16 waves are faster."""
    a = bf16_bits_to_dev(synth.activation(m, k, seed=4900))
    wt = _weights(n, k, 4901, fmt, 16)[1]
    names = launched_kernels(lambda: razer.razer_linear(wt, a))
    assert len(names) == 1 and ", %d, false>" % waves in names[0] and "ring_kernel<4, 1," in names[0], names


def test_runs_of_activation_rows_keep_to_a_strided_output(oracle):
    n, k, m = 37, 256, 130
    a = synth.activation(m, k, seed=4700)
    wq, w = _weights(n, k, 4701, razer.WEIGHT, 16)
    buf = torch.full((m + 1, n + 11), 77.0, dtype=torch.bfloat16, device="cuda")
    razer.razer_linear(w, bf16_bits_to_dev(a), out=buf[:m, :n])
    y64, _ = oracle.linear(wq, a_bf16=a)
    assert max_rel_err(dev_to_bf16_bits(buf[:m, :n].contiguous()), y64) <= TOL
    assert bool((buf[:m, n:] == 77.0).all()) and bool((buf[m] == 77.0).all())


@pytest.mark.parametrize("m", [6, 40])
def test_infinite_activation_stays_infinite_with_a_ragged_last_step(oracle, m):
    """Lanes past K re-read the step's first elements with the activations cleared: an infinity there must not meet
    the weights of the tail (0 x Inf is NaN), and must not reach other rows."""
    n, k = 48, 96
    wq, wt = _weights(n, k, 77, razer.WEIGHT, 16)
    a = torch.from_numpy(synth.bf16_bits_to_f32(synth.activation(m, k, seed=78))).to(torch.bfloat16)
    plain = razer.razer_linear(wt, a.cuda())
    a[2, 0] = float("inf")
    got = razer.razer_linear(wt, a.cuda()).float().cpu()
    w0 = torch.from_numpy(oracle.dequant(oracle.WEIGHT, *wq)["f32"])[:, 0].float()
    hit = w0 != 0
    assert torch.equal(got[2][hit], torch.sign(w0[hit]) * float("inf"))
    others = [i for i in range(m) if i != 2]
    assert torch.equal(got[others], plain.float().cpu()[others])


@pytest.mark.parametrize("m,ns,k,fmt,block,groups", [
    # rows of 256, 262, 518 and of 64 .. 4 bytes of scales, the last rows of a matrix, several matrices in one workgroup
    (8, (68, 33 * 4, 12), 4096, razer.WEIGHT, 16, 6), (5, (100, 7), 4192, razer.WEIGHT, 16, 6), (16, (37,), 8288, razer.WEIGHT, 16, 3), (32, (36, 20), 4096, razer.WEIGHT, 32, 6),
    (8, (50, 3), 8192 + 64, razer.WEIGHT, 64, 3), (33, (68, 5), 4608, razer.WEIGHT, 128, 4), (64, (37, 40), 6176, razer.WEIGHT, 16, 4), (50, (70,), 6144, razer.WEIGHT, 32, 4),
    (16, (36, 20), 4096, razer.WEIGHT_F16, 128, 6), (64, (52,), 8320, razer.WEIGHT_F16, 128, 3), (12, (21,), 38528, razer.WEIGHT, 16, 1),
    # up to 4 rows: two, three and four groups, one with 16 waves; 16 waves with whole steps and with halves
    (4, (4200,), 20512, razer.WEIGHT, 16, None), (3, (5000, 3300, 20), 8224, razer.WEIGHT, 16, None), (4, (13000,), 6208, razer.WEIGHT, 64, None), (3, (4200,), 20480, razer.WEIGHT_F16, 128, None),
    (4, (37,), 38432, razer.WEIGHT, 32, None), (8, (21,), 38432, razer.WEIGHT, 16, None), (12, (21,), 38464, razer.WEIGHT, 16, None), (16, (37,), 38528, razer.WEIGHT_F16, 128, None),
    # several workgroups per unit
    (8, (16485,), 2080, razer.WEIGHT, 16, None), (40, (16485,), 2048, razer.WEIGHT, 64, None), (16, (16485,), 5248, razer.WEIGHT_F16, 128, None)])
def test_scales_staged_by_the_workgroup(oracle, m, ns, k, fmt, block, groups):
    ws = [_weights(n, k, 5000 + i + n, fmt, block) for i, n in enumerate(ns)]
    a = synth.activation(m, k, seed=5100 + m)
    a_dev = bf16_bits_to_dev(a)
    print("staged scales", m, ns, k, fmt, block, groups, flush=True)
    got = []
    if groups:
        razer.razer_tune_force(binding.TUNE_SMALL_BATCH, (2, groups))
    try:
        names = launched_kernels(lambda: got.extend([razer.razer_linear(ws[0][1], a_dev)] if len(ns) == 1 else razer.razer_linear_grouped([w[1] for w in ws], a_dev)))
    finally:
        razer.razer_tune_force(binding.TUNE_SMALL_BATCH, None)
    assert names and all("staged_ring_kernel<" in x for x in names), names
    if k > 38400 and not groups:
        assert all(x.split("<")[1].split(",")[4].strip() == "16" for x in names), names      # (waves)
    for (wq, _), y in zip(ws, got):
        n = len(wq[0])
        cols = np.arange(n) if n < 300 else np.unique(np.r_[0:20, n - 37:n, np.random.default_rng(47).choice(n, size=200, replace=False)])
        y64, _ = oracle.linear((wq[0][cols], wq[1][cols], wq[2]), a_bf16=a)
        assert max_rel_err(dev_to_bf16_bits(y)[:, cols], y64) <= TOL


@pytest.mark.parametrize("m,n,k,block,groups", [
    # ragged rows, steps and last slices; outputs that are no multiple of 4; two and four groups per workgroup
    (64, 37, 8192 + 96, 16, 2), (33, 100, 8192, 32, 2), (40, 1000, 11008, 16, 2), (64, 129, 9216 + 64, 64, 2), (64, 4096, 11008, 16, 2), (64, 5120, 13824, 16, 4),
    (56, 5121, 13824, 32, 4)])
def test_k_slices(oracle, m, n, k, block, groups):
    """Few weight rows with long K: slices of K, their sums in the workspace; one infinite activation stays in its row."""
    print("k slices", m, n, k, block, flush=True)
    wq, wt = _weights(n, k, 5200 + n, razer.WEIGHT, block)
    a = synth.activation(m, k, seed=5300 + m)
    a_dev = bf16_bits_to_dev(a)
    got = []
    names = launched_kernels(lambda: got.append(razer.razer_linear(wt, a_dev)))
    assert any("sliced_ring_kernel<16, %d," % groups in x for x in names) and any("slice_reduce" in x for x in names) and len(names) == 2, names
    cols = np.arange(n) if n < 300 else np.unique(np.r_[0:20, n - 37:n, np.random.default_rng(48).choice(n, size=200, replace=False)])
    y64, _ = oracle.linear((wq[0][cols], wq[1][cols], wq[2]), a_bf16=a)
    assert max_rel_err(dev_to_bf16_bits(got[0])[:, cols], y64) <= TOL
    a_dev[2, k - 3] = float("inf")
    z = razer.razer_linear(wt, a_dev).float().cpu()
    wc = torch.from_numpy(oracle.dequant(oracle.WEIGHT, wq[0][cols], wq[1][cols], wq[2])["f32"])[:, k - 3].float()
    assert bool((z[2][torch.from_numpy(cols)[wc != 0]] == torch.sign(wc[wc != 0]) * float("inf")).all())
    others = [i for i in range(m) if i != 2]
    assert torch.equal(z[others], got[0].float().cpu()[others])


@pytest.mark.parametrize("m,n,k,block", [(32, 2048, 12288, 16), (17, 16, 14336, 16), (20, 1000, 11008, 16), (24, 520, 12288, 128), (16, 300, 16384, 16), (5, 4096, 4096, 16)])
def test_the_workspace_is_not_written_up_to_32_rows(m, n, k, block):
    """It is asked for and checked, but calls that overlap may share it and its bytes are the caller's."""
    print("workspace", m, n, k, block, flush=True)
    _, wt = _weights(n, k, 5400 + n, razer.WEIGHT, block)
    a_dev = bf16_bits_to_dev(synth.activation(m, k, seed=5500 + m))
    ws = torch.full((max(razer.razer_workspace_bytes(binding.OP_LINEAR, n, k, m), 16),), 0xA5, dtype=torch.uint8, device="cuda")
    razer.razer_linear(wt, a_dev, workspace=ws)
    out = torch.empty((m, n), dtype=torch.bfloat16, device="cuda")
    razer.prepare_linear(wt, a_dev, out, workspace=ws)()
    assert bool((ws == 0xA5).all())


@pytest.mark.parametrize("m,n,k,block", [(64, 4096, 11008, 16), (40, 1000, 11008, 32), (64, 5120, 13824, 16), (33, 100, 8192, 16), (32, 2048, 12288, 16), (17, 16, 14336, 16), (64, 4096, 4096, 16),
                                         (64, 1000, 16384, 16), (100, 2048, 4096, 16)])
def test_a_group_of_one_matrix_is_the_single_call(m, n, k, block):
    """Up to 128 rows the same kernels, launched alike: the same bits."""
    print("group of one", m, n, k, block, flush=True)
    _, wt = _weights(n, k, 5600 + n, razer.WEIGHT, block)
    a_dev = bf16_bits_to_dev(synth.activation(m, k, seed=5700 + m))
    one, group = [], []
    single = launched_kernels(lambda: one.append(razer.razer_linear(wt, a_dev)))
    grouped = launched_kernels(lambda: group.extend(razer.razer_linear_grouped([wt], a_dev)))
    assert torch.equal(one[0], group[0]), (single, grouped)


@pytest.mark.parametrize("m,n,k", [(40, 1000, 11008), (64, 5120, 13824), (33, 1003, 11008)])
def test_k_slices_into_any_output(oracle, m, n, k):
    """Rows of the output further apart than N, one that starts 2 bytes behind an 8-byte boundary, the entry without a
    workspace argument, activations in their own format: the same sums."""
    print("k slices, outputs", m, n, k, flush=True)
    wq, wt = _weights(n, k, 5800 + n, razer.WEIGHT, 16)
    a_dev = bf16_bits_to_dev(synth.activation(m, k, seed=5900 + m))
    want = razer.razer_linear(wt, a_dev)
    ld = (n + 11) // 8 * 8
    for ld_y, offset in ((ld, 0), (ld + 3, 0), (ld, 1), (ld + 1, 3)):
        buf = torch.full((m * ld_y + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
        out = torch.as_strided(buf, (m, n), (ld_y, 1), offset)
        names = launched_kernels(lambda: razer.razer_linear(wt, a_dev, out=out))
        assert any("sliced_ring_kernel<" in x for x in names), names
        assert torch.equal(out, want), (ld_y, offset)
        out.fill_(7.0)
        assert bool((buf == 7.0).all()), (ld_y, offset)                  # (nothing beside the outputs)
    out = torch.empty_like(want)
    assert torch.equal(razer.razer_linear_static(wt, a_dev, out), want)
    aq = razer.razer_quantize(a_dev, razer.ACT, (5.0,))
    names = launched_kernels(lambda: razer.razer_linear(wt, aq, out=out))
    assert any("sliced_ring_kernel<" in x for x in names), names
    y64, _ = oracle.linear(wq, a_q=tuple(x.cpu().numpy() for x in (aq.codes, aq.scales)) + (np.float32(aq.tensor_scale.item()),))
    assert max_rel_err(dev_to_bf16_bits(out), y64) <= TOL
