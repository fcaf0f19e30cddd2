"""The 256 x 256 tiles of the register-decode GEMM (64 weight rows per wave, three copy stages) where they end: ragged
rows, ragged K (a last tile of 32 elements), odd and even numbers of K-tiles, tiles past the matrices of a group, each
block size -- against the CPU oracle on sampled rows."""
import numpy as np
import pytest
import torch

import paper_2501_04052_amd as razer
from paper_2501_04052_amd import binding, synth
from gpu_util import TOL, bf16_bits_to_dev, dev_to_bf16_bits, launched_kernels, max_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,ns,k,block", [(300, (16500,), 2048, 16), (257, (16640, 40), 2080, 16), (512, (12000, 5000), 2112, 32),
                                          (300, (17000,), 2176, 128), (512, (17000,), 2080, 32), (512, (12000, 5000), 2080, 32),
                                          (2048, (24600,), 2080, 16)])          # (the last one: more than three rounds of 128-wide tiles)
def test_wide_tiles(oracle, m, ns, k, block):
    print("wide tiles m", m, "ns", ns, "k", k, "block", block, flush=True)
    a = synth.activation(m, k, seed=8100 + m)
    rows = np.sort(np.random.default_rng(8).choice(m, size=12, replace=False))
    rows[-1], rows[0] = m - 1, 0
    rng = np.random.default_rng(81 + k)
    ws = []
    for n in ns:
        wq = (rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8), rng.integers(0, 256, size=(n, k // block), dtype=np.uint8),
              np.float32(2.0 ** -9))
        ws.append((wq, razer.RazerTensor.from_host(*wq, razer.WEIGHT, (5.0, 8.0))))
    a_dev = bf16_bits_to_dev(a)
    ys = [razer.razer_linear(ws[0][1], a_dev)] if len(ns) == 1 else razer.razer_linear_grouped([w[1] for w in ws], a_dev)
    torch.cuda.synchronize()
    for (wq, _), y in zip(ws, ys):
        cols = np.r_[0:40, 240:272, wq[0].shape[0] - 40:wq[0].shape[0]] if wq[0].shape[0] > 300 else np.arange(wq[0].shape[0])
        y64, _ = oracle.linear((wq[0][cols], wq[1][cols], wq[2]), a_bf16=a[rows])
        assert max_rel_err(dev_to_bf16_bits(y)[rows][:, cols], y64) <= TOL


@pytest.mark.parametrize("m,n,k,block,kernel", [
    # 256 x 128 tiles with two K groups: 42 and 43 K-tiles per slice, the shortest slices that take it with few and with many workgroups
    (257, 260, 21568, 16, "gemm_rb_kernel<8, 2, 2, 8, false>"), (140, 130, 22016, 16, "gemm_rb_kernel<8, 2, 2, 8, false>"),
    (300, 389, 21696, 16, "gemm_rb_kernel<8, 2, 2, 8, false>"), (257, 389, 21760, 32, "gemm_rb_kernel<8, 2, 2, 8, true>"),
    (300, 261, 21504, 64, "gemm_rb_kernel<8, 2, 2, 8, true>"), (300, 389, 9152, 16, "gemm_rb_kernel<8, 2, 2, 8, false>"),
    (512, 1664, 15360, 16, "gemm_rb_kernel<8, 2, 2, 8, false>"),
    # the LDS-staged tiles: shorter slices, K that ends inside a K-tile, one width of tiles as good as the other
    (512, 1664, 14848, 16, "gemm_pp_kernel<256, 128,"), (600, 1280, 9280, 16, "gemm_pp_kernel<256, 128,"), (257, 260, 22048, 16, "gemm_pp_kernel<256, 128,"), (257, 260, 8320, 32, "gemm_pp_kernel<256, 128,"),
    (140, 130, 8256, 64, "gemm_pp_kernel<256, 128,"), (129, 100, 8192, 16, "gemm_pp_kernel<256, 256,"), (130, 37, 8224, 16, "gemm_pp_kernel<256, 256,"),
    (300, 5, 8288, 16, "gemm_pp_kernel<256, 256,")])
def test_k_slices_of_few_tiles(oracle, m, n, k, block, kernel):
    """Few tiles, K cut into slices whose last one is shorter, against the CPU oracle on sampled rows, each on the kernel
    that its lengths call for."""
    rng = np.random.default_rng(m + n + k)
    wq = (rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8), rng.integers(0, 256, size=(n, k // block), dtype=np.uint8), np.float32(2.0 ** -9))
    w = razer.RazerTensor.from_host(*wq, razer.WEIGHT, (5.0, 8.0))
    a = synth.activation(m, k, seed=9100 + m)
    rows = np.unique(np.r_[0, rng.choice(m, size=22, replace=False), 127, 128, m - 1])
    print("k slices", m, n, k, block, flush=True)
    razer.razer_tune_force(binding.TUNE_GEMM_SLICES, (2,))       # (a forced shape keeps the call off the small-batch kernel)
    try:
        got = []
        names = launched_kernels(lambda: got.append(razer.razer_linear(w, bf16_bits_to_dev(a))))
    finally:
        razer.razer_tune_force(binding.TUNE_GEMM_SLICES, None)
    assert any(kernel in x for x in names), names
    y64, _ = oracle.linear(wq, a_bf16=a[rows])
    assert max_rel_err(dev_to_bf16_bits(got[0])[rows], y64) <= TOL


@pytest.mark.parametrize("m,n,k,column,kernel", [(257, 260, 22016, 43 * 64, "gemm_rb_kernel<8, 2, 2, 8,"),          # (K-slices of 43 tiles)
                                                 (2000, 4096, 1088, 1087, "gemm_rb_kernel<8, 2, 2, 8,"),             # (17 tiles in one slice)
                                                 (300, 389, 8224, 3, "gemm_pp_kernel"), (257, 260, 22048, 22016, "gemm_pp_kernel")])
def test_infinite_activation_stays_infinite(oracle, m, n, k, column, kernel):
    """256 x 128 tiles: a K-tile that one of two K groups does not have, and the half of a last K-tile past K, must not
    multiply an infinity by a weight of 0 (NaN), and the infinity must not reach other rows."""
    rng = np.random.default_rng(m + n + k)
    wq = (rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8), rng.integers(0, 256, size=(n, k // 16), dtype=np.uint8), np.float32(2.0 ** -9))
    w = razer.RazerTensor.from_host(*wq, razer.WEIGHT, (5.0, 8.0))
    a = torch.from_numpy(synth.bf16_bits_to_f32(synth.activation(m, k, seed=9200 + m))).to(torch.bfloat16)
    print("infinity", m, n, k, column, flush=True)
    razer.razer_tune_force(binding.TUNE_GEMM_SLICES, (1,))       # (keeps the call off the small-batch kernel)
    try:
        plain = razer.razer_linear(w, a.cuda()).float().cpu()
        a[2, column] = float("inf")
        got = []
        names = launched_kernels(lambda: got.append(razer.razer_linear(w, a.cuda())))
    finally:
        razer.razer_tune_force(binding.TUNE_GEMM_SLICES, None)
    assert any(kernel in x for x in names), names
    got = got[0].float().cpu()
    wc = torch.from_numpy(oracle.dequant(oracle.WEIGHT, *wq)["f32"])[:, column].float()
    hit = wc != 0
    assert bool((got[2][hit] == torch.sign(wc[hit]) * float("inf")).all())
    others = [i for i in range(m) if i != 2]
    assert bool((got[others] == plain[others]).all())


@pytest.mark.parametrize("m,ns,k,block,kernel", [
    # one round of 256 x 128 tiles with two K groups: even and odd numbers of K-tiles, a last one of 32 elements, three rows of tiles
    (300, (12300,), 2048, 16, "gemm_halves_kernel<false>"), (257, (12300,), 2112, 16, "gemm_halves_kernel<false>"), (300, (12164,), 2080, 32, "gemm_halves_kernel<true>"),
    (520, (8200,), 2176, 64, "gemm_halves_kernel<true>"), (300, (6200, 36, 6000), 2112, 16, "gemm_halves_grouped_kernel<false>"),
    (300, (6200, 6100), 2176, 128, "gemm_halves_grouped_kernel<true>"),
    # whole 256 x 256 tiles and a last round of half tiles, the last half of a matrix past its rows
    (300, (32800,), 2048, 16, "gemm_wide_kernel<false>"), (513, (22100,), 2080, 16, "gemm_wide_kernel<false>"), (300, (20000, 13000), 2112, 16, "gemm_wide_grouped_kernel<false>"),
    (513, (9000, 40, 13100), 2080, 32, "gemm_wide_grouped_kernel<true>"),
    # long K-slices, the last one shorter, odd numbers of K-tiles in a slice
    (512, (4096,), 11008, 16, "gemm_halves_kernel<false>"), (400, (4100,), 11072, 16, "gemm_halves_kernel<false>"), (300, (5003,), 13888, 32, "gemm_halves_kernel<true>")])
def test_half_tiles(oracle, m, ns, k, block, kernel):
    """... and an infinite activation stays infinite and in its row."""
    rng = np.random.default_rng(m + sum(ns) + k)
    a = synth.activation(m, k, seed=9300 + m)
    rows = np.unique(np.r_[0, 2, rng.choice(m, size=10, replace=False), 255, 256, m - 1])
    ws = []
    for n in ns:
        wq = (rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8), rng.integers(0, 256, size=(n, k // block), dtype=np.uint8), np.float32(2.0 ** -9))
        ws.append((wq, razer.RazerTensor.from_host(*wq, razer.WEIGHT, (5.0, 8.0))))
    print("half tiles", m, ns, k, block, flush=True)
    a_dev = bf16_bits_to_dev(a)
    call = lambda: [razer.razer_linear(ws[0][1], a_dev)] if len(ns) == 1 else razer.razer_linear_grouped([w[1] for w in ws], a_dev)  # noqa: E731
    plain, got = [], []
    column = k - 7                                               # (in the last K-tile, whole or not)
    razer.razer_tune_force(binding.TUNE_GEMM_SLICES, (1,))       # (keeps the call off the small-batch kernel)
    try:
        names = launched_kernels(lambda: plain.extend(call()))
        a_dev[2, column] = float("inf")
        got = call()
    finally:
        razer.razer_tune_force(binding.TUNE_GEMM_SLICES, None)
    assert any(kernel in x for x in names) and all(kernel in x or "slice_reduce" in x for x in names), names
    for (wq, _), y, z in zip(ws, plain, got):
        n = len(wq[0])
        cols = np.arange(n) if n < 300 else np.unique(np.r_[0:40, 120:136, 250:262, n - 40:n, rng.choice(n, size=60, replace=False)])
        y64, _ = oracle.linear((wq[0][cols], wq[1][cols], wq[2]), a_bf16=a[rows])
        assert max_rel_err(dev_to_bf16_bits(y)[rows][:, cols], y64) <= TOL
        z, y = z.float().cpu(), y.float().cpu()
        wc = torch.from_numpy(oracle.dequant(oracle.WEIGHT, wq[0][cols], wq[1][cols], wq[2])["f32"])[:, column].float()
        hit = torch.from_numpy(cols)[wc != 0]
        assert bool((z[2][hit] == torch.sign(wc[wc != 0]) * float("inf")).all())
        others = [i for i in range(m) if i != 2]
        assert bool((z[others] == y[others]).all())


@pytest.mark.parametrize("m,ns,k,block,kernel", [
    # half tiles (16 and 17 K-tiles per group, the second group's last one ragged), whole ones, a launch of both
    (300, (12300,), 2080, 16, "gemm_halves_kernel<false>"), (257, (12164,), 2144, 32, "gemm_halves_kernel<true>"), (300, (6200, 36, 6000), 2080, 16, "gemm_halves_grouped_kernel<false>"),
    (257, (16640,), 2080, 16, "gemm_wide_kernel<false>"), (513, (22100,), 2080, 32, "gemm_wide_kernel<true>"), (300, (20000, 13000), 2144, 16, "gemm_wide_grouped_kernel<false>"),
    # 32 weight rows per wave: 64, 128 and 256 activation rows per tile, two K groups, with and without K-slices, grouped
    (64, (300,), 2080, 16, "gemm_rb_kernel<4, 2, 1, 2, false>"), (40, (300,), 96, 32, "gemm_rb_kernel<4, 2, 1, 2, true>"), (33, (130,), 32, 16, "gemm_rb_kernel<4, 2, 1, 2, false>"),
    (128, (300,), 8224, 16, "gemm_rb_kernel<4, 2, 1, 4, false>"), (100, (300, 40), 2144, 32, "gemm_rb_grouped_kernel<4, 2, 1, 4, true>"),
    (2040, (8200,), 1056, 16, "gemm_rb_kernel<4, 2, 1, 8, false>"), (300, (300, 40), 2080, 16, "gemm_rb_grouped_kernel<4, 2, 1, 8, false>"),
    (2000, (4090,), 1056, 16, "gemm_rb_kernel<8, 2, 2, 8, false>"), (2000, (4090,), 1120, 32, "gemm_rb_kernel<8, 2, 2, 8, true>"), (2000, (2040, 2044), 1056, 16, "gemm_rb_grouped_kernel<8, 2, 2, 8, false>")])
def test_infinities_in_rows_that_end_inside_a_k_tile(oracle, m, ns, k, block, kernel):
    """The last K-tile has 32 elements, and what stands in the place of the others may not be anything that a weight of 0
    makes a NaN of: a row with one infinity, at either end of the row or of a K-tile, is infinite wherever that weight is not 0."""
    rng = np.random.default_rng(m + sum(ns) + k)
    a = torch.from_numpy(synth.bf16_bits_to_f32(synth.activation(m, k, seed=9400 + m))).to(torch.bfloat16).cuda()
    end = k // 64 * 64
    columns = {row: c for row, c in zip((0, 3, 6, 9, 12, 15, m - 5, m - 3, m - 1), (0, 7, 31, 32, 63, end - 1, end, k - 8, k - 1)) if 0 <= c < k}
    print("infinities", m, ns, k, block, flush=True)
    ws = [(rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8), rng.integers(0, 256, size=(n, k // block), dtype=np.uint8), np.float32(2.0 ** -9)) for n in ns]
    wts = [razer.RazerTensor.from_host(*wq, razer.WEIGHT, (5.0, 8.0)) for wq in ws]
    call = lambda: [razer.razer_linear(wts[0], a)] if len(ns) == 1 else razer.razer_linear_grouped(wts, a)  # noqa: E731
    got = []
    razer.razer_tune_force(binding.TUNE_GEMM_SLICES, (1,))       # (keeps the call off the small-batch kernel)
    try:
        plain = call()
        for row, column in columns.items():
            a[row, column] = float("inf") if row % 2 else -float("inf")
        names = launched_kernels(lambda: got.extend(call()))
    finally:
        razer.razer_tune_force(binding.TUNE_GEMM_SLICES, None)
    assert any(kernel in x for x in names), names
    others = [i for i in range(m) if i not in columns]
    for wq, y, z in zip(ws, plain, got):
        sample = np.arange(len(wq[0])) if len(wq[0]) < 300 else np.unique(np.r_[0:40, 120:136, len(wq[0]) - 140:len(wq[0]), rng.choice(len(wq[0]), size=60, replace=False)])
        w = torch.from_numpy(oracle.dequant(oracle.WEIGHT, wq[0][sample], wq[1][sample], wq[2])["f32"])
        y, z = y.float().cpu()[:, sample], z.float().cpu()[:, sample]
        for row, column in columns.items():
            hit = w[:, column] != 0
            assert torch.equal(z[row][hit], torch.sign(w[hit, column]) * (float("inf") if row % 2 else -float("inf"))), (row, column)
        assert torch.equal(z[others], y[others])


@pytest.mark.parametrize("m,ns,k,kernel", [(2000, (10500,), 2048, "gemm_wide_kernel"), (700, (31000,), 2080, "gemm_wide_kernel"), (2048, (4096, 4096, 4096), 2048, "gemm_wide_grouped_kernel"),
                                           (1100, (9000, 40, 7400), 2112, "gemm_wide_grouped_kernel"), (1900, (4000,), 5120, "gemm_halves_kernel"), (700, (8100,), 1024, "gemm_"),
                                           (3, (4096,), 4096, "gemv_"), (4, (37,), 11008, "ring_kernel"), (13, (4096,), 11008, "ring_kernel"), (50, (1000,), 11008, "sliced_ring_kernel"), (500, (4096,), 4096, "ring_kernel")])
def test_equal_rows_of_a_call_have_equal_results(m, ns, k, kernel):
    """What an activation row gives does not depend on where it stands in the call: the order of the sum over K is a
    matter of the output's column."""
    rng = np.random.default_rng(m + k)
    ws = [razer.RazerTensor.from_host(rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8), rng.integers(0, 256, size=(n, k // 16), dtype=np.uint8), np.float32(2.0 ** -9), razer.WEIGHT, (5.0, 8.0)) for n in ns]
    a_dev = bf16_bits_to_dev(synth.activation(1, k, seed=9500 + m)).expand(m, k).contiguous()
    print("equal rows", m, ns, k, flush=True)
    got = []
    if kernel.startswith("gemm"):
        razer.razer_tune_force(binding.TUNE_GEMM_SLICES, (1,))   # (keeps the call off the small-batch kernel)
    try:
        names = launched_kernels(lambda: got.extend([razer.razer_linear(ws[0], a_dev)] if len(ns) == 1 else razer.razer_linear_grouped(ws, a_dev)))
    finally:
        razer.razer_tune_force(binding.TUNE_GEMM_SLICES, None)
    assert any(kernel in x for x in names), names
    for y in got:
        assert torch.equal(y, y[:1].expand_as(y))


@pytest.mark.parametrize("m,n,k,kernel", [(300, 12300, 2080, "gemm_halves_kernel"), (513, 22100, 2048, "gemm_wide_kernel"), (512, 4100, 11008, "gemm_halves_kernel"), (300, 32803, 2048, "gemm_wide_kernel")])
def test_half_tiles_into_any_output(oracle, m, n, k, kernel):
    """Rows of the output further apart than N, one that starts 2 bytes behind a 16-byte boundary, the entry without a
    workspace argument, activations in their own format: the same sums."""
    rng = np.random.default_rng(m + n + k)
    wq = (rng.integers(0, 256, size=(n, k // 2), dtype=np.uint8), rng.integers(0, 256, size=(n, k // 16), dtype=np.uint8), np.float32(2.0 ** -9))
    w = razer.RazerTensor.from_host(*wq, razer.WEIGHT, (5.0, 8.0))
    a_dev = bf16_bits_to_dev(synth.activation(m, k, seed=9600 + m))
    print("half tiles, outputs", m, n, k, flush=True)
    razer.razer_tune_force(binding.TUNE_GEMM_SLICES, (1,))       # (keeps the call off the small-batch kernel)
    try:
        want = razer.razer_linear(w, a_dev)
        ld = (n + 11) // 8 * 8
        for ld_y, offset in ((ld, 0), (ld + 3, 0), (ld, 1), (ld + 4, 4)):
            buf = torch.full((m * ld_y + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
            out = torch.as_strided(buf, (m, n), (ld_y, 1), offset)
            names = launched_kernels(lambda: razer.razer_linear(w, a_dev, out=out))
            assert any(kernel in x for x in names), names
            assert torch.equal(out, want), (ld_y, offset)
            out.fill_(7.0)
            assert bool((buf == 7.0).all()), (ld_y, offset)              # (nothing beside the outputs)
        out = torch.empty_like(want)
        assert torch.equal(razer.razer_linear_static(w, a_dev, out), want)
        aq = razer.razer_quantize(a_dev, razer.ACT, (5.0,))
        names = launched_kernels(lambda: razer.razer_linear(w, aq, out=out))
    finally:
        razer.razer_tune_force(binding.TUNE_GEMM_SLICES, None)
    assert any(kernel in x for x in names), names
    rows, cols = np.unique(np.r_[0, rng.choice(m, size=6, replace=False), 255, 256, m - 1]), np.unique(np.r_[0:40, 120:136, n - 140:n, rng.choice(n, size=60, replace=False)])
    y64, _ = oracle.linear((wq[0][cols], wq[1][cols], wq[2]), a_q=(aq.codes.cpu().numpy()[rows], aq.scales.cpu().numpy()[rows], np.float32(aq.tensor_scale.item())))
    assert max_rel_err(dev_to_bf16_bits(out)[rows][:, cols], y64) <= TOL
