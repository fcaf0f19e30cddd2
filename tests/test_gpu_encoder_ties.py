"""The encoder on data whose decisions are ties or near ties, and on scales far from the ordinary range: multiples of a
quarter of the scale (every rounding boundary, exact ties between candidates), those moved by one unit in the last
place, one huge element (all other blocks on coarse subnormal scales), given scales that saturate; more runs than the
launch has threads.  Codes, scales and the tensor scale must equal the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import paper_2501_04052_amd as razer

pytestmark = pytest.mark.gpu


def _quarters(rng, shape):
    x = rng.integers(-28, 29, size=shape).astype(np.float32) / 4
    x[:, ::16] = 6.0                                   # block maximum 6 at scale 1: the boundaries fall on multiples of 1/4
    return x


def _inputs(kind, rng, shape):
    if kind == "quarters":
        return _quarters(rng, shape), 1.0
    if kind == "quarters_ulp":
        x = _quarters(rng, shape) * np.float32(0.37)
        return np.nextafter(x, np.where(rng.random(shape) < 0.5, -1e9, 1e9).astype(np.float32)), 0.37
    if kind == "mirrored":                             # +v and -v in every block: the two signs of a candidate tie
        x = rng.standard_normal((shape[0], shape[1] // 2)).astype(np.float32)
        return np.stack([x, -x], axis=-1).reshape(shape).copy(), None
    if kind == "one_huge":
        x = rng.standard_normal(shape).astype(np.float32)
        x[0, 3] = 900.0
        return x, None
    return rng.standard_normal(shape).astype(np.float32), 1e-2     # "saturated": blocks far above the largest scale


@pytest.mark.parametrize("kind", ["quarters", "quarters_ulp", "mirrored", "one_huge", "saturated"])
@pytest.mark.parametrize("fmt,sv,block", [(razer.WEIGHT, (5.0, 8.0), 16), (razer.WEIGHT, (2.5, 7.5), 64), (razer.ACT, (5.0, 5.0), 16),
                                          (razer.ACT, (9.5, 9.5), 32), (razer.WEIGHT_F16, (5.0, 9.0), 128)])
def test_ties_and_far_scales(oracle, kind, fmt, sv, block):
    x, ts = _inputs(kind, np.random.default_rng(31), (96, 512))
    dev = None if ts is None else torch.tensor([ts], dtype=torch.float32, device="cuda")
    t = razer.razer_quantize(torch.from_numpy(x).cuda(), fmt, sv, tensor_scale=dev, block=block)
    codes, scales, rts = oracle.quantize(fmt, x, sv=sv, given_tensor_scale=ts, block=block)
    assert np.array_equal(t.codes.cpu().numpy(), codes)
    assert np.array_equal(t.scales.cpu().numpy().view(scales.dtype), scales)
    assert np.float32(t.tensor_scale.cpu().numpy()[0]) == rts


def test_more_runs_than_threads(oracle):
    x = np.random.default_rng(32).standard_normal((4096 + 33, 4096 + 32)).astype(np.float32)    # 4096 x 256 threads of 16 elements, and some
    t = razer.razer_quantize(torch.from_numpy(x).cuda(), razer.ACT, (5.0,))
    codes, scales, rts = oracle.quantize(razer.ACT, x, sv=(5.0, 5.0))
    assert np.array_equal(t.codes.cpu().numpy(), codes) and np.array_equal(t.scales.cpu().numpy(), scales)
    assert np.float32(t.tensor_scale.cpu().numpy()[0]) == rts


def _lattice(rng, shape, top):
    """Integers up to 64 under block maxima of `top`: elements scaled to multiples of 6 / top, so that the gains of two
    special values tie, exactly or up to the rounding of the quotients, in a good part of the blocks."""
    x = rng.integers(-64, 65, size=shape).astype(np.float32)
    x[:, ::16] = top
    return x


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fmt,sv,block", [(f, sv, b) for f, sv in [(razer.WEIGHT, (5.0, 8.0)), (razer.WEIGHT, (5.0, 5.0)), (razer.WEIGHT, (7.5, 2.5)),
                                                                    (razer.ACT, (5.0, 5.0))] for b in (16, 32, 64, 128)] +
                         [(razer.WEIGHT_F16, (5.0, 8.0), 128)])
def test_two_candidates_that_tie(oracle, dtype, fmt, sv, block):
    rng = np.random.default_rng(33 + block)
    x = _lattice(rng, (96, 1024), 64.0)
    xs = x / np.float32(64.0 / 6.0)
    gain = np.maximum((5.0 - np.floor(np.abs(xs))) * (2 * np.abs(xs) - np.floor(np.abs(xs)) - 5.0), 0.0) * (np.abs(xs) >= 4.5) * (np.abs(xs) < 5.0)
    side = [np.where(s * xs > 0, gain, 0.0).reshape(96, -1, block).sum(-1) for s in (1, -1)]
    assert np.count_nonzero((np.abs(side[0] - side[1]) < 1e-3) & (side[0] > 0)) >= 5        # (exact ties of +5 and -5 from below)
    for given in (None, 64.0 / 6.0, 64.0 / 6.0 * 2.0 ** -62):
        v = x * np.float32(2.0 ** -62) if given and given < 1e-9 else x
        dev = None if given is None else torch.tensor([given], dtype=torch.float32, device="cuda")
        t = razer.razer_quantize(torch.from_numpy(v).cuda().to(dtype), fmt, sv, tensor_scale=dev, block=block)
        codes, scales, rts = oracle.quantize(fmt, v, sv=sv, given_tensor_scale=None if given is None else np.float32(given), block=block)
        assert np.array_equal(t.codes.cpu().numpy(), codes), given
        assert np.array_equal(t.scales.cpu().numpy().view(scales.dtype), scales), given


@pytest.mark.parametrize("fmt,sv,block", [(razer.WEIGHT, (5.0, 8.0), 16), (razer.ACT, (9.5, 9.5), 64), (razer.WEIGHT_F16, (5.0, 9.0), 128)])
@pytest.mark.parametrize("clip", [8.0, 64.0, 511.0, 513.0, 4096.0])
def test_blocks_far_above_a_given_scale(oracle, fmt, sv, block, clip):
    """Block maxima of about `clip` times what the largest scale covers: below 512 the gains decide, above the fp64 sums."""
    grid = {razer.WEIGHT: 30.0, razer.ACT: 448.0, razer.WEIGHT_F16: 1.9990234375}[fmt]
    rng = np.random.default_rng(34)
    x = rng.standard_normal((64, 1024)).astype(np.float32)
    x[:, 5::block] = -clip * np.float32(grid)
    x[:, 6::2 * block] = clip * np.float32(grid)
    t = razer.razer_quantize(torch.from_numpy(x).cuda(), fmt, sv, tensor_scale=torch.tensor([1.0], device="cuda"), block=block)
    codes, scales, _ = oracle.quantize(fmt, x, sv=sv, given_tensor_scale=np.float32(1.0), block=block)
    assert np.array_equal(t.codes.cpu().numpy(), codes)
    assert np.array_equal(t.scales.cpu().numpy().view(scales.dtype), scales)


@pytest.mark.parametrize("dtype,rows", [(torch.float32, 65535), (torch.float32, 65536), (torch.float32, 65537), (torch.float32, 786433),
                                        (torch.bfloat16, 131073), (torch.bfloat16, 1572865), (torch.float32, 3), (torch.bfloat16, 40000), (torch.float32, 128001)])
def test_tensor_scale_sees_every_element(dtype, rows):
    """Eq. 1's maximum at the first and last element, around the end of the unrolled loads and at either side of each
    stride of what is left; below and above the size that is read around the caches."""
    cols = 32
    n = rows * cols
    x = torch.full((n,), 90.0, dtype=dtype, device="cuda")             # (a tensor scale of 0.5; of an all-zero tensor 1)
    stride = 256 * 256 * (16 // x.element_size())
    whole = n // (8 * stride) * 8 * stride
    for i in {0, n - 1, n // 2} | {min(max(whole + j * stride + d, 0), n - 1) for j in range(9) for d in (-1, 0)}:
        x[i] = -360.0
        t = razer.razer_quantize(x.view(rows, cols), razer.WEIGHT, (5.0, 8.0))
        assert float(t.tensor_scale) == 2.0, i
        x[i] = 90.0
