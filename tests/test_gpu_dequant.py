"""The stand-alone dequantiser against the oracle, bit for bit, where its two kernels and their runs of eight symbols meet:
sizes around whole runs, channels shorter than, equal to and not a multiple of a run, symbols on any byte."""
import numpy as np
import pytest
import torch

from paper_2406_06237_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("channel_len", [0, 1, 3, 7, 8, 9, 64, 1000])
def test_runs_and_channels(orc, channel_len, dtype):
    rng = np.random.default_rng(channel_len)
    q = rng.integers(0, 256, 4200).astype(np.uint8)
    scales = rng.uniform(-0.1, 0.1, 4200).astype(np.float32)
    qd, sd = torch.from_numpy(q).cuda(), torch.from_numpy(scales).cuda()
    for n in (1, 7, 8, 9, 15, 16, 2047, 2048, 2049, 4100):
        for first in (0, 1, 8, 16):                       # multiples of sixteen take the runs (but for channels of one symbol), the others one symbol at a time
            want = orc.dequant(q[first:first + n], 100, 0.0173, dtype, channel_len, scales if channel_len else None)
            got = B.bits_of(B.dequant_zp(qd[first:first + n], 100, 0.0173, dtype, channel_len, sd if channel_len else None))
            assert np.array_equal(got, want.view(np.uint32) if dtype == "f32" else want), (n, first)


def test_channels_without_a_scale_are_zero():
    q = torch.full((4096,), 9, dtype=torch.uint8, device="cuda:0")
    scales = torch.ones(3, device="cuda:0")
    for first in (0, 1):
        got = B.dequant_zp(q[first:first + 4000], 7, 0.0, "f32", 1001, scales)
        assert torch.equal(got, torch.where(torch.arange(4000, device="cuda:0") < 3003, 2.0, 0.0))
