"""The streaming kernel's blocks of steps: windows that use all their bits, runs of steps of every length between two
scales, workgroups of few and of many chunks.  Expected values are the symbols themselves (whole numbers, or one product
of an integer and the scale rounded once), so every comparison is exact."""
import numpy as np
import pytest
import torch

from paper_2406_06237_amd import binding as B

pytestmark = pytest.mark.gpu


def _symbols(n, rng, bursts):
    """Sixteen common symbols, each at least 100 of 4096 states, and 200 rare ones of one state each, which read twelve
    bits: none scattered, but `bursts` runs of 40 in a row in one stream (of 64), next to nothing elsewhere."""
    s = rng.integers(0, 16, size=n).astype(np.uint8)
    for b in range(bursts):
        steps = n // 64
        first, lane = int(rng.integers(0, max(1, steps - 40))), int(rng.integers(0, 64))
        at = (first + np.arange(min(40, steps))) * 64 + lane
        s[at] = 16 + rng.integers(0, 200, size=len(at))
    return s


def _check(layers, table_log, chunk, dtype, channel_lens):
    rng = np.random.default_rng(9)
    n = len(layers)
    scales = [None if not c else (0.005 + 0.04 * rng.random(-(-len(l) // c))).astype(np.float32) for l, c in zip(layers, channel_lens)]
    host = B.pack_layers(layers, table_log, 64, chunk, [8] * n, [0.0125] * n, [8] * n, channel_lens, scales, dtype)
    d = B.to_device(host)
    out = B.alloc_out(d)
    out.view(torch.uint8).fill_(0xA5)
    B.decode(d, out=out, variant=B.VARIANT_STREAMING)
    assert d.read_status() == (0, 0)
    got, at = out[:host.numel].cpu(), 0
    for l, c, sc in zip(layers, channel_lens, scales):
        part = got[at:at + len(l)]
        at += len(l)
        if dtype == "u8":
            assert np.array_equal(part.numpy(), l)
            continue
        per = np.float32(0.0125) if sc is None else np.repeat(sc, c)[:len(l)]
        want = torch.from_numpy((l.astype(np.float32) - np.float32(8)) * per)
        assert torch.equal(part, want if dtype == "f32" else want.to(torch.bfloat16))


@pytest.mark.parametrize("dtype", ["u8", "f32", "bf16"])
@pytest.mark.parametrize("bursts", [0, 40])
def test_steps_of_twelve_bits(dtype, bursts):
    rng = np.random.default_rng(bursts + 1)
    layers = [_symbols(65536 + 777, rng, bursts) for _ in range(3)]
    _check(layers, 12, 16384, dtype, [0, 0, 0])


def test_eight_bits_every_step():
    # 256 symbols of one state each: two words per block of eight steps, more than the common fetch ahead
    rng = np.random.default_rng(4)
    _check([np.tile(rng.permutation(256).astype(np.uint8), 700) for _ in range(2)], 8, 32768, "u8", [0, 0])


@pytest.mark.parametrize("channel_len", [64, 128, 192, 320, 448, 576, 832, 4096 + 64, 96])
def test_runs_of_every_length_between_scales(channel_len):
    # 1, 2, 3, 5, 7, 9, 13, 65 steps a channel, more than 64 channels a chunk for the short ones; 96: not whole steps
    rng = np.random.default_rng(channel_len)
    _check([_symbols(100 * 1024 + 64 * 3 + 5, rng, 10), _symbols(40 * 1024, rng, 0)], 12, 40 * 1024, "bf16", [channel_len, channel_len])


@pytest.mark.parametrize("n_chunks", [1, 255, 257, 8 * 256, 9 * 256 + 3, 15 * 256])
def test_few_and_many_chunks_per_workgroup(n_chunks):
    rng = np.random.default_rng(n_chunks)
    _check([_symbols(n_chunks * 1024 - 33, rng, 5)], 11, 1024, "bf16", [0])


def test_the_shortest_chunks():
    rng = np.random.default_rng(8)
    for n in (64, 65, 127, 128, 64 * 4, 64 * 7 + 1, 64 * 9, 64 * 13 + 63):
        _check([rng.integers(0, 16, size=n).astype(np.uint8)], 10, 1024, "f32", [0])
