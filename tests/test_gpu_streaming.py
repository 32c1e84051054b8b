"""The streaming kernel's blocks of steps: windows that use all their bits, runs of steps of every length between two
scales, workgroups of few and of many chunks.  Expected values are the symbols themselves (whole numbers, or one product
of an integer and the scale rounded once), so every comparison is exact."""
import dataclasses

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
    # (256 CUs: one to nine or ten chunks in a workgroup, in one round; the last in two rounds of seven or eight)
    rng = np.random.default_rng(n_chunks)
    _check([_symbols(n_chunks * 1024 - 33, rng, 5)], 11, 1024, "bf16", [0])


def test_the_shortest_chunks():
    rng = np.random.default_rng(8)
    for n in (64, 65, 127, 128, 64 * 4, 64 * 7 + 1, 64 * 9, 64 * 13 + 63):
        _check([rng.integers(0, 16, size=n).astype(np.uint8)], 10, 1024, "f32", [0])


# The kernel has two forms: for at most twelve chunks per workgroup the next block's words are asked for ahead, for more
# they are read block by block.  Workgroups: as many as CUs, in rounds of at most fourteen chunks each.
def _most_chunks_of_a_workgroup(n_chunks):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    groups = min(n_chunks, cus * -(-n_chunks // (cus * 14)))
    return -(-n_chunks // groups)


def _many_chunks(per_group, dtype, channel_len, chunk=64 * 512, unique=29, last=64 * 300 + 17):
    """A layer of enough chunks for `per_group` chunks in the fullest workgroup: `unique` of them (streams of about 70
    words, more than two rings of 32, and one shorter chunk at the end) over and over, each at its own place."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n_chunks = cus * (per_group - 1) + 1
    assert _most_chunks_of_a_workgroup(n_chunks) == per_group
    rng = np.random.default_rng(per_group)
    symbols = _symbols(unique * chunk + last, rng, 60)
    numel = (n_chunks - 1) * chunk + last
    scales = None if not channel_len else (0.005 + 0.04 * rng.random(-(-numel // channel_len))).astype(np.float32)
    host = B.pack_layers([symbols], 12, 64, chunk, [8], [0.0125], [8], [channel_len], [scales], dtype)
    assert int(host.stream_hdr[:unique * 64].max() >> 16) > 64
    which = np.append(np.arange(n_chunks - 1) % unique, unique)
    chunks = host.chunks[which].copy()
    chunks["out_offset"] = np.arange(n_chunks, dtype=np.uint64) * chunk
    d = B.to_device(dataclasses.replace(host, chunks=chunks, numel=numel))
    s = torch.from_numpy(symbols).to("cuda:0")
    want = torch.cat([s[:unique * chunk].repeat(-(-(n_chunks - 1) // unique))[:(n_chunks - 1) * chunk], s[unique * chunk:]])
    if dtype != "u8":
        per = np.float32(0.0125) if scales is None else torch.from_numpy(scales).to("cuda:0").repeat_interleave(channel_len)[:numel]
        want = (want.float() - 8.0) * per
    return d, want if dtype != "bf16" else want.to(torch.bfloat16)


@pytest.mark.parametrize("per_group", [7, 8, 11, 12, 13, 14])
@pytest.mark.parametrize("dtype,channel_len", [("u8", 0), ("f32", 0), ("bf16", 0), ("bf16", 64 * 5), ("f32", 4096), ("bf16", 100)])
def test_both_forms_with_rings_that_wrap(per_group, dtype, channel_len):
    d, want = _many_chunks(per_group, dtype, channel_len)
    out = B.alloc_out(d)
    out.view(torch.uint8).fill_(0xA5)
    B.decode(d, out=out, variant=B.VARIANT_STREAMING)
    assert d.read_status() == (0, 0)
    assert torch.equal(out[:d.host.numel], want)


@pytest.mark.parametrize("per_group", [3, 13])
def test_a_wait_that_gives_up_drains_both_forms(per_group):
    """The bound of the waits lowered from the host: the launch reports it, ends, and writes nothing outside; with the
    default bound back the same container decodes."""
    d, want = _many_chunks(per_group, "bf16", 0)
    guard = 4096
    buf = torch.full((d.host.numel + 2 * guard,), 0x5A5A, dtype=torch.int16, device="cuda:0")
    out = buf[guard:guard + d.host.numel].view(torch.bfloat16)
    try:
        B.lib().anszp_test_set_spin_limit(1)
        B.decode(d, out=out, variant=B.VARIANT_STREAMING)
        torch.cuda.synchronize()
        st = d.read_status()
        assert st[0] & B.ST_INTERNAL and st[1] >= 1, st
        assert bool((buf[:guard] == 0x5A5A).all()) and bool((buf[guard + d.host.numel:] == 0x5A5A).all())
    finally:
        B.lib().anszp_test_set_spin_limit(0)
    d.status.zero_()
    B.decode(d, out=out, variant=B.VARIANT_STREAMING)
    assert d.read_status() == (0, 0) and torch.equal(out, want)
