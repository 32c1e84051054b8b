"""GPU: the binding's native calls (csrc/anszp_torch.cpp) and the path they leave to Python give the same results and the same
errors: integers of other types, sizes given one by one, payload limits, empty inputs."""
import numpy as np
import pytest
import torch

from paper_2406_06237_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture
def without(monkeypatch):
    """Runs a call with the native functions declining."""
    def run(call):
        with monkeypatch.context() as m:
            m.setattr(B, "_call", lambda *args: None)
            return call()
    return run


def _inputs(sizes, seed=1):
    rng = np.random.default_rng(seed)
    sym = [rng.choice(6, n, p=[0.5, 0.2, 0.1, 0.1, 0.05, 0.05]).astype(np.uint8) for n in sizes]
    freqs = np.stack([B.normalize_freqs(np.bincount(np.concatenate([s, np.arange(6)]), minlength=256), 10) for s in sym])
    return torch.from_numpy(np.concatenate(sym)).to("cuda:0"), torch.from_numpy(freqs.astype(np.int32)).to("cuda:0")


def _same(a, b):
    torch.cuda.synchronize()
    assert len(a) == len(b)
    for x, y in zip(a, b):
        assert x.dtype == y.dtype and x.shape == y.shape and torch.equal(x, y)


@pytest.mark.parametrize("sizes,chunk", [([5000], 700), ([1, 4097, 300], 512), ([3000, 0, 50], [100, 7, 64]), (np.array([900, 31]), np.int64(64)), ((64, 64), [16, 32, 99])])
def test_sets(without, sizes, chunk):
    sym, freqs = _inputs(sizes)
    call = lambda: B.pack_layers_device(sym, sizes, freqs, 10, 32, chunk)
    _same(call(), without(call))
    plain = lambda: B.pack_layers_device(sym, [int(n) for n in sizes], freqs, 10, 32, chunk if np.isscalar(chunk) else list(chunk))
    _same(call(), plain())


@pytest.mark.parametrize("n", [0, 1, 1000])
def test_a_layer(without, n):
    sym, freqs = _inputs([max(n, 1)])
    sym = sym[:n]
    for kw in ({}, {"layer_id": 3, "out_offset": 40, "payload_word_offset": 8, "stream_offset": 96}, {"payload_cap_words": 17}, {"layer_id": np.int64(2)}):
        call = lambda: B.pack_layer_device(sym, freqs, 10, 16, 128, **kw)
        _same(call(), without(call))


def test_what_is_refused_is_refused(without):
    sym, freqs = _inputs([1000])
    for call, error in ((lambda: B.pack_layers_device(sym, [-1], freqs, 10, 32, 64), OverflowError), (lambda: B.pack_layers_device(sym, [1000], freqs, 10, 32, 0), ZeroDivisionError),
                        (lambda: B.pack_layer_device(sym, freqs, 13, 32, 64), B.AnszpError), (lambda: B.pack_layer_device(sym, freqs, 10, 65, 64), B.AnszpError),
                        (lambda: B.pack_layer_device(sym, freqs, 10, 32, 64, payload_word_offset=2), B.AnszpError), (lambda: B.build_tables_device(freqs, 13), B.AnszpError),
                        (lambda: B.dequant_zp(sym, -1, 0.5), OverflowError), (lambda: B.dequant_zp(sym, 8, 0.5, "u8"), B.AnszpError), (lambda: B.dequant_zp(sym, 8, 0.5, "f16"), KeyError)):
        with pytest.raises(error):
            call()
        with pytest.raises(error):
            without(call)


@pytest.mark.parametrize("n", [0, 1, 7, 8, 9, 5000])
def test_dequantised(without, n):
    sym, _ = _inputs([max(n, 1)])
    sym = sym[:n]
    scales = 0.01 + torch.rand(max(1, -(-n // 7)), device="cuda:0")
    for call in (lambda: B.dequant_zp(sym, 3, 0.25), lambda: B.dequant_zp(sym, 3, np.float32(0.3), "f32"), lambda: B.dequant_zp(sym, 2, 0.5, "f32", 7, scales)):
        _same((call(),), (without(call),))


def test_tables_and_their_status(without):
    _, freqs = _inputs([1000, 2000])
    freqs[1, 0] += 1
    for st in (None, torch.zeros(2, dtype=torch.int32, device="cuda:0")):
        call = lambda: B.build_tables_device(freqs, 10, st)
        _same((call(),), (without(call),))
        assert st is None or st.tolist() == [B.ST_BAD_FREQ, 2]


def test_threads_with_streams_of_their_own():
    import threading
    sizes = [[4000, 300], [70001], [512] * 20, [9, 5000, 31]]
    inputs = [_inputs(s, seed) for seed, s in enumerate(sizes)]
    pack = lambda k: B.pack_layers_device(inputs[k][0], sizes[k], inputs[k][1], 10, 32, 1000)
    expect = [(pack(k), B.dequant_zp(inputs[k][0], 2, 0.5)) for k in range(4)]
    torch.cuda.synchronize()
    wrong = []

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            got = [(pack(k), B.dequant_zp(inputs[k][0], 2, 0.5)) for _ in range(25)]
            torch.cuda.current_stream().synchronize()
        for packed, weights in got:
            if not (all(torch.equal(a, b) for a, b in zip(packed, expect[k][0])) and torch.equal(weights, expect[k][1])):
                wrong.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def test_without_the_module(monkeypatch):
    sym, freqs = _inputs([3000, 700])
    calls = (lambda: B.pack_layers_device(sym, [3000, 700], freqs, 10, 32, 512), lambda: B.pack_layer_device(sym, freqs[:1], 10, 32, 512),
             lambda: (B.dequant_zp(sym, 2, 0.5),), lambda: (B.build_tables_device(freqs, 10),))
    expect = [call() for call in calls]
    monkeypatch.setattr(B, "_host", False)                # (what a failed import leaves)
    for call, e in zip(calls, expect):
        _same(call(), e)
