"""Which devices the binding's device entry points accept, with the library stubbed (nothing is launched): a tensor or a
device that is no GPU is refused before the library is called, since a kernel would dereference its host pointer."""
import pytest
import torch

from paper_2406_06237_amd import binding as B


@pytest.fixture
def calls(monkeypatch):
    """Names of the library's device functions that were called; GPU 0 is there and current."""
    seen, real = [], B.lib()

    class Stub:
        def __getattr__(self, name):
            if name in ("anszp_pack_bound", "anszp_plan_bytes"):      # host only
                return getattr(real, name)
            return lambda *args: seen.append(name) or 0

    stub = Stub()
    monkeypatch.setattr(B, "lib", lambda: stub)
    monkeypatch.setattr(B, "_torch_with_gpu", torch)
    monkeypatch.setattr(B, "_index_of_name", {})
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 0, raising=False)
    return seen



@pytest.mark.parametrize("device", ["cpu", "cpu:0", "meta", torch.device("cpu"), torch.device("cpu", 0)])
@pytest.mark.parametrize("call", [
    lambda dev: B.decode_raw(B.DecodeArgs(), dev), lambda dev: B.decode_raw(B.DecodeArgs(), dev, B.VARIANT_MERGED),
    lambda dev: B.plan_decode(B.DecodeArgs(), dev), lambda dev: B.decode_planned_raw(B.DecodeArgs(), torch.zeros(16), dev),
    lambda dev: B.decode_static_plan_raw(B.DecodeArgs(), True, dev), lambda dev: B.conv_fused_raw(B.ConvArgs(), dev),
    lambda dev: B.build_tables([[4096] + [0] * 255], 12, dev),
    lambda dev: B.build_tables_device(torch.zeros(256, dtype=torch.int32, device=dev), 12),
    lambda dev: B.dequant_zp(torch.zeros(64, dtype=torch.uint8, device=dev), 8, 0.5),
    lambda dev: B.pack_layer_device(torch.zeros(64, dtype=torch.uint8, device=dev), torch.zeros(256, dtype=torch.int32, device=dev), 12, 64, 64),
    lambda dev: B.pack_layers_device(torch.zeros(64, dtype=torch.uint8, device=dev), [64], torch.zeros(256, dtype=torch.int32, device=dev), 12, 64, 64),
], ids=["decode", "decode_variant", "plan_decode", "decode_planned", "decode_static_plan", "conv_fused", "build_tables",
        "build_tables_device", "dequant_zp", "pack_layer_device", "pack_layers_device"])
def test_no_host_memory_reaches_a_kernel(calls, call, device):
    for _ in range(2):                                    # (a refusal is not remembered as an index)
        with pytest.raises(ValueError, match="cuda device"):
            call(device)
    assert calls == []


@pytest.mark.parametrize("device", [0, None, "cuda", "cuda:0", torch.device("cuda"), torch.device("cuda", 0)])
def test_every_name_of_a_gpu_is_accepted(calls, device):
    for _ in range(2):
        B.decode_raw(B.DecodeArgs(), device)
    assert calls == ["anszp_decode"] * 2


def test_a_set_is_not_packed_under_capture(calls, monkeypatch):
    """The jobs come from pinned memory that is free again when the call returns: a graph would copy whatever lies there later."""
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    monkeypatch.setattr(B, "_device_index", lambda torch, device: 0)
    with pytest.raises(RuntimeError, match="captur"):
        B.pack_layers_device(torch.zeros(64, dtype=torch.uint8), [64], torch.zeros(256, dtype=torch.int32), 12, 64, 64)
    assert calls == []
