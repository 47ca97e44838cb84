"""GPU: the native entry points of the binding refuse what its Python path refuses, with the same message,
and take what it takes, with the same results."""
import pytest
import torch

import paper_2602_09323_amd as coopt
from paper_2602_09323_amd import binding

pytestmark = pytest.mark.gpu

S, HQ, HK, D, NB, WIDTH = 2, 8, 2, 64, 12, 4


def _state(kv):
    g = torch.Generator(device="cuda").manual_seed(5)
    shape = coopt.Shape(S, HQ, HK, D, 16, NB, WIDTH, kv, 0.125)
    code = 2 if kv == coopt.COOPT_KV_FP16 else 1
    rows = 37 + 20
    a = {"k": torch.randn(rows, HK, D, device="cuda", generator=g).half(),
         "v": torch.randn(rows, HK, D, device="cuda", generator=g).half(),
         "slots": torch.cat([torch.arange(0, 37), torch.arange(64, 84)]).cuda(),
         "kc": torch.zeros(NB, HK, 16 * D * code, dtype=torch.uint8, device="cuda"),
         "vc": torch.zeros(NB, HK, 16 * D * code, dtype=torch.uint8, device="cuda"),
         "ks": torch.zeros(NB, HK, 16, device="cuda") if code == 1 else None,
         "vs": torch.zeros(NB, HK, 16, device="cuda") if code == 1 else None,
         "q": torch.randn(S, HQ, D, device="cuda", generator=g).half(),
         "bt": torch.tensor([[0, 1, 2, -1], [4, 5, -1, -1]], dtype=torch.int32, device="cuda"),
         "cl": torch.tensor([37, 20], dtype=torch.int32, device="cuda"),
         "out": torch.empty(S, HQ, D, dtype=torch.float16, device="cuda"),
         "ws": torch.empty(coopt.decode_workspace_bytes(shape), dtype=torch.uint8, device="cuda"),
         "sched": torch.empty(coopt.decode_schedule_bytes(shape), dtype=torch.uint8, device="cuda"),
         "tmp": torch.empty(S, HQ, 4, D, device="cuda"), "mx": torch.empty(S, HQ, 4, device="cuda"),
         "sm": torch.empty(S, HQ, 4, device="cuda"),
         "starts": torch.tensor([0, 1, 2], dtype=torch.int32, device="cuda"),
         "pws": torch.empty(coopt.prefill_workspace_bytes(shape, 1), dtype=torch.uint8, device="cuda"),
         "ko": torch.empty(9, HK, D, dtype=torch.float16, device="cuda"),
         "vo": torch.empty(9, HK, D, dtype=torch.float16, device="cuda")}
    a["new"], a["newslots"] = a["k"][:S], torch.tensor([36, 83], device="cuda")
    return a, shape


def _calls(kv):
    write = ("kv_cache_write_fp16", "k v slots kc vc") if kv == coopt.COOPT_KV_FP16 else \
        ("kv_cache_write_fp8", "k v slots kc vc ks vs")
    return [write,
            ("paged_gqa_decode", "q kc vc ks vs bt cl out ws"),
            ("paged_gqa_decode_step", "new new newslots q kc vc ks vs bt cl out ws"),
            ("decode_schedule_prepare", "bt cl newslots sched"),
            ("paged_gqa_decode_scheduled", "new new newslots q kc vc ks vs cl out ws sched"),
            ("paged_gqa_decode_partitioned", "q kc vc ks vs bt cl 16 tmp mx sm 4"),
            ("paged_gqa_reduce", "tmp mx sm cl 16 4 out"),
            ("paged_gqa_prefill_chunk_ws", "q kc vc ks vs bt cl starts 2 1 out pws"),
            ("gather_cached_kv", "kc vc ks vs bt 0 3 12 ko vo")]


def _args(names, a):
    return [int(n) if n.isdigit() else a[n] for n in names.split()]


@pytest.mark.parametrize("kv", [coopt.COOPT_KV_E4M3, coopt.COOPT_KV_FP16], ids=["e4m3", "fp16"])
def test_native_and_python_path_agree(kv, monkeypatch):
    coopt.load_library()
    assert binding._fast() is not None, "the native part is not built"
    results = []
    for native in (binding._fast(), False):
        monkeypatch.setattr(binding, "_native", native)
        a, shape = _state(kv)
        got = []
        for name, names in _calls(kv):
            getattr(coopt, name)(*_args(names, a), shape)
            got += [t.clone() for n, t in sorted(a.items())
                    if n in ("kc", "vc", "ks", "vs", "out", "ko", "vo") and t is not None and n in names.split()]
        torch.cuda.synchronize()
        results.append(got)
    assert len(results[0]) == len(results[1])
    for x, y in zip(*results):
        assert torch.equal(x, y)


@pytest.mark.parametrize("kv", [coopt.COOPT_KV_E4M3, coopt.COOPT_KV_FP16], ids=["e4m3", "fp16"])
def test_both_refuse_the_same(kv, monkeypatch):
    """Every tensor argument in turn missing, on the host, strided, of another type, too small; each is
    refused before anything is launched."""
    coopt.load_library()
    native, refused = binding._fast(), 0
    a, shape = _state(kv)
    for name, names in _calls(kv):
        args = _args(names, a)
        for i, t in enumerate(args):
            if not isinstance(t, torch.Tensor):
                continue
            wide = torch.stack([t, t], dim=-1)[..., 0]
            other = t.double() if t.dtype != torch.uint8 else t[:1]
            for bad in (None, t.cpu(), wide, other, t.flatten()[:1]):
                if isinstance(bad, torch.Tensor) and bad.is_cuda and bad.is_contiguous() and bad.numel() >= t.numel() \
                        and bad.dtype == t.dtype:
                    continue
                said = []
                for path in (native, False):
                    monkeypatch.setattr(binding, "_native", path)
                    try:
                        getattr(coopt, name)(*args[:i], bad, *args[i + 1:], shape)
                        said.append("taken")
                    except Exception as e:  # noqa: BLE001
                        said.append(f"{type(e).__name__}: {e}")
                torch.cuda.synchronize()
                assert said[0] == said[1], (name, i, said)
                refused += said[0] != "taken"
    assert refused > 100
