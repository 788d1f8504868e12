"""What the benchmark says of a 16-bit layer is what it timed: the path, the kernel, and an accuracy taken from the timed call's
own output, on a layer of each path."""
import argparse

import pytest

import bench
import dwm_workloads as wl
import paper_2002_00552_amd as dwm

pytestmark = pytest.mark.gpu

LAYERS = [  # layer, forward variant, path, stages
    (wl.Layer("many", 2, 32, 12, 12, 40, 3, 3, 1, 1, "uniform"), -1, "single kernel for many channels", ["wide16_forward"]),
    (wl.Layer("many_staged", 2, 32, 12, 12, 40, 3, 3, 1, 1, "uniform"), 0, "staged", ["input_transform", "contract_output"]),
    (wl.Layer("few", 2, 3, 32, 32, 20, 5, 5, 1, 2, "uniform"), -1, "single kernel", ["fused16_forward"]),
    # rows of 64 tiles from many small images: more than LDS holds
    (wl.Layer("declined", 64, 32, 9, 9, 32, 3, 3, 2, 0, "uniform"), -1, "staged", ["input_transform", "contract_output"]),
]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("layer,forward,path,stages", LAYERS)
def test_path_stages_and_checked_output(layer, forward, path, stages, bf16, monkeypatch):
    x, w = wl.make_layer_tensors(layer, 5)
    args = argparse.Namespace(steps=2, warmup=1, contract_variant=-1, forward_variant=forward, no_check=False)
    calls = []
    for name in ("conv_forward", "contract_output"):
        full = "dwm_%s_%s" % ("bf16" if bf16 else "f16", name)
        real = getattr(dwm, full)
        monkeypatch.setattr(dwm, full, lambda *a, real=real, name=name: (calls.append(name), real(*a))[1])
    out = bench.bench_half(args, layer, x, w, bf16=bf16)
    assert out["config"]["path"] == path and list(out["stages"]) == stages
    assert (out["roofline"]["kernel"] == "wide16_kernel") == (stages == ["wide16_forward"])
    assert calls[-1] == "conv_forward"  # the last to write y before it is compared
    assert out["accuracy"]["max_rel_err"] < (3e-2 if bf16 else 4e-3)
