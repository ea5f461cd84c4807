"""The stage diagnostics run the kernels the forward runs: the names of the
kernels that moeq_route and moeq_bucket launch are among the forward's, on
every path and around every size at which the forward changes kernels (16 and
24 tokens, the decode path's limit, and the largest call one workgroup buckets).
So a stage test of a size covers what a forward of that size executes."""
import numpy as np
import pytest
import torch

import layers
from inputs import synth

pytestmark = pytest.mark.gpu


def _kernels(fn):
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        fn()
        torch.cuda.synchronize()
    # (demangled or not: the name with its template arguments identifies the kernel)
    return {e.name for e in prof.events() if "moeq" in e.name}


@pytest.fixture(scope="module")
def layer(gpu_lib):
    shape = synth.LayerShape(hidden=128, inter=128, n_experts=16, n_kept=16, n_shared=1, n_group=1, topk_group=1,
                             top_k=8)
    data = layers.quantized_layer(shape, "all4", "stage-kernels")
    L = gpu_lib.Layer(shape, data.mask, data.routed(), data.shared(), max_tokens=2800)
    yield shape, L
    L.close()


@pytest.mark.parametrize("path", [0, 1, 2])
@pytest.mark.parametrize("n", [2, 15, 16, 23, 24, 64, 65, 2730, 2731])
def test_stage_kernels_are_the_forwards(layer, n, path):
    shape, L = layer
    L.set_path(path)
    x = torch.from_numpy(synth.activations(n, shape.hidden, "stage-kernels", n).view(np.int16)).cuda()
    x = x.view(torch.bfloat16)
    logits = torch.from_numpy(synth.normal_logits(n, shape.n_experts, "stage-kernels", n)).cuda()
    idx, _ = L.route(logits)
    forward = _kernels(lambda: L.forward(x, logits))
    route, bucket = _kernels(lambda: L.route(logits)), _kernels(lambda: L.bucket(idx))
    L.set_path(0)
    assert forward and route and bucket
    assert any("route" in k for k in route)
    assert route <= forward, route - forward
    assert bucket <= forward, bucket - forward
