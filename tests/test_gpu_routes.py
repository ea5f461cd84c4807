"""The branches that sizes and widths choose between, at their edges, against
the CPU oracle:

* the decode path around 24 tokens, where buckets of more than 2 tokens begin
  to take the grouped GEMMs and the many-token router replaces the small one;
* the prefill path around 16 tokens, where the tile lists' launch begins to
  build the buckets;
* the buckets built by one workgroup with the tile lists, at the edges of its
  64-token chunks, of the LDS it may use, of its 16-bit counts and of the sizes
  it is the faster at, and a forward above 65535 tokens;
* the grouped GEMMs at the edges of their 32-token tiles, for every width in the
  register decoder, rows of an odd number of 128-weight units, and lists of
  64- and 128-token tiles;
* the matrix-vector kernels at odd numbers of 128-weight units per row, with 8
  tokens staged per pass (up to 13 units) and with fewer;
* one token whose routing is a launch of its own (regrouped or more than 256
  experts), which the gate/up takes in 16 rows per workgroup;
* one and two tokens with a 5/6/8-bit shared down tensor, with one shared expert
  (the down kernel ends the forward) and two (a combine follows).

Tolerance of y: 2e-3 per token, normwise (h and, in the grouped GEMMs, the
weights are rounded once to 11 significant bits; measured about 2e-4)."""
import dataclasses

import numpy as np
import pytest
import torch

import layers
from inputs import synth
from oracle import bucket as obucket
from oracle import moe, router

pytestmark = pytest.mark.gpu

TOL = 2e-3


def _dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return t if dtype is None else t.view(dtype)


def _check(moeq, data, L, n, key, logits, path):
    s = data.shape
    x_bits = synth.activations(n, s.hidden, key, n)
    L.set_path(path)
    y = L.forward(_dev(x_bits.view(np.int16), torch.bfloat16), _dev(logits))
    torch.cuda.synchronize()
    idx, w = router.route(logits, data.mask, n_group=s.n_group, topk_group=s.topk_group, top_k=s.top_k,
                          group_topn=s.group_topn, norm_topk=s.norm_topk, routed_scale=s.routed_scale,
                          regroup=bool(s.regroup))
    err = moe.token_errors(y.cpu().numpy(), layers.oracle_forward(data, x_bits, idx, w))
    assert err.max() <= TOL, (n, err.max(), int(err.argmax()))
    return idx


def _layer(moeq, shape, plan, key, max_tokens):
    data = layers.quantized_layer(shape, plan, key)
    return data, moeq.Layer(shape, data.mask, data.routed(), data.shared(), max_tokens=max_tokens)


@pytest.mark.parametrize("plan", ["all4", "p234_602020", "wide_all"])
def test_few_tokens_around_switches(gpu_lib, plan):
    data, L = _layer(gpu_lib, synth.TINY, plan, f"routes-16-{plan}", 25)
    for n in (15, 16, 17, 23, 24, 25):
        logits = synth.normal_logits(n, data.shape.n_experts, "routes-16", n)
        idx = _check(gpu_lib, data, L, n, "routes-16", logits, gpu_lib.MOEQ_PATH_DECODE)
        sizes = np.bincount(idx.ravel())
        assert (sizes[sizes > 0] <= 2).any() and (sizes > 2).any()
        _check(gpu_lib, data, L, n, "routes-16", logits, gpu_lib.MOEQ_PATH_PREFILL)
    L.close()


@pytest.mark.parametrize("E,k,sizes", [(16, 2, (15, 16, 63, 64, 65, 128, 129)), (256, 8, (16, 64, 65, 2559, 2561)),
                                       (1024, 4, (17, 576, 577)), (8, 2, (65535, 65536)),
                                       (8, 8, (2730, 2731, 70001)), (1, 1, (65535, 65537)),
                                       (64, 32, (303, 304))])
def test_bucket_one_workgroup(gpu_lib, E, k, sizes):
    shape = synth.LayerShape(hidden=128, inter=128, n_experts=E, n_kept=E, n_shared=0, n_group=1, topk_group=1, top_k=k,
                             group_topn=min(2, E))
    one = layers.quantized_layer(shape, "all2", "routes-bucket")
    t = one.tensor("r", 0, 0), one.tensor("r", 0, 1), one.tensor("r", 0, 2)
    L = gpu_lib.Layer(shape, np.ones(E, np.uint8), {e: t for e in range(E)}, [], max_tokens=max(sizes))
    L.set_path(gpu_lib.MOEQ_PATH_PREFILL)
    r = np.random.default_rng(E)
    for n in sizes:
        # skewed: low ids often, some experts never
        idx = np.argsort(r.gumbel(size=(n, E)) - 1.5 * np.log1p(np.arange(E)), axis=1)[:, -k:].astype(np.int32)
        off, perm = L.bucket(_dev(idx))
        torch.cuda.synchronize()
        roff, rperm, _ = obucket.bucket(idx, E)
        assert np.array_equal(off.cpu().numpy(), roff) and np.array_equal(perm.cpu().numpy(), rperm), n
    L.close()


def test_forward_above_16_bit_counts(gpu_lib):
    """70001 tokens that all take all 8 experts: every expert's count is past
    65535.  The oracle checks tokens spread over the batch and its ends."""
    shape = synth.LayerShape(hidden=128, inter=128, n_experts=8, n_kept=8, n_shared=1, n_group=1, topk_group=1, top_k=8)
    n = 70001
    data, L = _layer(gpu_lib, shape, "p234_602020", "routes-70001", n)
    x_bits = synth.activations(n, shape.hidden, "routes-70001")
    logits = synth.normal_logits(n, 8, "routes-70001")
    y = L.forward(_dev(x_bits.view(np.int16), torch.bfloat16), _dev(logits))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(0, n, 997), np.arange(65530, 65545), np.arange(n - 4, n)]))
    idx, w = router.route(logits[rows], data.mask, n_group=1, topk_group=1, top_k=8, group_topn=shape.group_topn,
                          norm_topk=shape.norm_topk, routed_scale=shape.routed_scale)
    err = moe.token_errors(y.cpu().numpy()[rows], layers.oracle_forward(data, x_bits[rows], idx, w))
    assert err.max() <= TOL, err.max()
    L.close()


@pytest.mark.parametrize("plan", ["p234_602020", "all5", "all6", "all8", "wide_all"])
def test_gemm_tile_edges_odd_units(gpu_lib, plan):
    """Three and five units per row; every token takes the same two of four
    experts, so their buckets (and the shared expert's) hold n tokens."""
    shape = synth.LayerShape(hidden=384, inter=640, n_experts=4, n_kept=4, n_shared=1, n_group=1, topk_group=1, top_k=2)
    data, L = _layer(gpu_lib, shape, plan, f"routes-odd-{plan}", 129)
    # the reported weight bytes are the canonical packing's, whatever the layout pads
    canonical = sum(t["codes"].nbytes + t["scales"].nbytes for tr in [*data.routed().values(), *data.shared()] for t in tr)
    assert L.bytes()[0] == canonical
    for n in (1, 31, 32, 33, 64, 65, 96, 97, 128, 129):
        logits = synth.normal_logits(n, 4, "routes-odd", n)
        logits[:, [1, 2]] += 20.0
        _check(gpu_lib, data, L, n, "routes-odd", logits, gpu_lib.MOEQ_PATH_PREFILL)
    L.close()


@pytest.mark.parametrize("plan", ["p234_602020", "wide_all"])
def test_gemm_128_token_tiles(gpu_lib, plan):
    """Buckets larger than 64 tokens on average that fill the chip: 128-token
    tiles, with remainders of every token-tile count."""
    shape = synth.LayerShape(hidden=256, inter=1024, n_experts=8, n_kept=8, n_shared=1, n_group=1, topk_group=1, top_k=2)
    data, L = _layer(gpu_lib, shape, plan, f"routes-128-{plan}", 5600)
    logits = synth.normal_logits(5600, 8, "routes-128")
    idx = _check(gpu_lib, data, L, 5600, "routes-128", logits, gpu_lib.MOEQ_PATH_PREFILL)
    assert 5600 * 2 > 64 * 8 and 5600 * 3 // 128 * 8 >= 1024   # (the rule's own two conditions)
    assert len(np.unique(np.ceil(np.bincount(idx.ravel()) % 128 / 32))) > 1
    L.close()


@pytest.mark.parametrize("n_shared", [1, 2])
@pytest.mark.parametrize("bits", [5, 6, 8])
def test_decode_wide_shared_down(gpu_lib, n_shared, bits):
    shape = dataclasses.replace(synth.TINY, n_shared=n_shared)
    data, L = _layer(gpu_lib, shape, f"gu3_d4_sh{bits}", f"routes-sh{bits}-{n_shared}", 2)
    for n in (1, 2):
        logits = synth.normal_logits(n, shape.n_experts, "routes-sh", n)
        _check(gpu_lib, data, L, n, "routes-sh", logits, gpu_lib.MOEQ_PATH_AUTO)
    L.close()


@pytest.mark.parametrize("plan", ["p234_602020", "wide_all"])
@pytest.mark.parametrize("shape", [
    synth.LayerShape(hidden=384, inter=640, n_experts=16, n_kept=12, n_shared=1, n_group=4, topk_group=2, top_k=3,
                     regroup=1),
    synth.LayerShape(hidden=128, inter=384, n_experts=320, n_kept=240, n_shared=2, n_group=8, topk_group=4, top_k=6)],
    ids=["regroup", "320_experts"])
def test_one_token_routed_apart(gpu_lib, shape, plan):
    data, L = _layer(gpu_lib, shape, plan, f"routes-apart-{shape.n_experts}", 2)
    for n in (1, 2):
        logits = synth.normal_logits(n, shape.n_experts, "routes-apart", n)
        _check(gpu_lib, data, L, n, "routes-apart", logits, gpu_lib.MOEQ_PATH_DECODE)
    L.close()


@pytest.mark.parametrize("hu,iu,plan", [(3, 5, "p234_602020"), (3, 5, "wide_all"), (5, 11, "wide_all"),
                                        (11, 3, "p234_602020"), (11, 3, "wide_all"), (13, 9, "p234_602020"),
                                        (14, 13, "p234_602020"), (9, 14, "p234_602020")])
def test_decode_odd_units(gpu_lib, hu, iu, plan):
    """hu / iu units of 128 weights per gate/up / down row."""
    shape = synth.LayerShape(hidden=128 * hu, inter=128 * iu, n_experts=8, n_kept=6, n_shared=1, n_group=2,
                             topk_group=1, top_k=2)
    data, L = _layer(gpu_lib, shape, plan, f"routes-units-{hu}-{iu}-{plan}", 12)
    for n in (1, 2, 4, 5, 6, 12):
        logits = synth.normal_logits(n, 8, "routes-units", n)
        _check(gpu_lib, data, L, n, "routes-units", logits, gpu_lib.MOEQ_PATH_DECODE)
    L.close()


@pytest.mark.parametrize("iu", [13, 14])
def test_decode_many_buckets(gpu_lib, iu):
    """More than 2048 gate/up workgroups: 12 tokens over 40 experts make buckets
    of one token on average, 21 tokens of two and more."""
    shape = synth.LayerShape(hidden=128, inter=128 * iu, n_experts=48, n_kept=40, n_shared=1, n_group=1, topk_group=1,
                             top_k=4)
    data, L = _layer(gpu_lib, shape, "p234_602020", f"routes-many-{iu}", 21)
    for n in (12, 21):
        logits = synth.normal_logits(n, 48, "routes-many", n)
        idx = _check(gpu_lib, data, L, n, "routes-many", logits, gpu_lib.MOEQ_PATH_DECODE)
        assert (np.bincount(idx.ravel()) == 1).any() and iu * 4 * 41 > 2048
    L.close()
