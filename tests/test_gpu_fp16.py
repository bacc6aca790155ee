"""GPU parity of the binary16 path of swaa_attn_fwd_ex (the precision the paper serves its
models in, Sec. 4.1.1) against the fp64 CPU oracle reading the same binary16 inputs.  The
acceptance tolerances of the bfloat16 path apply (binary16 rounds three bits finer).
"""
import math

import numpy as np
import pytest
import torch

from oracle import input_format, swaa_attn_oracle, swaa_decode_oracle
from paper_2512_10411_amd import binding
from paper_2512_10411_amd.inputs import make_qkv, sample_rows
from gpu_util import assert_parity, forward_packed, to_device

pytestmark = pytest.mark.gpu

# (prompts of one length and few rows run on the short prompts' kernel, packed ones on row tiles)
on_both_kernels = pytest.mark.parametrize("packed", [False, True])


def run_gpu(q, k, v, W, S, scale, packed):
    if packed:
        return forward_packed(q, k, v, W, S, scale, fmt="fp16")
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, "fp16"), to_device(k, "fp16"), to_device(v, "fp16"), W, S, None, scale)
    torch.cuda.synchronize()
    return out, lse


def check(B, Hq, Hkv, Nq, Nk, D, W, S, P, seed, rows=None):
    tag = f"fp16 B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} D{D} W{W} S{S} P{P}"
    print(f"[case] {tag} seed {seed}", flush=True)
    scale = 1 / math.sqrt(D)
    q, k, v = make_qkv(B, Hq, Hkv, Nk, D, seed, n_query=None if Nq == Nk else Nq, fmt="fp16")
    out, lse = binding.swaa_attn_fwd_ex(to_device(q, "fp16"), to_device(k, "fp16"), to_device(v, "fp16"), W, S, P, scale)
    torch.cuda.synchronize()
    assert out.dtype == torch.float16
    with input_format("fp16"):
        if Nq == Nk:
            ro, rl = swaa_attn_oracle(q, k, v, W, S, scale, rows=rows, n_prompt=P)
        else:
            ro, rl = swaa_decode_oracle(q, k, v, W, S, scale, n_prompt=P)
    assert_parity(out, lse, ro, rl, rows=rows, tag=tag)


@pytest.mark.parametrize("D", [64, 96, 128, 256])
def test_small_shapes(D):
    for N in (1, 63, 65, 257, 700):
        for W, S, P in ((1, 0, None), (7, 4, None), (64, 70, None), (N, 0, None), (50, 3, N // 2)):
            check(1, 4, 1, N, N, D, W, S, P, seed=9600 + N + D)
    check(2, 10, 2, 333, 333, D, 100, 3, None, seed=9700 + D)   # GQA 5 = 4 + 1, two batch entries
    check(1, 4, 2, 100, 777, D, 64, 4, None, seed=9710 + D)     # a chunk of a longer prefill


@on_both_kernels
def test_sink_heavy_scores_keep_probabilities_in_range(packed):
    # scores tens of nats apart (k scaled by 4): later keys outgrow the reference taken from the
    # first half tile by more than binary16 holds in places, which must end in the max-based pass
    B, Hq, Hkv, N, D = 1, 4, 1, 2000, 128
    q, k, v = make_qkv(B, Hq, Hkv, N, D, seed=9720, k_mult=4.0, fmt="fp16")
    out, lse = run_gpu(q, k, v, 512, 4, 1 / math.sqrt(D), packed)
    with input_format("fp16"):
        ro, rl = swaa_attn_oracle(q, k, v, 512, 4, 1 / math.sqrt(D))
    assert_parity(out, lse, ro, rl, tag="fp16 peaked softmax")


@on_both_kernels
@pytest.mark.parametrize("spike", [0.0, 24.0, 40.0, 160.0])
def test_late_score_spike_against_the_binary16_range(spike, packed):
    # one key deep inside the windows scores 3 * spike / sqrt(D) nats above the rest: 6 nats stay
    # inside binary16 with the fixed reference (P up to 2^13), 10 nats and more overflow a P and
    # must be caught; a very negative key and small values ride along
    B, Hq, Hkv, N, D, W, S = 1, 4, 1, 3100, 128, 1024, 4
    q, k, v = make_qkv(B, Hq, Hkv, N, D, seed=9740, fmt="fp16")
    qf = q.view(np.float16).astype(np.float32)
    kf = k.view(np.float16).astype(np.float32)
    qf[..., 0] = 3.0
    kf[..., 0] = 0.0
    kf[:, :, 2500, 0] = spike
    kf[:, :, 2700, 0] = -spike
    q = qf.astype(np.float16).view(np.uint16)
    k = kf.astype(np.float16).view(np.uint16)
    scale = 1 / math.sqrt(D)
    out, lse = run_gpu(q, k, v, W, S, scale, packed)
    with input_format("fp16"):
        ro, rl = swaa_attn_oracle(q, k, v, W, S, scale)
    assert_parity(out, lse, ro, rl, tag=f"fp16 late spike {spike}")


@on_both_kernels
def test_all_scores_far_below_the_reference(packed):
    # rows whose first visited half tile is invisible to them start from reference 0; with every
    # score near -30 nats their binary16 probabilities vanish altogether and the kernel has to
    # notice (the sum of the rounded P is zero although the fp32 sum is in range)
    B, H, N, D, W, S = 1, 2, 900, 128, 70, 0
    scale = 1 / math.sqrt(D)
    q, k, v = make_qkv(B, H, H, N, D, seed=9750, fmt="fp16")
    qf = q.view(np.float16).astype(np.float32)
    kf = k.view(np.float16).astype(np.float32)
    a = math.sqrt(30.0 / scale)
    qf[..., 0] = a
    kf[..., 0] = -a
    q = qf.astype(np.float16).view(np.uint16)
    k = kf.astype(np.float16).view(np.uint16)
    out, lse = run_gpu(q, k, v, W, S, scale, packed)
    with input_format("fp16"):
        ro, rl = swaa_attn_oracle(q, k, v, W, S, scale)
    assert float(rl.max()) < -15.0
    assert_parity(out, lse, ro, rl, tag="fp16 scores far below the reference")


def test_mid_size_sampled_rows():
    B, Hq, Hkv, N, D, W, S = 1, 32, 8, 16384, 128, 2048, 4
    rows = sample_rows(N, W, S, count=128, seed=9730)
    check(B, Hq, Hkv, N, N, D, W, S, None, seed=9730, rows=rows)
