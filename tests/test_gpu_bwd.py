"""GPU parity of swaa_attn_bwd (dQ, dK, dV) against the fp64 CPU oracle, through the C ABI.

The forward results the backward call consumes (out, lse) come from the library's own
forward call, as in training.

Tolerance (no figure is given for the backward pass; this one is derived from the arithmetic).
Every gradient element is a sum  x = c * sum_t a_t b_t  whose factor a_t (P for dV, dS for dQ
and dK) is rounded to bf16 before the product, accumulated in fp32, and rounded to bf16 at the
end.  With u = 2^-9 (half a bf16 step, relative) and rounding errors spread evenly over
[-u, u] (standard deviation u / sqrt 3):

    |error(x)|  <=  u |x|  +  4 * (u / sqrt 3) * rss(terms)          (four standard deviations)

and rss(terms) <= max|x| over the tensor for the elements that matter (an element is large
exactly when its terms align), so  error <= (1 + 4 / sqrt 3) u max|ref| = 6.5e-3 max|ref|; the
bar is MAX_REL = 8e-3.  One more channel reaches dQ and dK only: delta_i = <dO_i, O_i> is formed
from the forward's bf16 output, whose elements carry independent roundings of up to u |O_id|
(the forward divides by the sum of the ROUNDED P, so a row that sees a single key returns that
key's value row exactly and delta is exact there; the one-signed error of up to 2^-8 |delta| that
an earlier forward left in rows dominated by one key is gone).  So delta_i is off by about
(u / sqrt 3) * sqrt(sum_d dO_id^2 O_id^2), 0.013 for D = 128 and 0.009 for D = 64 with N(0,1)
data, dS_ij by P_ij times that, and dQ_i (dK_j) by scale * that * |P-weighted mean of k| (of q):
at four standard deviations and |k|, |q| <= 4.5 this is scale * 4.5 * 4 * 0.013 = 2e-2 for both
head dimensions, reached only by rows that put nearly all weight on one key with a large
component; rows that spread over many keys average it out.  Hence

    max-abs error  <=  8e-3 * max|ref| + abs,    abs = 2e-2 (dQ, dK), 2e-3 (dV)
    mean-abs error <=  4e-3 * mean|ref| + 1e-3

Measured over every case below: max-abs error <= 5.8e-3 max|ref| (dQ), 4.6e-3 (dK), 4.4e-3 (dV);
the absolute terms are never drawn upon by more than 1e-6 (they matter where the true gradient
is zero).
"""
import math

import numpy as np
import pytest
import torch

from oracle import swaa_attn_bwd_oracle
from paper_2512_10411_amd import binding
from paper_2512_10411_amd.inputs import f32_to_bf16_bits, make_qkv
from gpu_util import to_device

pytestmark = pytest.mark.gpu

MAX_REL = 8e-3
MAX_ABS = {"dq": 2e-2, "dk": 2e-2, "dv": 2e-3}
MEAN_REL, MEAN_ABS = 4e-3, 1e-3


def make_dout(shape, seed):
    rng = np.random.Generator(np.random.Philox(seed))
    return f32_to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))


def assert_grad(name, got, ref, tag):
    g = got.float().cpu().numpy().astype(np.float64)
    assert g.shape == ref.shape and np.isfinite(g).all(), (tag, name)
    err = np.abs(g - ref)
    rmax, rmean = np.abs(ref).max(), np.abs(ref).mean()
    print(f"[grad] {tag} {name}: max-abs err {err.max():.3e} (max|ref| {rmax:.3e}), mean-abs err {err.mean():.3e} "
          f"(mean|ref| {rmean:.3e})", flush=True)
    assert err.max() <= MAX_REL * rmax + MAX_ABS[name], (tag, name, err.max(), rmax)
    assert err.mean() <= MEAN_REL * rmean + MEAN_ABS, (tag, name, err.mean(), rmean)


def whole_key_tiles(B, Hq, Hkv, N, D, W, S, P):
    """A workspace one byte too small for a plan that cuts the key tiles' steps into pieces: the call runs without."""
    need = binding.swaa_attn_bwd_workspace_bytes(B, Hq, Hkv, N, D, W, S, P)
    return torch.empty(need - 1, dtype=torch.uint8, device="cuda")


def check(B, Hq, Hkv, N, D, W, S, P, seed, whole=False):
    tag = f"bwd B{B} Hq{Hq} Hkv{Hkv} N{N} D{D} W{W} S{S} P{P}" + (" whole key tiles" if whole else "")
    print(f"[case] {tag} seed {seed}", flush=True)
    scale = 1 / math.sqrt(D)
    q, k, v = make_qkv(B, Hq, Hkv, N, D, seed)
    dout = make_dout(q.shape, seed + 1)
    qd, kd, vd, dd = to_device(q), to_device(k), to_device(v), to_device(dout)
    n_prompt = N if P is None else P
    out, lse = binding.swaa_attn_fwd_fa_decode(qd, kd, vd, W, S, n_prompt, scale)
    ws = whole_key_tiles(B, Hq, Hkv, N, D, W, S, n_prompt) if whole else None
    dq, dk, dv = binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, W, S, n_prompt, scale, workspace=ws)
    torch.cuda.synchronize()
    rq, rk, rv = swaa_attn_bwd_oracle(q, k, v, dout, W, S, scale, n_prompt=n_prompt)
    assert_grad("dq", dq, rq, tag)
    assert_grad("dk", dk, rk, tag)
    assert_grad("dv", dv, rv, tag)


@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 130, 300, 700])
@pytest.mark.parametrize("D", [64, 128])
def test_small_shapes_sweep_the_mask(N, D):
    seed = 9000 + N + D
    for W, S, P in ((1, 0, None), (7, 4, None), (64, 0, None), (65, 70, None), (N, 0, None), (50, 3, N // 2),
                    (200, 0, 0)):
        if W == 1 and S == 0:
            continue  # dK = dQ = 0 exactly: a relative bar has nothing to measure (covered below)
        check(1, 4, 1, N, D, W, S, P, seed)


def test_window_one_gives_zero_dq_dk_and_dv_equal_to_dout():
    B, Hq, Hkv, N, D = 1, 4, 2, 333, 128
    q, k, v = make_qkv(B, Hq, Hkv, N, D, seed=9100)
    dout = make_dout(q.shape, 9101)
    qd, kd, vd, dd = to_device(q), to_device(k), to_device(v), to_device(dout)
    out, lse = binding.swaa_attn_fwd(qd, kd, vd, 1, 0)
    dq, dk, dv = binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, 1, 0)
    torch.cuda.synchronize()
    # a row that sees one key has O = v exactly, so dP - delta vanishes up to the order of two
    # fp32 sums of 128 products of N(0,1) values: 1e-5 at most, times scale * |k| <= 0.4
    print(f"[grad] W=1: max |dq| {dq.float().abs().max().item():.3e}, max |dk| {dk.float().abs().max().item():.3e}",
          flush=True)
    assert dq.float().abs().max().item() <= 1e-4 and dk.float().abs().max().item() <= 1e-4
    want = dd.float().view(B, Hkv, 2, N, D).sum(dim=2)
    assert (dv.float() - want).abs().max().item() <= 2.0 ** -7 * want.abs().max().item()


@pytest.mark.parametrize("G", [1, 2, 3, 5, 8])
def test_gqa_group_sizes_and_batches(G):
    check(2, 2 * G, 2, 333, 128, 100, 3, None, seed=9200 + G)
    check(1, G, 1, 515, 64, 65, 10, 400, seed=9300 + G)


@pytest.mark.parametrize("N,W,S,P,G", [
    (31, 31, 0, None, 1),     # one row block for three parts
    (97, 97, 0, None, 2),     # eight entries in the list: the last step is not full
    (161, 20, 0, None, 3),    # two or three blocks in a key tile's band, a key tile of 33 keys
    (1037, 90, 10, None, 1),  # sink segments, cut at whole 64-row tiles, the last one short
    (1037, 90, 140, 900, 4),  # two sink key tiles, generated rows
    (545, 33, 0, 500, 5),     # a second range that starts inside a block
])
def test_row_blocks_of_head_dimension_64(N, W, S, P, G):
    check(1, 2 * G, 2, N, 64, W, S, P, seed=9600 + N)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hkv,N,W,S,P", [
    (65, 8, 300, 64, 4, None),   # 520 key tiles with sinks: one segment each, of all rows beyond the band
    (33, 8, 500, 100, 200, 450),  # two to a pair, generated rows
])
def test_more_sink_key_tiles_than_there_are_segments(B, Hkv, N, W, S, P, D):
    check(B, Hkv, Hkv, N, D, W, S, P, seed=9650 + N + D)


@pytest.mark.parametrize("N,W,S,P,G", [
    (32, 32, 0, None, 1),     # one half of a tile, the other a padding half
    (33, 33, 0, None, 4),     # one key in the second half
    (97, 97, 0, None, 2),     # odd number of halves: padding half behind the end
    (300, 64, 33, None, 1),   # two halves with sinks, then the band's, odd and even counts
    (300, 40, 32, None, 5),   # sinks end with a half; windows that begin inside one
    (600, 33, 4, None, 8),    # many halves that a wave leaves out
    (515, 70, 40, 400, 4),    # generated rows see all halves, the others of their workgroup do not
])
def test_half_tiles_of_dq_head_dimension_64(N, W, S, P, G):
    check(1, 2 * G, 2, N, 64, W, S, P, seed=7400 + N + W)


# Head dimension 128 has two dK/dV kernels, of eight waves ("8") and of one wave per SIMD ("1"); which one runs depends on the
# shape and on whether the key tiles' steps are cut into pieces.  The last entry: the kernel in pieces, then that of whole key
# tiles (a workspace too small for pieces), which is run too; one letter where the plan has no pieces.
# tests/test_host_bwd_plan.py checks the letters.
UNITS = [
    (1, 2, 1, 33, 33, 0, None, "8"),       # one tile, its second row half one row long
    (1, 2, 2, 193, 31, 0, None, "8"),      # a window inside a 32-key unit, a key tile of 65 keys
    (1, 2, 3, 259, 97, 0, None, "8"),      # three tiles of query rows in a band, the last key tile has three keys
    (1, 2, 1, 1029, 64, 33, None, "8"),    # sinks that end inside the second unit: segments, one of them short
    (1, 2, 4, 1029, 160, 130, 901, "81"),  # two sink key tiles, generated rows that start inside a tile
    (1, 2, 5, 545, 545, 0, 511, "81"),     # no window; the row before a tile is generated
    (1, 2, 4, 449, 449, 0, None, "81"),    # a key tile of 65 keys
    (1, 2, 4, 515, 515, 4, None, "81"),    # the last key tile has three keys
    (1, 2, 2, 1029, 150, 33, None, "81"),  # sinks that end inside the second unit, a window that ends inside a unit
    (1, 2, 3, 1029, 135, 4, 700, "81"),    # the same with generated rows
    (1, 2, 8, 929, 139, 1, None, "81"),    # a window two rows longer than a whole number of units, a key tile of 33 keys
    (1, 1, 2, 2049, 1500, 140, 1849, "11"),  # pieces and segments of one wave per SIMD, a key tile of one key, generated rows
    (1, 4, 5, 1281, 1281, 4, None, "11"),  # pieces that begin inside a head's list
]
LINE = [
    (1, 2, 4, 384, 384, 0, None, "88"), (1, 2, 4, 385, 385, 0, None, "81"),        # few workgroups, on both sides of the rule
    (1, 2, 4, 1024, 192, 4, None, "81"), (1, 2, 4, 1024, 193, 4, None, "81"),
    (1, 2, 4, 1024, 128, 4, None, "88"), (1, 2, 4, 1024, 129, 4, None, "81"),      # with segments of sinks
    (1, 2, 1, 768, 768, 0, None, "88"), (1, 2, 1, 769, 769, 0, None, "81"),        # one head per KV head
    (8, 16, 4, 256, 256, 0, None, "8"),                                            # a full chip
    (1, 2, 4, 640, 64, 0, 256, "8"), (1, 2, 4, 640, 64, 0, 200, "8"),              # generated rows count half
    (1, 2, 4, 640, 64, 0, 129, "8"), (1, 2, 4, 640, 64, 0, 128, "1"),
    (1, 1, 4, 1536, 1536, 0, None, "81"), (1, 1, 4, 1537, 1537, 0, None, "11"),    # eight pieces
    (1, 8, 4, 896, 896, 4, None, "81"), (1, 8, 4, 897, 897, 4, None, "11"),        # five and four
    (1, 8, 1, 1536, 1536, 0, None, "81"), (1, 8, 1, 1537, 1537, 0, None, "11"),    # one head per KV head: three and two
]


def runs(cases):
    return [(*c[:7], whole) for c in cases for whole in range(len(c[7]))]


@pytest.mark.parametrize("B,Hkv,G,N,W,S,P,whole", runs(UNITS))
def test_units_and_tiles_of_head_dimension_128(B, Hkv, G, N, W, S, P, whole):
    check(B, Hkv * G, Hkv, N, 128, W, S, P, seed=9800 + N, whole=whole)


@pytest.mark.parametrize("B,Hkv,G,N,W,S,P,whole", runs(LINE))
def test_both_kernels_of_head_dimension_128_at_the_line_between_them(B, Hkv, G, N, W, S, P, whole):
    check(B, Hkv * G, Hkv, N, 128, W, S, P, seed=9900 + N + W, whole=whole)


# of the tests of NaN below, as UNITS; then (head dimension, window, whole key tiles?)
NAN_LINE = [(1, 1, 4, 700, 90, 4, None, "88"), (1, 1, 4, 700, 140, 4, None, "81"), (1, 1, 4, 700, 400, 4, None, "81")]
NAN_RUNS = [(64, 90, 0), (64, 90, 1)] + [(128, c[4], whole) for c in NAN_LINE for whole in (0, 1)]


@pytest.mark.parametrize("what", ["dout", "q"])
@pytest.mark.parametrize("D,W,whole", NAN_RUNS)
def test_an_upstream_row_without_a_number_stays_in_its_blocks(D, W, whole, what):
    # 32 rows x 32 keys are computed together, so NaN in one row of dO (or Q) may reach the keys of
    # those blocks in which some row of its 32 sees some key, and no others
    N, row = 700, 333
    q, k, v = make_qkv(1, 4, 1, N, D, seed=9710)
    qd, kd, vd, dd = to_device(q), to_device(k), to_device(v), to_device(make_dout(q.shape, 9711))
    out, lse = binding.swaa_attn_fwd(qd, kd, vd, W, 4)
    ws = whole_key_tiles(1, 4, 1, N, D, W, 4, None) if whole else None
    want = binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, W, 4, workspace=ws)
    (dd if what == "dout" else qd)[:, :, row] = float("nan")
    got = binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, W, 4, workspace=ws)
    torch.cuda.synchronize()
    first = row // 32 * 32
    reached = torch.zeros(N, dtype=torch.bool, device="cuda")
    reached[:32], reached[max(0, first - W + 1) // 32 * 32:first + 32] = True, True
    rows = torch.arange(N, device="cuda") != row
    assert torch.equal(got[0][:, :, rows], want[0][:, :, rows])
    for x, y in zip(got[1:], want[1:]):  # dK, dV
        assert torch.equal(x[:, :, ~reached], y[:, :, ~reached])


@pytest.mark.parametrize("D,W,whole", NAN_RUNS)
def test_a_row_without_a_number_reaches_only_the_keys_it_sees(D, W, whole):
    # NaN in one row's log-sum-exp: P = 0 where the row does not see the key, whatever the row holds
    N, row = 700, 333
    q, k, v = make_qkv(1, 4, 1, N, D, seed=9700)
    qd, kd, vd, dd = to_device(q), to_device(k), to_device(v), to_device(make_dout(q.shape, 9701))
    out, lse = binding.swaa_attn_fwd(qd, kd, vd, W, 4)
    ws = whole_key_tiles(1, 4, 1, N, D, W, 4, None) if whole else None
    want = binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, W, 4, workspace=ws)
    lse[:, :, row] = float("nan")
    got = binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, W, 4, workspace=ws)
    torch.cuda.synchronize()
    seen = torch.zeros(N, dtype=torch.bool, device="cuda")
    seen[:4], seen[max(0, row - W + 1):row + 1] = True, True
    rows = torch.arange(N, device="cuda") != row
    assert torch.equal(got[0][:, :, rows], want[0][:, :, rows])
    for x, y in zip(got[1:], want[1:]):  # dK, dV
        assert torch.equal(x[:, :, ~seen], y[:, :, ~seen])
        assert not torch.isfinite(x[:, :, seen].float()).any()


@pytest.mark.parametrize("D,N", [(64, 97), (128, 97), (128, 500)])
def test_the_sums_of_delta_are_no_deeper_than_a_tree(D, N):
    # delta = <dO, O> stands at the front of the workspace.  Products of bf16 are exact in fp32; a sum of additions at most
    # 12 deep (eight in a row, then pairs) is off by at most 12 u of the sum of the absolute values, u = 2^-24.
    # One product of 2^24 in front of 127 of 0.75: adding those one by one loses them all, 47 u and more.
    Hq, Hkv = 4, 2
    q, k, v = make_qkv(1, Hq, Hkv, N, D, seed=9720)
    qd, kd, vd, dd = to_device(q), to_device(k), to_device(v), to_device(make_dout(q.shape, 9721))
    out, lse = binding.swaa_attn_fwd(qd, kd, vd, 64, 4)
    dd[:, 1], out[:, 1] = 1.0, 0.75
    dd[:, 1, :, 0], out[:, 1, :, 0] = 4096.0, 4096.0
    dd[:, 2], out[:, 2] = 1.0, 0.75
    dd[:, 2, :, 24], out[:, 2, :, 24] = 4096.0, -4096.0
    ws = torch.empty(binding.swaa_attn_bwd_workspace_bytes(1, Hq, Hkv, N, D, 64, 4), dtype=torch.uint8, device="cuda")
    binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, 64, 4, workspace=ws)
    torch.cuda.synchronize()
    delta = ws[:4 * Hq * N].view(torch.float32).view(Hq, N).double()
    x = dd[0].double() * out[0].double()
    off = (delta - x.sum(-1)).abs() / x.abs().sum(-1) * 2.0**24
    print(f"[delta] D{D}: off by {[round(o, 2) for o in off.amax(-1).tolist()]} u", flush=True)
    assert off.max().item() <= 12


def test_run_to_run_determinism_and_errors():
    q, k, v = make_qkv(1, 8, 2, 1000, 128, seed=9400)
    qd, kd, vd = to_device(q), to_device(k), to_device(v)
    dd = to_device(make_dout(q.shape, 9401))
    out, lse = binding.swaa_attn_fwd(qd, kd, vd, 256, 4)
    a = binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, 256, 4)
    b = binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, 256, 4)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    with pytest.raises(binding.SwaaError) as e:
        binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, 256, 4, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    assert e.value.status == binding.SWAA_ERR_WORKSPACE
    with pytest.raises(binding.SwaaError):
        binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, 0, 4)


@pytest.mark.parametrize("shape", [(1, 8, 2, 4096 + 37, 128, 512, 4, None), (1, 16, 4, 8192, 128, 1024, 4, 8192 - 300),
                                   (2, 10, 2, 2048, 128, 2048, 0, None)])
def test_mid_size_every_element(shape):
    B, Hq, Hkv, N, D, W, S, P = shape
    check(B, Hq, Hkv, N, D, W, S, P, seed=9500 + N)


def test_benchmark_workload_at_full_size_two_kv_heads():
    """The launch configuration bench.py times (workload mid_bwd, all 32 heads), checked on
    every element of the first and the last KV head with their query heads: heads are
    independent, so the oracle runs on those slices only (about 20 s on the host)."""
    from paper_2512_10411_amd.inputs import WORKLOADS, make_workload

    w = WORKLOADS["mid_bwd"]
    q, k, v = make_workload(w)
    dout = make_dout(q.shape, w.seed + 1)
    qd, kd, vd, dd = to_device(q), to_device(k), to_device(v), to_device(dout)
    out, lse = binding.swaa_attn_fwd(qd, kd, vd, w.window, w.n_sink, w.scale)
    dq, dk, dv = binding.swaa_attn_bwd(qd, kd, vd, out, lse, dd, w.window, w.n_sink, None, w.scale)
    torch.cuda.synchronize()
    G = w.Hq // w.Hkv
    for kvh in (0, w.Hkv - 1):
        tag = f"mid_bwd full size, KV head {kvh}"
        print(f"[case] {tag}", flush=True)
        hs = slice(kvh * G, (kvh + 1) * G)
        rq, rk, rv = swaa_attn_bwd_oracle(np.ascontiguousarray(q[:, hs]), np.ascontiguousarray(k[:, kvh:kvh + 1]),
                                          np.ascontiguousarray(v[:, kvh:kvh + 1]), np.ascontiguousarray(dout[:, hs]),
                                          w.window, w.n_sink, w.scale)
        assert_grad("dq", dq[:, hs], rq, tag)
        assert_grad("dk", dk[:, kvh:kvh + 1], rk, tag)
        assert_grad("dv", dv[:, kvh:kvh + 1], rv, tag)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hkv,G,N,W,S,P", [
    (1, 1, 4, 100, 100, 0, None),    # a single key tile, its pieces shorter than a head's list
    (1, 2, 5, 129, 129, 4, None),    # the last key tile has one key, and fewer steps than there are pieces
    (2, 2, 4, 1000, 128, 200, None),  # two key tiles with sinks: pieces and segments
    (1, 4, 4, 600, 200, 4, 500),     # generated rows behind the band
    (1, 1, 1, 1500, 1500, 0, None),  # one head: pieces of its list of tiles
])
def test_key_tiles_in_pieces(B, Hkv, G, N, W, S, P, D):
    args = (B, G * Hkv, Hkv, N, D, W, S, N if P is None else P)
    whole = 4 * (B * G * Hkv * N + 3) // 4 * 4
    need = binding.swaa_attn_bwd_workspace_bytes(*args)
    assert need > whole  # partial sums of all key tiles
    check(B, G * Hkv, Hkv, N, D, W, S, P, seed=9800 + N + D)
    # a workspace full of NaN patterns gives the same, and so, but for the order of the sums, does one too small for pieces
    q, k, v, dd = (to_device(x) for x in (*make_qkv(B, G * Hkv, Hkv, N, D, seed=9800 + N + D), make_dout((B, G * Hkv, N, D), 9801 + N + D)))
    out, lse = binding.swaa_attn_fwd_fa_decode(q, k, v, W, S, args[7])
    runs = [binding.swaa_attn_bwd(q, k, v, out, lse, dd, W, S, args[7], workspace=torch.full((n,), 255, dtype=torch.uint8, device="cuda"))
            for n in (need, need, need - 1)]
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(runs[0], runs[1]))
    for x, y in zip(runs[0], runs[2]):  # fp32 sums in another order, then one rounding each to bf16
        assert (x.float() - y.float()).norm() <= 2.0 ** -8 * x.float().norm()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hkv,G,N,W,S", [(1, 2, 4, 1000, 1000, 0), (16, 2, 16, 1000, 512, 500)])  # delta alone; segments too
def test_no_memory_for_pieces(B, Hkv, G, N, W, S, D, monkeypatch):
    # where the partial sums of pieces find no memory the call runs on whole key tiles, as with a workspace too small for pieces
    q, k, v, dd = (to_device(x) for x in (*make_qkv(B, G * Hkv, Hkv, N, D, seed=9900 + D), make_dout((B, G * Hkv, N, D), 9901 + D)))
    out, lse = binding.swaa_attn_fwd(q, k, v, W, S)
    want = binding.swaa_attn_bwd(q, k, v, out, lse, dd, W, S, workspace=whole_key_tiles(B, G * Hkv, Hkv, N, D, W, S, None))
    need = binding.swaa_attn_bwd_workspace_bytes(B, G * Hkv, Hkv, N, D, W, S)
    empty = torch.empty

    def little(*args, **kwargs):
        if kwargs.get("dtype") == torch.uint8 and args[0] >= need:
            raise torch.cuda.OutOfMemoryError("no memory")
        return empty(*args, **kwargs)

    monkeypatch.setattr(torch, "empty", little)
    got = binding.swaa_attn_bwd(q, k, v, out, lse, dd, W, S)
    torch.cuda.synchronize()
    monkeypatch.undo()
    assert all(torch.equal(x, y) for x, y in zip(got, want))


@pytest.mark.parametrize("B,Hkv,G,N,W,S,P", [
    (16, 2, 8, 130, 50, 3, 100),      # more than a round of 32-row units of short sequences: rows together, edges of 64 and 256 rows
    (16, 2, 5, 230, 230, 0, None),    # ... groups of four heads and one
    (20, 1, 3, 601, 65, 70, 333),     # ... of two and one, sinks next to the band, generated rows
    (4, 2, 4, 1000, 300, 4, None),    # 1024 units: a head's 32 rows
    (1, 4, 4, 2500, 300, 4, 2400),    # 1264, few generated rows are the time: a head's 32 rows, quarters that differ
    (1, 4, 4, 2500, 300, 4, None),    # ... none: rows together
])
def test_both_dq_kernels_of_head_dimension_128(B, Hkv, G, N, W, S, P):
    check(B, Hkv * G, Hkv, N, 128, W, S, P, seed=9900 + N + G)


@pytest.mark.parametrize("B,Hkv,G,N,W,S,P", [
    (16, 2, 8, 130, 50, 3, 100),      # more than 1024 units of 32 rows: 256 rows together
    (16, 2, 5, 230, 230, 0, None),    # ... groups of four heads and one; the forward too (1280 and 1536 units)
    (20, 1, 3, 865, 65, 70, 333),     # ... of two and one, sinks next to the band, generated rows
    (4, 2, 4, 1000, 300, 4, None),    # 1024 units: a head's 32 rows
    (1, 4, 4, 2500, 300, 4, 2400),    # 1264, few generated rows are the time: a head's 32 rows
    (1, 4, 4, 2500, 300, 4, None),    # ... none: together
])
def test_both_dq_kernels_of_head_dimension_64(B, Hkv, G, N, W, S, P):
    check(B, Hkv * G, Hkv, N, 64, W, S, P, seed=9950 + N + G)
