"""GPU tests of calls on a stream other than torch's current one: the memory that a call allocates belongs to the
stream it runs on, so that calls on different streams may overlap."""
import pytest
import torch

from paper_2512_10411_amd import binding
from paper_2512_10411_amd.inputs import make_qkv
from gpu_util import to_device

pytestmark = pytest.mark.gpu


def split_call(seed):
    q, k, v = (to_device(x) for x in make_qkv(1, 8, 2, 6000, 128, seed=seed, n_query=64))
    return lambda stream=None: binding.swaa_attn_fwd_ex(q, k, v, 10**9, 4, stream=stream)


@pytest.mark.parametrize("how", ["stream", "handle", "default stream's handle"])
def test_split_calls_on_two_streams_have_scratch_of_their_own(how, monkeypatch):
    first, second = split_call(9801), split_call(9802)  # of one size: a pool would hand out the same block twice
    want = [tuple(t.clone() for t in f()) for f in (first, second)]
    lib, scratch = binding.load_library(), []
    launch = lib.swaa_attn_fwd_ex_ws

    def recording(args, workspace, workspace_bytes):
        scratch.append(workspace)
        return launch(args, workspace, workspace_bytes)

    monkeypatch.setattr(lib, "swaa_attn_fwd_ex_ws", recording)
    side = torch.cuda.Stream()
    current, other = {"stream": (torch.cuda.default_stream(), side), "handle": (torch.cuda.default_stream(), side.cuda_stream),
                      "default stream's handle": (side, 0)}[how]
    torch.cuda.synchronize()
    with torch.cuda.stream(current):
        got = [first(), second(other)]
    torch.cuda.synchronize()
    assert len(scratch) == 2 and scratch[0] != scratch[1]
    for (o, l), (wo, wl) in zip(got, want):
        assert torch.equal(o, wo) and torch.equal(l, wl)


def cases():
    q, k, v = (to_device(x) for x in make_qkv(1, 8, 2, 300, 128, seed=9810))
    new = q[:, :, -2:].contiguous()
    out, lse = binding.swaa_attn_fwd(q, k, v, 100, 4)
    return {
        "fwd": lambda **s: binding.swaa_attn_fwd(q, k, v, 100, 4, **s),
        "fwd_fa_decode": lambda **s: binding.swaa_attn_fwd_fa_decode(q, k, v, 100, 4, 200, **s),
        "fwd_ex": lambda **s: binding.swaa_attn_fwd_ex(q, k, v, 100, 4, **s),
        "decode": lambda **s: binding.swaa_attn_decode(new, k, v, 100, 4, **s),
        "decode_ex": lambda **s: binding.swaa_attn_decode_ex(new, k, v, 100, 4, **s),
        "bwd": lambda **s: binding.swaa_attn_bwd(q, k, v, out, lse, q, 100, 4, **s),
    }


@pytest.mark.parametrize("call", ["fwd", "fwd_fa_decode", "fwd_ex", "decode", "decode_ex", "bwd"])
def test_what_a_call_allocates_comes_from_the_launch_streams_pool(call, monkeypatch):
    f = cases()[call]
    want = [t.clone() for t in f()]
    side, pools = torch.cuda.Stream(), []
    for name in ("empty", "empty_like", "empty_strided"):
        def recording(*args, real=getattr(torch, name), **kwargs):
            pools.append(torch.cuda.current_stream().cuda_stream)
            return real(*args, **kwargs)
        monkeypatch.setattr(torch, name, recording)
    torch.cuda.synchronize()
    got = f(stream=side)
    again = f(stream=side.cuda_stream)
    torch.cuda.synchronize()
    assert len(pools) >= 4 and all(p == side.cuda_stream for p in pools)
    assert torch.cuda.current_stream() == torch.cuda.default_stream()
    assert all(torch.equal(x, w) and torch.equal(y, w) for x, y, w in zip(got, again, want))
