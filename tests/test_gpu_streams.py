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
