"""The caller's stream belongs to one call: a later call, of any size and
kind, neither uses nor waits for a stream that an earlier call was given.
Answers against the oracle, equal.
"""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2508_20735_amd import binding as B
from paper_2508_20735_amd import workloads as W

pytestmark = pytest.mark.gpu

SMALL = W.random_dfa(500, 3, 0.3, 1)      # whole in one workgroup
MIDDLE = W.random_dfa(20_000, 3, 0.3, 2)  # one launch per round
CAPTURE_RELAXED = 2


class Stream:
    """A stream of the HIP runtime itself (torch never destroys its own)."""

    def __init__(self):
        self.hip = B.load()  # (the runtime's functions are found through the library)
        self.cuda_stream = ctypes.c_void_p()
        self.ok(self.hip.hipStreamCreateWithFlags(ctypes.byref(self.cuda_stream), 1))
        self.cuda_stream = self.cuda_stream.value

    @staticmethod
    def ok(rc):
        assert rc == 0, rc

    def begin_capture(self):
        self.ok(self.hip.hipStreamBeginCapture(ctypes.c_void_p(self.cuda_stream), CAPTURE_RELAXED))

    def end_capture(self):
        """Nodes of the graph."""
        graph, nodes = ctypes.c_void_p(), ctypes.c_size_t()
        self.ok(self.hip.hipStreamEndCapture(ctypes.c_void_p(self.cuda_stream),
                                             ctypes.byref(graph)))
        self.ok(self.hip.hipGraphGetNodes(graph, None, ctypes.byref(nodes)))
        self.ok(self.hip.hipGraphDestroy(graph))
        return nodes.value

    def destroy(self):
        self.ok(self.hip.hipStreamDestroy(ctypes.c_void_p(self.cuda_stream)))


def device(d):
    import torch
    return (torch.from_numpy(d.delta.view(np.int32)).cuda(), torch.from_numpy(d.accepting).cuda())


def device_call(kind, d, stream):
    import torch
    delta, acc = device(d)
    torch.cuda.synchronize()
    if kind == "minimise":
        block = B.minimise_device(delta, acc, stream=stream).block.cpu().numpy().view(np.uint32)
        np.testing.assert_array_equal(block, oracle.hopcroft(d.delta, d.accepting)[0])
    elif kind == "equivalent":
        assert B.equivalent_device(delta, acc, d.start, delta, acc, d.start, stream=stream)[0]
    else:  # a target out of range: the call ends with an error
        delta[3, 1] = d.n
        torch.cuda.synchronize()
        with pytest.raises(B.DfaError):
            B.minimise_device(delta, acc, stream=stream)


def host_calls(d):
    np.testing.assert_array_equal(B.minimise(d.delta, d.accepting).block,
                                  oracle.hopcroft(d.delta, d.accepting)[0])
    other = W.mutate_one(d, 3)[0]
    args = (d.delta, d.accepting, d.start, other.delta, other.accepting, other.start)
    assert B.equivalent(d, other)[0] == oracle.equiv_hk(*args)
    assert B.equivalent(d, other, method="product")[0] == oracle.equiv_hk(*args)
    assert B.included(d, other)[0] == oracle.included(*args)
    np.testing.assert_array_equal(
        B.minimise(d.delta, d.accepting, prune=True).block,
        oracle.minimise_reachable(d.delta, d.accepting, d.start)[0])


@pytest.mark.parametrize("later", [SMALL, MIDDLE], ids=["small", "middle"])
@pytest.mark.parametrize("kind", ["minimise", "equivalent", "error"])
def test_nothing_goes_to_an_earlier_calls_stream(kind, later):
    """The stream is being captured by then: whatever a call put there would
    be in the graph."""
    stream = Stream()
    device_call(kind, SMALL, stream)
    stream.begin_capture()
    try:
        host_calls(later)
    finally:
        nodes = stream.end_capture()
    assert nodes == 0
    stream.destroy()


@pytest.mark.parametrize("later", [SMALL, MIDDLE], ids=["small", "middle"])
@pytest.mark.parametrize("kind", ["minimise", "equivalent", "error"])
def test_the_stream_may_go_when_the_call_has_returned(kind, later):
    stream = Stream()
    device_call(kind, SMALL, stream)
    stream.destroy()
    host_calls(later)
    import torch
    device_call("minimise", later, torch.cuda.current_stream())
