"""The extension module behind the binding's per-step calls: what reaches the entry point for each kind of
argument, and what is refused before it is called."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding


@pytest.fixture()
def entry():
    binding.load()
    seen = []

    @ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_uint64] * 4, *[ctypes.c_int32] * 2, *[ctypes.c_uint64] * 3)
    def record(*args):
        seen.append(args)
        return -3
    address = ctypes.cast(record, ctypes.c_void_p).value
    return seen, lambda kinds, *args: binding._call(address, kinds, *args), record


class Stream:
    cuda_stream = 0xFFFF_8000_0000_0010


def test_arguments_arrive(entry):
    seen, call, _ = entry
    t = torch.zeros((3, 4))
    assert call("hppsiipps", 2**63 + 1, t, None, Stream(), -5, np.int64(7), 2**40 + 8, t[1:], None) == -3
    assert seen == [(2**63 + 1, t.data_ptr(), 0, Stream.cuda_stream, -5, 7, 2**40 + 8, t[1:].data_ptr(), 0)]
    assert call("hppsiipps", 0, 0, 16, 32, True, 0, None, None, 48) == -3
    assert seen[1] == (0, 0, 16, 32, 1, 0, 0, 0, 48)


def test_refusals(entry):
    seen, call, _ = entry
    t = torch.zeros((4, 4))
    for error, kinds, args in [(ValueError, "p", (t.t()[:, :2],)), (TypeError, "i", (1.0,)), (TypeError, "i", (None,)),
                               (AttributeError, "p", (1.5,)), (AttributeError, "p", (np.zeros(3),)),
                               (AttributeError, "s", ("x",)), (TypeError, "pp", (t,)), (TypeError, "p", (t, t)),
                               (TypeError, "h" * 10, (0,) * 10), (TypeError, "", ())]:
        with pytest.raises(error):
            call(kinds, *args)
    with pytest.raises((TypeError, OverflowError)):
        binding._call(None, "h", 0)
    assert seen == []


def test_every_step_call_states_its_entry_point_s_arguments():
    """The kinds of a call are as many as the entry point takes, pointers where it takes pointers."""
    import inspect
    import re
    lib = binding.load()
    calls = re.findall(r'"(eep_[a-z_]+)",\s*"([hpis]+)"', inspect.getsource(binding))
    calls += re.findall(r'\["(eep_[a-z_]+)"\],\s*"([hpis]+)"', inspect.getsource(binding))
    assert len(calls) == 10
    for name, kinds in calls:
        want = ["i" if a is ctypes.c_int32 else "p" for a in getattr(lib, name).argtypes]
        assert [{"h": "p", "s": "p"}.get(c, c) for c in kinds] == want, name
