"""Which form a layout takes when its mask may change while it runs: with several contexts in an
instance, and without a context, one workgroup or tiles (each pair is mapped once), never the
form in which eight workgroups map every pair for themselves; beyond one workgroup, with several contexts,
workgroups that agree on a mask first."""
import numpy as np
import pytest

from paper_2605_10670_amd import binding

from test_gpu_layout_edges import instance


def workgroups(R, S, E, k, T, several):
    return binding.load().eep_host_layout_workgroups(R, S, E, k, T, int(several))


def test_form_by_size_and_number_of_contexts():
    R, S, E, k = 32, 9, 256, 8
    for T in range(0, 2049, 32):
        assert workgroups(R, S, E, k, T, False) == (8 if 0 < T <= 512 else 0), T
        assert workgroups(R, S, E, k, T, True) == (1 if 0 < T <= 384 else 0), T
    # by pairs: 4096 and 3072
    assert workgroups(4, 20, 64, 32, 128, False) == 8 and workgroups(4, 20, 64, 32, 132, False) == 0
    assert workgroups(4, 20, 64, 32, 96, True) == 1 and workgroups(4, 20, 64, 32, 100, True) == 0
    # tables that leave no room for the bitmaps in LDS
    assert workgroups(1, 1200, 300, 2, 512, False) == workgroups(1, 1200, 300, 2, 512, True) == 0
    for bad in [(0, 9, 256, 8, 0, 0), (32, 0, 256, 8, 0, 0), (32, 9, 0, 8, 0, 0), (32, 9, 256, 0, 0, 0),
                (32, 9, 256, 33, 0, 0), (32, 9, 256, 8, 33, 0), (32, 9, 256, 8, -32, 0)]:
        assert binding.load().eep_host_layout_workgroups(*bad) == binding.ERR_INVALID_ARG


@pytest.mark.gpu
@pytest.mark.parametrize("T,k,R,S,E", [(32, 8, 32, 9, 256), (384, 8, 32, 9, 256), (416, 8, 32, 9, 256),
                                       (512, 8, 32, 9, 256), (96, 32, 4, 20, 64), (500, 3, 4, 6, 16),
                                       (260, 8, 65, 2, 96), (1024, 8, 32, 9, 256)])
def test_captured_layout_outlives_a_change_of_the_number_of_contexts(oracle, T, k, R, S, E):
    import torch
    import gpu_util as gu
    S_prim = S - 1
    shape = dict(num_ranks=R, slots_per_rank=S, primary_slots=S_prim, num_logical=E, max_tokens=T,
                 topk=k, hidden=64, strict_coverage=False)
    ctx = binding.Context(**shape)
    stream = torch.cuda.Stream()
    other = None
    try:
        p2l, active, idx = instance(T, k, R, S, E, seed=T + k)
        idx_dev = gu.to_dev(idx)
        ctx.update_placement(p2l, stream)
        ctx.dispatch_layout(idx_dev, T, stream)
        stream.synchronize()
        ctx.graph_begin(stream)
        ctx.dispatch_layout(idx_dev, T, stream)
        graph = ctx.graph_end(stream)

        def check(mask, c=ctx):
            got = c.read_layout(T, stream)
            gu.assert_layout_equal(got, oracle.step_layout(idx, p2l, mask, E, R, S, S_prim, binding.SPREAD),
                                   T, k)
            assert c.check_layout(T, stream).tolist() == [0, 0, 0, 0]

        for mask in (active, np.ones(R, np.int32)):
            for several in (False, True, False):
                if several:
                    other = binding.Context(**shape, parent=ctx)
                    other.update_placement(p2l, stream)
                    other.set_membership(mask, stream)
                    other.dispatch_layout(idx_dev, T, stream)      # launched while there are two
                    check(mask, other)
                else:
                    if other is not None:
                        other.destroy()
                        other = None
                    ctx.set_membership(mask, stream)
                graph.launch(stream)                               # captured while there was one
                check(mask)
                ctx.dispatch_layout(idx_dev, T, stream)
                check(mask)
        graph.destroy()
    finally:
        if other is not None:
            other.destroy()
        ctx.destroy()


@pytest.mark.gpu
def test_attaching_leaves_another_threads_capture_alone():
    """Attaching waits for the device; it may neither fail nor spoil a capture because an unrelated
    context is being captured meanwhile."""
    import threading
    import torch
    import gpu_util as gu
    shape = dict(num_ranks=4, slots_per_rank=2, primary_slots=2, num_logical=8, max_tokens=64, topk=2,
                 hidden=64)
    a, b = binding.Context(**shape), binding.Context(**shape)
    p2l = np.arange(8, dtype=np.int32)
    idx = gu.to_dev(np.tile(np.array([0, 1], np.int32), (64, 1)))
    for ctx in (a, b):
        ctx.update_placement(p2l)
        ctx.dispatch_layout(idx, 64)
    torch.cuda.synchronize()
    capturing, attached, errors = threading.Event(), threading.Event(), []

    def capture():
        try:
            stream = torch.cuda.Stream()
            b.graph_begin(stream)
            b.dispatch_layout(idx, 64, stream)
            capturing.set()
            attached.wait(60)
            b.dispatch_layout(idx, 64, stream)
            graph = b.graph_end(stream)
            graph.launch(stream)
            stream.synchronize()
            graph.destroy()
        except Exception as exc:
            errors.append(repr(exc))
            capturing.set()

    thread = threading.Thread(target=capture)
    try:
        thread.start()
        assert capturing.wait(60)
        others = [binding.Context(**shape, parent=a), a.staging()]
    finally:
        attached.set()
        thread.join(60)
    assert not errors, errors
    for ctx in others + [b, a]:
        ctx.destroy()
