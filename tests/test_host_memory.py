"""What a block call does on the host when the device's memory or an attribute is refused (no GPU: a recording HIP runtime)."""
from tests import _fake_hip as H


def test_a_buffer_that_cannot_double_grows_to_what_the_call_needs():
    """A stream's buffer grows to at least twice its size, but a device that has room for the call's need alone must serve the
    call (raw weights and the tiled schedule have no other memory; fp32 would fall to the scalar kernel)."""
    r = H.run("""
a = (F32, 1, 56, 56, 256, 64, 4)                   # row schedule
b = (F32, 1, 64, 64, 256, 64, 4)
first = [e for e in call('ex', *a, stream=16)[1] if e[0] == 'malloc']
need = [e for e in call('ex', *b, stream=32)[1] if e[0] == 'malloc']
tight = int(need[0][1])
st, ev = call('ex', *b, stream=16, limit=tight)
st2, ev2 = call('ex', *b, stream=16)
st3, ev3 = call('ex', BF16, 128, 7, 7, 2048, 512, 1, flags=16, stream=48)
big = [int(e[1]) for e in ev3 if e[0] == 'malloc'][0]
st4, ev4 = call('ex', BF16, 150, 7, 7, 2048, 512, 1, flags=16, stream=64)
big4 = [int(e[1]) for e in ev4 if e[0] == 'malloc'][0]
st5, ev5 = call('ex', BF16, 150, 7, 7, 2048, 512, 1, flags=16, stream=48, limit=big4)
result = [first, tight, [st, ev], [st2, ev2], big, big4, [st5, ev5]]
""")
    first, tight, (st, ev), (st2, ev2), big, big4, (st5, ev5) = r
    assert int(first[0][1]) < tight < 2 * int(first[0][1])
    assert st == 0 and [e[1:] for e in ev if e[0] == "malloc"] == [[str(2 * int(first[0][1])), "1"], [str(tight), "0"]]
    assert any("rows_conv2" in e[1] for e in ev)
    assert st2 == 0 and not [e for e in ev2 if e[0] == "malloc"]              # the buffer has that size now
    assert big < big4 < 2 * big
    assert st5 == 0 and [e[1:] for e in ev5 if e[0] == "malloc"] == [[str(2 * big), "1"], [str(big4), "0"]]


def test_no_memory_at_all():
    """fp32 then runs the kernel that needs none; a call whose weights have to be repacked is refused with nothing enqueued."""
    (st, ev), (st2, ev2) = H.run("""
result = [call('ex', F32, 1, 56, 56, 256, 64, 4, stream=16, limit=1024), call('ex', BF16, 2, 14, 14, 1024, 256, 2, stream=16, limit=1024)]
""")
    assert st == 0 and [H.kernel_name(e[1]) for e in ev if e[0] == "launch"][-1] == "bneck_generic_kernel"
    assert st2 == -5 and not [e for e in ev2 if e[0] in ("launch", "copy")]


def test_a_call_that_fails_has_enqueued_nothing():
    """The slab kernels' attributes are set with the others, before the repack, the copy and the first convolution."""
    st, ev = H.run("result = call('ex', BF16, 2, 14, 14, 1024, 256, 2, attr_fail=1)")
    assert st == -5
    assert not [e for e in ev if e[0] in ("launch", "copy")], ev


def test_no_launch_beyond_the_limit_of_threads():
    """fp32 maps of 1.1e9 pixels: a launch of 2^32 threads is an error, so the scalar kernel (whose grid is bounded) runs."""
    r = H.run("""
result = []
for N, h, w, C, M, S in ((1100, 1000, 1000, 4, 12, 1), (2000, 1000, 1000, 1, 8, 10), (1000, 1000, 1000, 4, 12, 1), (90000, 64, 32, 8, 2000, 1)):
    st, ev = call('ex', F32, N, h, w, C, M, S, flags=4)
    result.append([st, [[e[1], int(e[2]) * int(e[3])] for e in ev if e[0] == 'launch']])
""")
    for (st, launches), scalar in zip(r, (True, True, False, True)):
        assert st == 0 and launches and all(n < 1 << 32 for _, n in launches), launches
        assert (H.kernel_name(launches[0][0]) == "bneck_generic_kernel") == scalar


def test_planned_workspace_for_the_slab_schedule():
    """What the header says a caller has to bring: 4*N*H*W*M + 512 bytes, also for maps that the tiled schedule does not take (the
    query answers 0 there, and without a workspace the fused kernel runs); never more than the query's answer where it has one."""
    shapes = [(1, 25, 42, 2048, 512, 1), (1, 50, 60, 1024, 256, 2), (2, 14, 14, 1024, 256, 2), (3, 7, 7, 2048, 512, 1), (1, 1, 1, 2048, 512, 1)]
    r = H.run("""
result = []
for N, h, w, C, M, S in %r:
    q, need = L.lasnet_workspace_bytes(BF16, N, h, w, C, M, S), 4 * N * h * w * M + 512
    runs = [[st, kernels(ev), [e for e in ev if e[0] == 'malloc']] for st, ev in
            (call('planned', BF16, N, h, w, C, M, S, flags=4, ws=b, capturing=c) for b in ((need, 0) if q == 0 else (q,)) for c in (0, 1))]
    result.append([q, need, runs])
""" % shapes)
    for shape, (q, need, runs) in zip(shapes, r):
        assert q == 0 or q + 512 >= need
        assert (q == 0) == (shape[1] * shape[2] > (196 if shape[3] == 1024 else 49))
        for i, (st, names, mallocs) in enumerate(runs):
            assert st == 0 and not mallocs
            assert all(("slab" if i < 2 else "fused") in n for n in names), (shape, names)
