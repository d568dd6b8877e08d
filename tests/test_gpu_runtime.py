"""The library's device-memory handling on the GPU: a rule book freed while
another stream still reads it, and the release of cached blocks."""
import numpy as np
import pytest
import torch

from oracle import sscn_oracle as O
from paper_1711_10275_amd import sscn
from paper_1711_10275_amd import synthetic as S
from tests.gpu_common import coords_for, dev, host
from tests.parity import assert_close

pytestmark = pytest.mark.gpu


def test_free_while_another_stream_reads():
    """Build on stream A, run the forward on stream B, free the rule book at
    once and rebuild (a row-shuffled set of the same size, so the freed
    blocks are handed out again and rewritten) on A.  The freed storage goes
    back to A's cache only after B's reads: every forward must still match
    the oracle."""
    coords, size = coords_for("shapes128")
    shuf = S.shuffled(coords, 5)
    X, W = S.features(coords.shape[0], 16, 91), S.weights(27, 16, 16, 92)
    ref = O.forward(X, W, O.ssc_rulebook(coords, size, 3))
    tc, ts, tX, tW = dev(coords), dev(shuf), dev(X), dev(W)
    A, B = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    outs, keep = [], []
    for _ in range(4):
        with torch.cuda.stream(A):
            rb = sscn.ssc_rulebook_build(tc, size, 3)
        B.wait_stream(A)
        with torch.cuda.stream(B):
            outs.append(sscn.sparse_conv_forward(tX, tW, rb))
        rb.free()
        with torch.cuda.stream(A):
            keep.append(sscn.ssc_rulebook_build(ts, size, 3))
    torch.cuda.synchronize()
    for y in outs:
        assert_close(host(y), ref, "f32", "forward on the reading stream")
    # the rule books built after each free are intact too
    rs = O.ssc_rulebook(shuf, size, 3)
    assert all(k.n_pairs == rs.n_pairs() for k in keep)


def test_release_cached_blocks():
    coords, size = coords_for("shell32")
    X, W = S.features(coords.shape[0], 8, 93), S.weights(27, 8, 8, 94)
    ref = O.forward(X, W, O.ssc_rulebook(coords, size, 3))
    for _ in range(3):
        rb = sscn.ssc_rulebook_build(dev(coords), size, 3)
        y = sscn.sparse_conv_forward(dev(X), dev(W), rb)
        rb.free()
        sscn.release_cached()
        assert_close(host(y), ref, "f32", "after release")


def test_affine_relu_rejects_bad_out():
    x = torch.zeros((10, 4), device="cuda:0")
    s = torch.ones(4, device="cuda:0")
    with pytest.raises(ValueError):
        sscn.affine_relu(x, s, s, out=torch.empty((5, 4), device="cuda:0"))
    with pytest.raises(ValueError):
        sscn.affine_relu(x, s, s, out=torch.empty((10, 3), device="cuda:0"))
    with pytest.raises(ValueError):
        sscn.affine_relu(x, torch.ones(4), s)


def test_kernel_timer_brackets_the_row_kernel():
    """sscn_time_next_launch: the armed events bracket the next row-block
    launch only (a forward's weight copy stays outside), once."""
    coords, size = coords_for("shapes128")
    rb = sscn.ssc_rulebook_build(dev(coords), size, 3)
    X, W = dev(S.features(coords.shape[0], 64, 95)), dev(S.weights(27, 64, 64, 96))
    sscn.sparse_conv_forward(X, W, rb)
    t = sscn.KernelTimer()
    t.arm()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    sscn.sparse_conv_forward(X, W, rb)
    e1.record()
    torch.cuda.synchronize()
    kernel_ms, call_ms = t.ms(), e0.elapsed_time(e1)
    assert 0.0 < kernel_ms <= call_ms
    # used once: a later call leaves the events where they were
    sscn.sparse_conv_forward(X, W, rb)
    torch.cuda.synchronize()
    assert t.ms() == kernel_ms


@pytest.mark.parametrize("dtype,cin,cout", [(torch.bfloat16, 32, 20), (torch.float32, 8, 6), (torch.float32, 32, 20)])
def test_kernel_timer_brackets_a_per_site_layer(dtype, cin, cout):
    """The same of a filter-size-1 layer, whether the row-block kernel runs it or
    the per-site kernel in its place: the forward takes the request, and a wgrad
    after it finds none."""
    coords, size = coords_for("shell32")
    rb = sscn.ssc_rulebook_build(dev(coords), size, 1)
    n = coords.shape[0]
    X, W, G = (dev(a, dtype) for a in (S.features(n, cin, 97), S.weights(1, cin, cout, 98), S.features(n, cout, 99)))
    t = sscn.KernelTimer()
    t.arm()
    sscn.sparse_conv_forward(X, W, rb)
    torch.cuda.synchronize()
    kernel_ms = t.ms()
    assert kernel_ms > 0.0
    sscn.sparse_conv_backward(X, W, G, rb, dgrad=False)
    torch.cuda.synchronize()
    assert t.ms() == kernel_ms


def test_device_memory_cap_gives_oom_and_recovers():
    """A cap on the library's device memory below what a build needs makes
    the build fail with the out-of-memory status (after the idle blocks are
    released, as on a real failure), and leaves the library usable: without
    the cap the same build succeeds with the oracle's pair count."""
    coords, size = coords_for("shapes128")
    tc = dev(coords)
    sscn.release_cached()  # no idle block of earlier tests serves the build
    try:
        sscn.set_device_memory_cap(1 << 20)
        with pytest.raises(sscn.SSCNError) as err:
            sscn.ssc_rulebook_build(tc, size, 3)
        assert err.value.code == "oom"
    finally:
        sscn.set_device_memory_cap(0)
    rb = sscn.ssc_rulebook_build(tc, size, 3)
    orb = O.ssc_rulebook(coords, size, 3)
    assert rb.n_pairs == sum(len(x) for x in orb.outs)
