"""Convolution plans on a device made of host memory (tests/sanitize/device_stubs.cpp): what a plan allocates and what it does
without memory for it.  Runs in the child of tests/test_sanitize_host.py; elsewhere there is no such device."""
import pytest

import bcr_inputs as gen
import paper_2108_11033_amd as g


@pytest.fixture
def device():
    lib = g.load_library()
    if not hasattr(lib, "grim_stub_device"):
        pytest.skip("the library of this process runs on a GPU")
    lib.grim_stub_device(1, -1)
    yield lib
    lib.grim_stub_device(0, -1)


@pytest.fixture
def rules(device):
    """With the library's own rules for the convolutions' launch forms."""
    device.grim_stub_conv_rules(1)
    yield device
    device.grim_stub_conv_rules(0)


def _matrix(M, K, BR, BC, kr, kc):
    mask = gen.random_mask(M, K, BR, BC, kr, kc, seed=M + K)
    W = gen.normal_weights(M, K, gen.F16, seed=3)
    return g.pack(W, gen.F16, BR, BC, mask.row_ptr, mask.row_idx, mask.col_ptr, mask.col_idx)


def test_a_plan_without_memory_for_the_layout_of_64_row_runs(device):
    """4 x 16 blocks at stride 2 ask for the second layout; its allocation failing leaves a plan on the 16-row runs."""
    A = _matrix(128, 64 * 9, 4, 16, 2, 4)
    live = device.grim_stub_live_allocations()
    plan = g.ConvPlan(A, 64, 28, 28, 3, 3, 2)
    assert device.grim_stub_live_allocations() == live + 2
    del plan
    assert device.grim_stub_live_allocations() == live
    device.grim_stub_device(1, 1)
    plan = g.ConvPlan(A, 64, 28, 28, 3, 3, 2)
    assert device.grim_stub_live_allocations() == live + 1
    del plan
    device.grim_stub_device(1, 0)
    with pytest.raises(g.GrimError) as e:
        g.ConvPlan(A, 64, 28, 28, 3, 3, 2)
    assert e.value.name == "GRIM_ERR_ALLOC"
    device.grim_stub_device(1, -1)
    A.free()


@pytest.mark.parametrize("M,cin,BR,BC,kr,kc,stride", [
    (128, 512, 16, 32, 16, 2, 2),      # runs of 64 rows would name nearly as many columns as four of 16
    (16, 32, 4, 16, 2, 4, 2),          # a single 16-row run
    (128, 32, 4, 16, 2, 4, 1),         # stride 1: too few steps
])
def test_a_plan_holds_no_layout_it_cannot_use(device, M, cin, BR, BC, kr, kc, stride):
    A = _matrix(M, cin * 9, BR, BC, kr, kc)
    live = device.grim_stub_live_allocations()
    plan = g.ConvPlan(A, cin, 28, 28, 3, 3, stride)
    assert device.grim_stub_live_allocations() == live + 1
    del plan
    A.free()


@pytest.mark.parametrize("octets", [4, 2, 1])
@pytest.mark.parametrize("M,cin,BR,BC,k", [(128, 64, 4, 16, 3), (40, 36, 8, 12, 3), (80, 20, 16, 20, 5), (64, 12, 64, 4, 3)])
def test_a_plan_with_a_dense_copy_and_without_memory_for_it(device, octets, M, cin, BR, BC, k):
    """A last run that is not full and channels that fill no chunk are written inside the copy (this runs under the address
    sanitizer); its allocation failing leaves a plan without it."""
    A = _matrix(M, cin * k * k, BR, BC, (BR // 2, BR), (BC // 2, BC))
    device.grim_stub_patch_octets(octets)
    try:
        live = device.grim_stub_live_allocations()
        plan = g.ConvPlan(A, cin, 28, 28, k, k, 2)
        assert device.grim_stub_live_allocations() >= live + 2
        del plan
        assert device.grim_stub_live_allocations() == live
        device.grim_stub_device(1, 1)
        plan = g.ConvPlan(A, cin, 28, 28, k, k, 2)
        assert device.grim_stub_live_allocations() == live + 1
        del plan
    finally:
        device.grim_stub_patch_octets(0)
        device.grim_stub_device(1, -1)
    A.free()


@pytest.mark.parametrize("cin,BC,k,batch,stride,kernel", [
    (256, 16, 3, 4, 1, "bcr_conv_patch"),
    (256, 16, 3, 16, 2, "bcr_conv_patch"),
    (258, 18, 3, 4, 1, "bcr_conv_tall"),         # channels that are no whole fours
    (768, 16, 1, 16, 1, "bcr_conv_tall"),
    (256, 16, 3, 1, 1, "bcr_conv_gather"),       # one image: the bits of the unplanned call
])
def test_the_kernel_a_plan_names(rules, cin, BC, k, batch, stride, kernel):
    A = _matrix(256, cin * k * k, 4, BC, 2, 4)
    assert g.conv2d_kernel_name(A, cin, 28, 28, k, k, batch, stride) == kernel
    A.free()
