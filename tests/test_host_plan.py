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


MIXED_32 = ((4, 8, 16), (4, 8, 16))


@pytest.mark.parametrize("cin,M,H,W,k,stride,batch,BR,BC,keep,dense", [
    # microseconds without and on the dense copy
    (224, 160, 47, 47, 3, 1, 8, 32, 32, MIXED_32, False),        # 29.0, 39.9
    (288, 224, 17, 17, 3, 1, 26, 16, 32, (8, 8), False),         # 25.2, 34.4: a few workgroups behind a full round
    (160, 192, 56, 56, 3, 2, 5, 16, 32, (8, 8), False),          # 11.0, 13.2
    (320, 384, 35, 35, 3, 1, 5, 16, 32, (8, 8), False),          # 31.6, 38.7
    (320, 64, 51, 41, 3, 1, 3, 8, 16, (4, 4), False),            # 14.3, 17.4
    (128, 288, 59, 59, 3, 2, 3, 32, 32, MIXED_32, False),        # 10.5, 12.2
    (320, 224, 8, 8, 3, 2, 7, 4, 16, (2, 4), False),             # 8.9, 12.7: 32-position tiles
    (256, 128, 10, 10, 3, 2, 4, 16, 16, (4, 8), False),          # 7.6, 9.5
    (128, 128, 35, 8, 5, 2, 4, 4, 16, (2, 4), False),            # 9.3, 13.0
    (384, 384, 68, 68, 3, 1, 4, 16, 32, (8, 8), False),          # 74.7, 86.4: a strip to a wave
    (256, 256, 28, 28, 3, 1, 4, 16, 32, (8, 8), True),           # 13.7, 11.2
    (448, 448, 103, 24, 3, 2, 7, 16, 32, (8, 8), True),          # 82.1, 36.1
    (512, 512, 14, 14, 3, 1, 8, 16, 32, (8, 8), True),           # 19.3, 17.4
    (192, 192, 18, 18, 5, 1, 4, 32, 32, (8, 16), True),          # 20.4, 18.9
    (32, 128, 28, 28, 3, 1, 24, 4, 16, (2, 4), True),            # 18.4, 12.5
])
def test_the_dense_copy_is_taken_where_it_is_quicker(rules, cin, M, H, W, k, stride, batch, BR, BC, keep, dense):
    A = _matrix(M, cin * k * k, BR, BC, *keep)
    assert (g.conv2d_kernel_name(A, cin, H, W, k, k, batch, stride) == "bcr_conv_patch") == dense
    A.free()


@pytest.mark.parametrize("cin,M,H,W,stride,BR,BC,keep,kernel,batch", [
    (64, 224, 7, 7, 1, 32, 32, (8, 8), "bcr_conv_patch", 83),            # to 128
    (32, 64, 46, 11, 2, 16, 32, (8, 8), "bcr_conv_patch", 77),           # to 85
    (64, 256, 16, 4, 2, 32, 32, MIXED_32, "bcr_conv_tall", 65),          # to 128; on the dense copy before and after
    (64, 256, 4, 35, 2, 32, 32, (8, 8), "bcr_conv_tall", 65),            # and all larger ones
    (192, 64, 9, 9, 2, 32, 32, MIXED_32, "bcr_conv_patch", 129),
])
def test_a_plan_holds_the_layouts_of_batches_above_64(rules, cin, M, H, W, stride, BR, BC, keep, kernel, batch):
    """A few batches, or all from some number on, run on a layout that smaller ones do not use."""
    A = _matrix(M, cin * 9, BR, BC, *keep)
    names = [g.conv2d_kernel_name(A, cin, H, W, 3, 3, b, stride) for b in list(range(1, 65)) + [batch]]
    assert kernel not in names[:64] and names[64] == kernel
    live = rules.grim_stub_live_allocations()
    plan = g.ConvPlan(A, cin, H, W, 3, 3, stride)
    assert rules.grim_stub_live_allocations() == live + 1 + len({"bcr_conv_patch", "bcr_conv_tall"} & set(names))
    del plan
    A.free()
