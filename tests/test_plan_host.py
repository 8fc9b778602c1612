"""Which kernel, rows per workgroup and split each layer of the five baseline configurations takes, on a 256-CU device,
through the C ABI's plan query (host code only: no GPU needed).  A change of the launch planner shows up here.  Storage 0: as an
arbitrary table of 16-bit entries would run; storage 2: as the configurations' own tables do, which have a byte form."""
import pytest

QUAD, XMAJOR, FAST, GENERIC, ROWS = 3, 2, 1, 0, -1


@pytest.fixture(scope="module")
def plan():
    from paper_2203_04071_amd import binding as B
    B.load()
    return lambda *a: B.adapt_plan_packed(*a, 256)


def test_headline_layer_runs_on_the_quad_kernel_unsplit(plan):
    # config 2: 3x3 s1 p1, batch 32, 64 -> 64 channels, 32x32: 32768 rows, 9 taps x 4 steps of 16 channels
    kernel, rows, ksplit, steps, wgs = plan(1, 8, 0, 64, 64, 3, 3, 1, 32 * 32 * 32, 32, 1)
    assert (kernel, rows, ksplit, steps, wgs) == (QUAD, 1024, 1, 36, 256)


def test_resnet20_layers(plan):
    # first layer: 3 channels (padded to 8): no quad tables; x-major copy, 128-byte lines, paired taps
    assert plan(1, 8, 0, 16, 3, 3, 3, 1, 128 * 32 * 32, 32, 1)[:3] == (XMAJOR, 1024, 1)
    # stage 1: 16 channels, 9 steps of 16, 131072 rows x 2 channel tiles: quad kernel, 4 rows per row slot, 256 workgroups
    assert plan(1, 8, 0, 16, 16, 3, 3, 1, 128 * 32 * 32, 32, 1) == (QUAD, 1024, 1, 9, 256)
    # a 1x1 layer of 32 channels has 2 steps: below the quad kernel's minimum of 4
    assert plan(1, 8, 0, 16, 32, 1, 1, 1, 128 * 32 * 32, 32, 1)[0] != QUAD
    # stage 2: 32 channels, 32768 rows: unsplit the quad kernel would cover half the compute units: 2 slices of 9 steps
    assert plan(1, 8, 0, 32, 32, 3, 3, 1, 128 * 16 * 16, 16, 1) == (QUAD, 1024, 2, 18, 256)
    # stage 3: 64 channels, 8192 rows: a quarter of the compute units: 4 slices of 9 steps
    assert plan(1, 8, 0, 64, 64, 3, 3, 1, 128 * 8 * 8, 8, 1) == (QUAD, 1024, 4, 36, 256)
    # too few steps to slice (a 1x1 layer of 64 channels, 4 steps, on a quarter of the chip): 128-byte-line kernels
    assert plan(1, 8, 0, 64, 64, 1, 1, 1, 128 * 8 * 8, 8, 1)[0] != QUAD
    # stride-2 layers never take the x-major copy
    assert plan(1, 8, 0, 32, 16, 3, 3, 1, 128 * 16 * 16, 16, 2)[0] in (FAST, GENERIC)
    assert plan(1, 8, 0, 64, 32, 3, 3, 1, 128 * 8 * 8, 8, 2)[0] in (FAST, GENERIC)
    # final linear layer, 128 rows: whole-table kernel
    assert plan(0, 8, 0, 10, 64, 1, 1, 1, 128, 128, 1)[0] == ROWS


def test_lstm_layers(plan):
    # input products of all time steps: 6400 rows x 512 -> 2048, 7-bit table: quad kernel, 2048 rows per workgroup
    k, rows, ksplit, steps, wgs = plan(0, 7, 0, 2048, 512, 1, 1, 1, 100 * 64, 100 * 64, 1)
    assert (k, rows, ksplit, steps) == (QUAD, 2048, 1, 32) and wgs == 4 * 256
    # one time step of the recurrence: 64 rows: whole-table kernel
    assert plan(0, 7, 0, 2048, 512, 1, 1, 1, 64, 64, 1)[0] == ROWS


@pytest.mark.parametrize("bits", [6, 8])
def test_generator_layers(plan, bits):
    # stride-2 4x4 transposed convolutions = 4 phases of 2x2 taps; rows per phase = batch x input pixels
    for cin, cout, hw in ((512, 256, 4), (256, 128, 8), (128, 64, 16), (64, 3, 32)):
        k, rows, ksplit, steps, wgs = plan(2, bits, 0, cout, cin, 4, 4, 2, 256 * hw * hw, hw, 1)
        assert (k, rows, ksplit, steps) == (QUAD, 2048, 1, 4 * cin // 16), (cin, cout)
        assert wgs == (256 * hw * hw // 2048) * ((cout + 7) // 8) * 4


def test_two_pass_tables_stay_off_the_quad_kernel(plan):
    assert plan(1, 8, 1, 64, 64, 3, 3, 1, 32 * 32 * 32, 32, 1)[0] != QUAD


def test_bad_arguments(plan):
    from paper_2203_04071_amd import binding as B
    with pytest.raises(B.AdaptError):
        plan(3, 8, 0, 64, 64, 3, 3, 1, 1024, 32, 1)
    with pytest.raises(B.AdaptError):
        plan(1, 9, 0, 64, 64, 3, 3, 1, 1024, 32, 1)


BYTE = 4


@pytest.mark.parametrize("bits,K,N,first_byte", [(8, 777, 999, 512), (8, 4096, 4096, 1024), (8, 4096, 64, 16), (7, 1024, 512, 512), (8, 64, 10, 4096)])
def test_linear_layers_with_byte_tables_change_kernel_once(plan, bits, K, N, first_byte):
    # from `first_byte` rows (of powers of two) on the derived tables are streamed; below, the whole-table kernel is faster
    for rows in (16, 64, 128, 256, 512, 1024, 2048, 4096, 16384):
        kernel, per_wg, ksplit, steps, wgs = plan(0, bits, 2, N, K, 1, 1, 1, rows, rows, 1)
        assert kernel == (BYTE if rows >= first_byte else ROWS)
        if kernel == BYTE:
            assert wgs == -(-rows // per_wg) * -(-N // 16) * ksplit


def test_handles_whose_inner_dimension_is_too_long_for_the_byte_kernel(plan):
    # its table of group offsets holds 2040 steps of 16 inner indices; longer products keep the other tables
    assert plan(0, 8, 2, 64, 32640, 1, 1, 1, 8192, 8192, 1)[::3] == (BYTE, 2040)
    for K in (32641, 32644, 40000):
        assert plan(0, 8, 2, 64, K, 1, 1, 1, 8192, 8192, 1) == plan(0, 8, 0, 64, K, 1, 1, 1, 8192, 8192, 1)
        assert plan(0, 8, 2, 64, K, 1, 1, 1, 1024, 1024, 1)[0] == ROWS
    # transposed: a phase counts, and strides above 8 have none
    assert plan(2, 8, 2, 64, 4080, 4, 4, 2, 4096, 32, 1)[0] == plan(2, 8, 2, 64, 8160, 4, 4, 2, 4096, 32, 1)[0] == BYTE
    assert plan(2, 8, 2, 64, 8164, 4, 4, 2, 4096, 32, 1) == plan(2, 8, 0, 64, 8164, 4, 4, 2, 4096, 32, 1)
    assert plan(2, 8, 2, 16, 16, 18, 18, 9, 4096, 32, 1)[0] == ROWS


def test_layers_of_the_configurations_on_their_own_tables(plan):
    # config 2: two slices of 18 steps; 1024 rows per workgroup
    assert plan(1, 8, 2, 64, 64, 3, 3, 1, 32 * 32 * 32, 32, 1) == (BYTE, 1024, 2, 36, 256)
    # config 3: every convolution fills the chip, the later stages by slices; the final linear layer stays on the whole table
    for cout, cin, hw, stride, ksplit, steps in ((16, 3, 32, 1, 1, 3), (16, 16, 32, 1, 1, 9), (32, 16, 16, 2, 2, 9), (32, 32, 16, 1, 2, 18),
                                                 (64, 32, 8, 2, 4, 18), (64, 64, 8, 1, 4, 36)):
        assert plan(1, 8, 2, cout, cin, 3, 3, 1, 128 * hw * hw, hw, stride) == (BYTE, 512, ksplit, steps, 256)
    assert plan(0, 8, 2, 10, 64, 1, 1, 1, 128, 128, 1)[0] == ROWS
    # config 4: input products of all steps; one step of the recurrence
    assert plan(0, 7, 2, 2048, 512, 1, 1, 1, 100 * 64, 100 * 64, 1) == (BYTE, 2048, 1, 32, 512)
    assert plan(0, 7, 2, 2048, 512, 1, 1, 1, 64, 64, 1)[0] == ROWS
    # config 5: 2048 rows per workgroup, the first layer in two slices
    for bits in (6, 8):
        for cin, cout, hw, ksplit in ((512, 256, 4, 2), (256, 128, 8, 1), (128, 64, 16, 1), (64, 3, 32, 1)):
            assert plan(2, bits, 2, cout, cin, 4, 4, 2, 256 * hw * hw, hw, 1)[:4] == (BYTE, 2048, ksplit, 4 * cin // 16)
