"""The work bench.py counts for the layer algorithm, against closed forms (no GPU)."""
import bench


def test_layer_flops_per_point():
    # one layer of n = 3 gates, 8 amplitudes: a gate's products forward 4 x 14 and back 8 x 4, its S_x and S_y 32;
    # the layer's conjugate phase 8 x 6 and diagonal products 4 x 4
    assert bench.layer_flops_per_point(3, 3) == 8 * (3 * (56 + 32 + 32) + 48 + 16)
    # a folded opening layer is neither applied nor undone, its sums remain
    assert bench.layer_flops_per_point(3, 3, 3) == 8 * (3 * 32 + 16)
    # 12 qubits, 8 layers, the opening one folded
    assert bench.layer_flops_per_point(96, 12, 12) == 4096 * (84 * 88 + 96 * 32 + 7 * 48 + 8 * 16)
    assert bench.layer_flops_per_point(96, 12, 12) < bench.executed_flops_per_point(96, 12, 12)


def test_matrix_core_share():
    assert bench.matrix_core_share(3, 0, 3) == 3 * 56 / (3 * 120 + 64)
    assert bench.matrix_core_share(96, 12, 12) == 84 * 56 / (84 * 88 + 96 * 32 + 7 * 48 + 8 * 16)
    assert bench.matrix_core_share(3, 3, 3) == 0.0
    assert bench.matrix_core_share(0) == 0.0
