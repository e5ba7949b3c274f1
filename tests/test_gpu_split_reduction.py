"""conv_ksplit_kernel, whose waves split the reduction (3x3, 96 channels and more, int8 120), through small nets against the CPU oracle
(bf16) and bit for bit against the integer oracle (int8); and which of its tile shapes the nets reach, on the CPU."""
import pytest

from tests.fake_hip import run
from tests.test_gpu_layer_kernels import _chain, _check_dense

# Chunks of eight cells that end inside a cell pair (104, 120, 200, 264 channels; int8: inside a cell), the shortest reductions (96;
# int8: 120, 128), filters that end inside a tile of 32, 64 and 96; maps of 8 x 8 (tiles over three images) to 29 x 29, ragged last tiles; one image; every tile shape
NETS = [(_chain([8, 120, 136, 40], 9), 1), (_chain([16, 264, 200], 15), 3), (_chain([8, 136, 120], 29), 5), (_chain([8, 200, 264, 24], 8), 7), (_chain([16, 360, 328], 14), 17),
        (_chain([16, 360, 360], 14), 24), (_chain([16, 520, 200], 8), 33), (_chain([8, 112, 112], 21), 30), (_chain([8, 96, 104], 21), 30), (_chain([8, 96, 128, 128], 28), 4)]


@pytest.mark.gpu
@pytest.mark.parametrize("arch,batch", NETS)
@pytest.mark.parametrize("int8", [False, True])
def test_split_reduction(arch, batch, int8):
    _check_dense(arch, batch, int8)


def test_nets_reach_every_tile_shape(tmp_path):
    out = run(tmp_path, '''
for dtype in ("bf16", "int8"):
    seen = set()
    for arch, batch in DATA:
        seen |= {tuple(k[1][1:]) for o, k in layers(arch, dtype, batch) if k[0] == "conv_ksplit_kernel"}
    print(sorted(seen))
''', NETS)
    assert out.splitlines() == [str([(1, 1), (1, 2), (2, 2), (2, 4), (3, 2)])] * 2, out
