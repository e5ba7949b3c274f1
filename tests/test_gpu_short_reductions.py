"""1x1 layers of at most 128 channels, which go to the small, the tile or the patch kernel by filters and pixels: small nets against
the CPU oracle, and which kernels their layers reach, on the CPU."""
import pytest

from tests.fake_hip import run
from tests.test_gpu_layer_kernels import _bottleneck, _check_dense

# pixels on both sides of 32768 (42 and 41 images of 28 x 28), 16 and 24 filters, residuals, filters of a 96-wide tile, ragged last tiles
NETS = [(_bottleneck([64, 96], [1, 1], 112, 0.25), 42), (_bottleneck([64, 96], [1, 1], 112, 0.25), 41), (_bottleneck([128, 72], [1, 1], 108, 0.125), 50)]


@pytest.mark.gpu
@pytest.mark.parametrize("arch,batch", NETS)
def test_short_reductions(arch, batch):
    _check_dense(arch, batch, False)


def test_kernel_of_each_layer(tmp_path):
    out = run(tmp_path, '''
for arch, batch in DATA:
    print(batch, sorted({"%d-%d%s %s" % (o["C"], o["K"], "r" if o["res"] else "", k[0][5:-7]) for o, k in layers(arch, "bf16", batch)
                         if o["kind"] == 0 and o["R"] == 1 and o["stride"] == 1 and o["C"] <= 128 and o["K"] != 24}))
''', NETS + [(_bottleneck([64, 192], [1, 1], 224, 0.25), n) for n in (168, 167)])  # 526848 and 523712 pixels: of either side of 2^19
    small = ["24-16 small", "64-16 small"]
    assert out.splitlines() == [
        "42 %s" % sorted(["16-64r tile", "24-64 tile", "24-96r tile", "64-96 patch"] + small),
        "41 %s" % sorted(["16-64r tile", "24-64 tile", "24-96r tile", "64-96 tile"] + small),
        "50 %s" % sorted(["16-72r tile", "16-128r tile", "24-128 tile", "128-72 patch", "24-16 small", "72-16 small", "128-16 small"]),
        "168 %s" % sorted(["16-64r tile", "24-64 tile", "48-192r tile", "64-192 patch", "64-48 tile"] + small),
        "167 %s" % sorted(["16-64r tile", "24-64 tile", "48-192r tile", "64-192 tile", "64-48 tile"] + small)], out
