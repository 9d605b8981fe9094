"""The decode plan (host arithmetic): well-formed for every shape, and covered by the workspace of any larger cache."""
import pytest

from tests import gpu_util as U

HEAD = 64 * 1024 + 256       # control words at the head of a workspace (keepkv.h)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("units", [1, 8, 40, 64, 256, 513, 1000])
def test_plan_and_workspace(units, G, D, dtype):
    kk = U.kk()
    bf16 = dtype == "bf16"
    lay = kk.Layout(units, G, 1, D, kk.BF16 if bf16 else kk.F32, 0.1)
    for cap in (1, 31, 64, 65, 500, 884, 4100, 32768, 1 << 20):
        ns, per, waves = kk.decode_plan(lay, cap)
        assert per % (32 if bf16 else 64) == 0 and per >= 64 and waves in ((4, 8) if bf16 else (4,))
        assert ns == -(-cap // per) and (ns == 1 or ns * units <= (512 if bf16 else 2048))
    for largest in (100, 600, 900, 5000, 16384, 32768):
        have = kk.workspace_bytes(lay, largest, max(1, largest // 10))
        for cap in range(1, largest + 1, max(1, largest // 61)):
            ns = kk.decode_plan(lay, cap)[0]
            assert ns == 1 or HEAD + units * G * ns * (D + 2) * 4 <= have, (largest, cap)


def test_combining_is_priced_per_output_element():
    """One long head: eight query heads give a thread two output elements to combine, so it is split less than one."""
    kk = U.kk()
    for cap in (50000, 100000):
        few, many = (kk.decode_plan(kk.Layout(1, g, 1, 128, kk.BF16, 0.1), cap)[0] for g in (8, 1))
        assert 16 < few < many


def test_layouts_without_a_kernel_still_get_a_size():
    kk = U.kk()
    assert kk.workspace_bytes(kk.Layout(2, 6, 2, 4096, kk.BF16, 0.1), 1000, 100) > HEAD
