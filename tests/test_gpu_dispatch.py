"""Shapes at which AJ_KERNEL_AUTO must not take the small tiles: the kernel that served them before is the faster one there
(times, small tiles and that kernel, in us)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,d,V,kernel", [
    (264, 7168, 21700, "pair5"),       # 178, 137 (wide kernel 186): 85 tiles in three row tiles are 33 on an XCD of 32 compute units
    (264, 1024, 21700, "pair5"),       # 36, 31 (wide kernel 44)
    (144, 8192, 72000, "wide"),        # 340, 334
    (2, 8192, 100000, "resident"),     # 294, 248: the smallest tiles stream W_lm at 5.7 TB/s here
    (16, 8192, 90000, "resident"),     # 262, 244
    (2, 3072, 100000, "resident"),     # 106, 102
    (2000, 72, 100000, "tile"),        # 208, 142: in short rows the reduction of a tile outweighs its loop
    (128, 264, 50257, "tile"),         # 24.9, 23.0
    (128, 64, 128256, "tall"),         # 32.8, 24.7
    (128, 352, 128256, "big"),         # 1.06 of the time
    (128, 4160, 128256, "big"),        # 257, 244
    (100, 256, 152064, "resident"),    # 46.0, 35.8
    (64, 256, 65536, "resident"),      # 20.6, 19.7
])
def test_kernel_of_shape(M, d, V, kernel):
    import paper_2504_20039_amd as aj
    h = aj.aj_create(M // 2 if M > 1024 else 1, 1 if M > 1024 else M - 1, d, 0, V, aj.AJ_BF16)
    name = aj.aj_kernel_name(h)
    aj.aj_destroy(h)
    assert name == f"lm_head_{kernel}_bf16"


@pytest.mark.parametrize("M,d,V,fp8,waves", [
    (45, 2048, 65130, False, 4),       # 53.5 with 16, 50.6
    (38, 4096, 62914, False, 4),       # 87, 84
    (45, 2048, 60000, False, 16),
    (62, 8192, 65536, False, 16),
    (96, 4096, 32312, True, 4),        # 50.5 with 8, 46.7
    (30, 2048, 78643, True, None),     # 45.8, 42.8: the accumulator-resident kernel
    (30, 2048, 66000, True, 4),
])
def test_waves_of_shape(M, d, V, fp8, waves):
    import paper_2504_20039_amd as aj
    h = aj.aj_create(1, M - 1, d, 0, V, aj.AJ_BF16, 1, 0, 0, aj.AJ_W_FP8_E4M3 if fp8 else aj.AJ_W_SAME)
    name = aj.aj_kernel_name(h)
    form = aj.aj_debug_form(h) if "slab" in name else None
    aj.aj_destroy(h)
    assert (form[0] if form else None) == waves and ("slab" in name or name == "lm_head_resident_fp8w")
