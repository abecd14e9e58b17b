"""Which kernel a layer takes where several can (no GPU needed: the rules are host functions of the library).
Each layer below was measured on both; the figures (us per call) are those of the two kernels on MI355X."""
import ctypes

import pytest

F32, BF16 = 0, 1


class TailArgs(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in ("B", "F_s", "L", "G", "F_in")] + [("dtype", ctypes.c_int32)]


def rule(name, shape, dtype):
    from paper_2606_01117_amd import lib
    fn = getattr(lib, f"_ZN5haste{len(name)}{name}ERKNS_8TailArgsE")   # haste::name(const TailArgs &)
    fn.restype = ctypes.c_bool
    return fn(ctypes.byref(TailArgs(*shape, dtype)))


# rule, (B, F_s, L, G, F_in), dtype, taken
FWD = [
    # few slots, rows or features: 34.3 against 8.2 on the vector ALUs, 31.6 and 7.0, 39.7 and 10.0, 320 and 47.2
    ("fwd_any_preferred", (4, 128, 334464, 16, 8), BF16, False),
    ("fwd_any_preferred", (1, 128, 297914, 2, 8), BF16, False),
    ("fwd_any_preferred", (4, 152, 399862, 2, 8), BF16, False),
    ("fwd_f32_preferred", (168, 128, 194244, 3, 8), F32, False),
    # few labels for the rows, on the kernels of small groups: 21.0 against 12.6, 26.2 and 17.9
    ("fwd_any_preferred", (1606, 128, 2432, 8, 128), BF16, False),
    ("fwd_any_preferred", (879, 128, 4346, 2, 128), BF16, False),
    # large layers, and a ragged one
    ("fwd_any_preferred", (256, 768, 655360, 1, 64), BF16, True),
    ("fwd_any_preferred", (256, 768, 655360, 4, 64), BF16, True),
    ("fwd_any_preferred", (256, 768, 131072, 32, 256), BF16, True),
    ("fwd_any_preferred", (77, 500, 65544, 24, 48), BF16, True),
    ("fwd_f32_preferred", (128, 768, 131072, 16, 64), F32, True),
    ("fwd_f32_preferred", (32, 256, 4096, 8, 32), F32, True),
    # supports whose lines the L2 does not keep on the vector ALUs: 204 there, 41 here
    ("fwd_any_preferred", (1, 256, 187422, 1, 69), BF16, True),
]

BWD_W = [
    # one to three labels a group, few slots or rows: 210 against 16.2 on the vector ALUs, 112 and 29.6, 598 and 364,
    # 307 and 56.1
    ("bwd_w_any_preferred", (17, 128, 195575, 1, 8), BF16, False),
    ("bwd_w_any_preferred", (16, 768, 98304, 1, 20), BF16, False),
    ("bwd_w_any_preferred", (256, 768, 98304, 1, 20), BF16, False),
    ("bwd_w_f32_preferred", (168, 128, 194244, 3, 8), F32, False),
    # 460 against 998, and the large layers
    ("bwd_w_any_preferred", (64, 768, 98304, 1, 256), BF16, True),
    ("bwd_w_any_preferred", (256, 768, 131072, 32, 256), BF16, True),
    ("bwd_w_any_preferred", (77, 500, 65544, 24, 48), BF16, True),
    ("bwd_w_f32_preferred", (128, 768, 131072, 16, 64), F32, True),
    ("bwd_w_f32_preferred", (32, 256, 4096, 8, 32), F32, True),
]

BWD_X = [
    # few large groups: 155 against 52.6 on the vector ALUs, 119 and 56.0
    ("bwd_x_f32_preferred", (275, 256, 952, 119, 195), F32, False),
    ("bwd_x_f32_preferred", (104, 486, 1356, 113, 253), F32, False),
    # 65.1 against 43.8 in LDS accumulators, 45.8 and 38.1
    ("bwd_x_any_preferred", (440, 512, 51228, 12, 32), BF16, False),
    ("bwd_x_any_preferred", (293, 768, 23104, 32, 128), BF16, False),
    # the large layers
    ("bwd_x_any_preferred", (256, 768, 655360, 32, 128), BF16, True),
    ("bwd_x_any_preferred", (128, 768, 131072, 16, 64), BF16, True),
    ("bwd_x_any_preferred", (256, 768, 131072, 32, 256), BF16, True),
    ("bwd_x_any_preferred", (512, 768, 2949120, 32, 64), BF16, False),
    ("bwd_x_f32_preferred", (128, 768, 131072, 16, 64), F32, True),
    ("bwd_x_f32_preferred", (32, 256, 4096, 8, 32), F32, True),
]


@pytest.mark.parametrize("name,shape,dtype,taken", FWD + BWD_W + BWD_X)
def test_route(name, shape, dtype, taken):
    assert rule(name, shape, dtype) == taken
