"""D3Q19 lattices whose two-step passes march through many planes per work-group:
(shape, storage, walls) with the planes, the kernel with the smaller column limit
(small) and the placement (separable: whole planes to a chunk) their plan takes on
256 compute units.  test_plans.py holds the plans to this, test_gpu_passes.py
runs them."""

MARCHES = [
    # shape, storage, walls, planes per work-group at least, small, separable
    ((128, 128, 70), "f32", True, 6, False, True),
    ((256, 64, 63), "f32", True, 6, False, True),
    ((128, 128, 64), "f64", True, 6, False, True),
    ((128, 128, 64), "f16", True, 6, False, True),
    ((150, 90, 61), "f32", True, 6, False, False),
    ((150, 90, 61), "f32", False, 6, False, False),
    ((150, 90, 61), "f64", True, 6, False, False),
    ((128, 96, 64), "f64", False, 6, False, True),
    ((120, 90, 61), "f16", True, 6, False, False),
    ((120, 90, 61), "bf16", True, 6, False, False),
    ((90, 90, 90), "f16", False, 6, False, False),
    ((90, 90, 90), "bf16", False, 6, False, False),
    ((8, 13, 4001), "f32", True, 6, True, False),
    ((8, 13, 4000), "f32", False, 6, True, False),
    ((7, 9, 5000), "f64", True, 6, True, False),
    ((8, 13, 8000), "f64", False, 6, True, False),
    ((4, 4, 9000), "bf16", True, 6, True, False),
]
