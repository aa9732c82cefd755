"""Boxes that reach each kernel of the passes of several steps, and which: threads
per block of the brick kernels, or the variant of the marching one, by storage (0:
single steps).  test_step_host.py checks these on the CPU for 256 compute units,
test_gpu_pass_shapes.py steps the boxes."""
from lbm_inputs import face

WALL, PER = face("wall", "adiabatic"), face("periodic", "periodic")
HOT, COLD = face("wall", "isothermal", 0.4), face("wall", "isothermal", -0.3)

# shape, flow populations, faces, {storage: threads}
FLOW = {
    "cube33": ((33, 33, 33), 19, [HOT, COLD, WALL, WALL, PER, PER], {"fp64": 768, "fp32": 0, "fp16": 0}),
    "cube40": ((40, 40, 40), 15, [HOT, COLD, PER, PER, WALL, WALL], {"fp64": 768, "fp32": 768, "fp16": 0}),
    "ragged": ((41, 38, 37), 19, [PER, PER, HOT, COLD, PER, PER], {"fp64": 768, "fp32": 0, "fp16": 0}),
    "rows48": ((48, 32, 26), 19, [PER] * 6, {"fp64": 512, "fp32": 768, "fp16": 768}),
    "rows40": ((40, 23, 29), 15, [WALL, WALL, HOT, COLD, WALL, WALL], {"fp64": 768, "fp32": 768, "fp16": 768}),
    "short": ((7, 90, 61), 19, [HOT, WALL, PER, PER, COLD, WALL], {"fp64": 512, "fp32": 512, "fp16": 512}),
    "cube13": ((13, 13, 13), 15, [HOT, COLD, WALL, WALL, PER, PER], {"fp64": 256, "fp32": 256, "fp16": 256}),
    "past": ((46, 46, 46), 19, [HOT, COLD, WALL, WALL, WALL, WALL], {"fp64": 0, "fp32": 0, "fp16": 0}),
}

# shape, faces, {storage: threads}
MELT = {
    "line": ((1, 17, 25), [PER, PER, HOT, COLD, PER, PER], {"fp64": 512, "fp32": 512}),
    "plane": ((1, 18, 16), [WALL, HOT, PER, PER, COLD, WALL], {"fp64": 512, "fp32": 512}),
    "column": ((3, 3, 2), [PER] * 6, {"fp64": 256, "fp32": 256}),
    "slab": ((160, 11, 10), [HOT, COLD, PER, PER, PER, PER], {"fp64": 1024, "fp32": 1024}),
    "past": ((60, 32, 32), [HOT, COLD, PER, PER, PER, PER], {"fp64": 0, "fp32": 0}),
}

# shape, faces, {storage: variant}; boxes whose halo planes or rows are their own
MARCH = {
    "two_planes": ((1024, 512, 2), [HOT, COLD, PER, PER, PER, PER], {"fp64": 2, "fp32": 0}),
    "two_planes_fp32": ((2018, 400, 2), [PER, PER, WALL, HOT, PER, PER], {"fp64": 0, "fp32": 2}),
    "two_walls": ((512, 512, 2), [HOT, COLD, WALL, WALL, HOT, COLD], {"fp64": 2, "fp32": 0}),
    "three_rows": ((1024, 3, 300), [WALL, HOT, PER, PER, PER, PER], {"fp64": 2, "fp32": 0}),
    "four_rows": ((1024, 4, 256), [PER, PER, PER, PER, COLD, WALL], {"fp64": 2, "fp32": 2}),
    "streamed": ((358, 100, 83), [HOT, COLD, PER, PER, WALL, WALL], {"fp64": 4, "fp32": 2}),
    "narrow": ((16, 256, 256), [HOT, COLD, PER, PER, PER, PER], {"fp64": 0, "fp32": 0}),
    "odd": ((129, 128, 128), [HOT, COLD, PER, PER, PER, PER], {"fp64": 0, "fp32": 0}),
}
