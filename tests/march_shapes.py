"""Grids on which the marches run the launch shapes of large grids: two nodes
per lane (overlapping last window of a walled odd row, 8-byte accesses at odd
row starts), four rows per wave, chunks of more than 40 rows (the per-row
values of 64 rows are fetched again within a chunk).  Which shape each grid
takes is checked in test_march_shapes.py; the results in
test_gpu_march_shapes.py."""
PER, WALL, SYM = 0, 1, 2

FACES2 = {"periodic": (PER, PER, PER, PER), "walls_y": (PER, PER, WALL, WALL), "walls_x": (WALL, SYM, PER, PER),
          "cavity": (WALL, WALL, SYM, WALL)}
# (nx, ny, precision, faces, axisymmetric): (nodes per lane, steps per launch, rows per chunk at least)
MARCH2D = {
    (1537, 1100, "f32", "cavity", 0): (2, 2, 2),
    (1541, 1103, "f32", "walls_x", 0): (2, 2, 2),
    (1536, 1537, "f32", "periodic", 0): (2, 2, 2),
    (3000, 1499, "f32", "walls_y", 0): (2, 2, 2),
    (2049, 1030, "f32", "walls_x", 1): (2, 2, 2),
    (4096, 2047, "f32", "periodic", 1): (2, 2, 2),
    (200, 40000, "f32", "cavity", 0): (2, 2, 40),
    (300, 30000, "f32", "periodic", 0): (1, 2, 41),
    (6001, 2001, "f32", "walls_x", 1): (2, 2, 41),
    (1280, 4096, "f64", "periodic", 1): (1, 2, 41),
    (1280, 4095, "f64", "walls_x", 1): (1, 2, 41),
    (1280, 4097, "f64", "cavity", 0): (1, 2, 41),
}

FACES2P = {"periodic": (PER, PER, PER, PER), "channel": (PER, PER, WALL, WALL), "slab": (WALL, SYM, PER, PER),
           "box": (SYM, WALL, WALL, SYM), "axis": (PER, PER, SYM, SYM), "axis_box": (WALL, WALL, SYM, WALL)}
# (nx, ny, precision, faces): (nodes per lane, rows per chunk at least)
TWO_PHASE = {
    (3001, 3501, "f32", "box"): (2, 41),
    (3001, 3501, "f32", "axis_box"): (2, 41),
    (3000, 3502, "f32", "channel"): (2, 41),
    (200, 21000, "f64", "periodic"): (1, 41),
    (201, 21001, "f64", "axis_box"): (1, 41),
}

FACES3 = {"periodic": (PER,) * 6, "duct": (PER, PER, WALL, WALL, WALL, SYM), "cavity": (WALL, SYM, WALL, WALL, SYM, WALL),
          "slab": (WALL, WALL, PER, PER, PER, PER), "channel_z": (PER, PER, PER, PER, WALL, WALL)}
# four rows per wave, rows of a grid 1, 2, 3 and 0 beyond a multiple of four
MARCH3D = [(200, 99, 70, "duct"), (200, 99, 70, "periodic"), (200, 99, 70, "channel_z"), (200, 201, 101, "periodic"),
           (200, 201, 101, "duct"), (200, 201, 101, "cavity"), (200, 201, 101, "slab"), (202, 198, 99, "cavity"),
           (202, 198, 99, "channel_z"), (100, 100, 100, "cavity"), (100, 100, 100, "slab")]
