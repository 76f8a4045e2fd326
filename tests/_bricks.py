"""Boards for the small-board kernel's tests: sizes and the brick (rows, planes owned)
each is stepped in on a device of 256 compute units, (0, 0) where the marching kernel
is faster."""

CUS = 256
B87, B88, B128, B1010, B168, MARCHING = (4, 3), (4, 4), (8, 4), (6, 6), (12, 4), (0, 0)

# the sizes of the bitwise tests around the bricks' edges
EDGES = {(8, 7, 6): B87, (28, 8, 9): B87, (29, 13, 10): B87, (56, 44, 30): B87, (57, 41, 45): B128,
         (66, 46, 30): B128, (84, 66, 42): B1010, (81, 67, 37): B1010, (131, 61, 41): MARCHING}

# every shape with whole bricks and with ragged ones (8x8: 28 x 4 x 4, 16x8: 28 x 12 x 4), and
# the first board past the line
SHAPES = {(56, 64, 32): B88, (57, 33, 35): B88, (200, 20, 20): B88, (48, 43, 36): B88,
          (112, 96, 28): B168, (113, 49, 33): B168, (130, 60, 40): B168, (113, 44, 37): B168,
          (48, 43, 30): B87, (1000, 4, 4): B87, (85, 37, 29): B128, (80, 72, 37): B1010,
          (2, 500, 20): MARCHING, (160, 120, 60): MARCHING}
