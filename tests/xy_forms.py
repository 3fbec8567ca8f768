"""Volumes and batches for each form of the iteration's xy pass (RSF force): the
CPU check asserts which form a plan takes, the GPU tests run them."""

# radius, (nz, ny, nx), waves of a workgroup (2: the small-volume form), row
# chunks: 8 waves in one and in two strips (the last one moved left), whole and
# in row chunks; 4 waves in many short row chunks; even and odd radii
VOLUMES = [
    (1, (128, 3, 800), 8, 1), (1, (128, 20, 512), 8, 2), (1, (64, 29, 800), 8, 2),
    (4, (128, 3, 800), 8, 1), (4, (96, 46, 512), 8, 2), (4, (64, 46, 800), 8, 2),
    (7, (128, 3, 745), 8, 1), (7, (96, 76, 500), 8, 2), (7, (64, 76, 745), 8, 2),
    (10, (128, 3, 745), 8, 1), (10, (96, 100, 500), 8, 2),
    (12, (128, 3, 745), 8, 1), (12, (64, 118, 745), 8, 2),
    (16, (128, 3, 745), 8, 1), (16, (64, 154, 745), 8, 2),
    (1, (96, 25, 5), 4, 7), (4, (96, 265, 5), 4, 10), (6, (96, 225, 5), 4, 10),
    (7, (96, 165, 5), 4, 10), (10, (96, 145, 5), 4, 10), (13, (96, 115, 5), 4, 9),
    (16, (3, 80, 65), 4, 16),
]

# radius, tiles, waves: unequal widths in workgroups of 8 waves (those past a
# narrower tile's strip leave) and in workgroups of 4, where the widest tile's
# strips of 8 would be partly filled
BATCHES = [
    (9, [(24, 40, 385), (20, 37, 512), (16, 50, 450), (12, 33, 401)], 8),
    (4, [(24, 40, 512), (20, 37, 497), (16, 50, 130)], 8),
    (12, [(16, 96, 100), (32, 128, 512), (32, 120, 512)], 8),
    (9, [(32, 96, 400), (32, 96, 600)], 4),
    (6, [(16, 60, 114), (16, 64, 274), (20, 50, 300)], 4),
]
