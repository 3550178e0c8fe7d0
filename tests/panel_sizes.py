"""Sectors that together reach every variant of the panel kernel with as many
target rows per workgroup as it is built for: (orbitals, N_alpha, N_beta) ->
(variant, most rows of a workgroup in a single launch on 256 compute units)."""

SINGLE = {
    (11, 5, 5): (0, 2),
    (12, 3, 3): (1, 1),
    (14, 3, 3): (1, 2),  # complex64 leaves this one to the sector kernel
    (12, 6, 6): (2, 4),
    (14, 4, 4): (3, 4),
    (13, 6, 5): (4, 4),
    (14, 5, 5): (5, 4),
    (14, 6, 7): (6, 2),
}

# batches of equal jobs: (sector, jobs) -> (variant, rows of a workgroup)
BATCHES = {
    ((10, 5, 5), 16): (0, 4),
    ((9, 4, 4), 12): (0, 3),
    ((14, 3, 3), 6): (1, 3),
}
