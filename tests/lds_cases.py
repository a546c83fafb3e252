"""Sizes of contractions over long k that take one round of large tiles (csrc/lds_tiles.h, LDS_LONG_TILES)."""

# M, N, K: rows and columns that end inside a tile or fill it, k that ends inside a stage or fills it, the shortest k that qualifies
LONG_CASES = [(232, 11016, 4104), (720, 4096, 4096), (128, 24608, 3848), (1288, 3336, 1544), (256, 16520, 1536), (1024, 4096, 4160)]
LONG_EXTRAS = [(232, 11016, 4104), (1288, 3336, 1544)]               # with bias and residual
LONG_BATCHES = [(136, 904, 4104, 12), (520, 520, 1544, 16), (392, 264, 2056, 32)]  # M, N, K, problems
