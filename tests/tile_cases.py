"""Products of every tile shape of gemm.hip: the test on the GPU runs them, the one on the CPU checks that each reaches the tile
it is listed under, so that a change of the rule that picks tiles cannot leave one without a test."""
BIAS_RES, BIAS_GELU = 1, 2

# tile configuration -> (M, N, K, epilogue): rows and columns that end inside a tile, K shorter than the ring and longer
TILES = {
    16: [(65, 2040, 64, BIAS_RES), (64, 1000, 256, BIAS_GELU), (160, 2832, 1024, BIAS_GELU)],      # 64x64
    18: [(33, 8192, 2048, BIAS_GELU), (64, 1000, 512, BIAS_GELU), (169, 80, 576, BIAS_RES), (177, 1272, 1024, BIAS_GELU)],     # 64x32
    17: [(129, 6136, 448, BIAS_GELU), (257, 5000, 1024, BIAS_RES), (156, 4288, 64, BIAS_RES)],     # 128x64
    40: [(758, 4512, 256, BIAS_GELU), (151, 8376, 64, BIAS_RES), (1281, 2040, 4096, BIAS_RES)],    # 128x128
    6: [(577, 8200, 256, BIAS_GELU), (1500, 4104, 64, BIAS_GELU), (1154, 3488, 64, BIAS_RES)],     # 128x128, two a CU
    35: [(2299, 2040, 8192, BIAS_RES), (2241, 2048, 8192, BIAS_RES), (539, 6576, 1024, BIAS_GELU)],   # 160x128
    34: [(731, 6144, 256, BIAS_GELU), (731, 6152, 2048, BIAS_GELU), (731, 7688, 1920, BIAS_GELU),     # 192x128
         (770, 4648, 64, BIAS_RES), (938, 5264, 320, BIAS_RES)],
    13: [(1345, 8192, 128, BIAS_RES), (920, 8336, 64, BIAS_GELU), (925, 8416, 1024, BIAS_RES)],    # 192x256
    32: [(577, 8200, 2048, BIAS_GELU), (772, 6648, 256, BIAS_RES), (735, 8768, 1024, BIAS_RES)],   # 256x128
    11: [(1537, 8192, 2048, BIAS_GELU), (1345, 8472, 64, BIAS_RES), (1348, 8224, 1024, BIAS_GELU)],   # 256x256
}

# tiles of QKV alone -> (D, dh, B, k)
QKV_TILES = {15: (1152, 128, 1, 131), 12: (1344, 64, 2, 1283)}   # 64x64 with eight stages, 256x192

# blocks whose out-proj and FC2 are cut into slices, on every tile that takes them: (D, H, dh, F) and (B, h, w, k)
SLICED_DIMS = [(448, 7, 64, 2048), (1024, 16, 64, 4096), (1088, 17, 64, 8192), (4224, 33, 128, 4352)]
SLICED_ROWS = [(1, 1, 17, 17), (1, 9, 9, 63), (1, 9, 9, 65), (3, 6, 8, 43), (1, 16, 17, 257), (2, 16, 16, 193), (1, 25, 25, 577)]
SLICED_ALONE = ((1472, 23, 64, 4096), (1, 18, 18, 321))   # 192x128
