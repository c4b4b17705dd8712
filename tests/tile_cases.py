"""Products of every tile shape of gemm_tiles.h: the test on the GPU runs them, the one on the CPU checks that each reaches the tile
it is listed under, so that a change of the rule that picks tiles cannot leave one without a test."""
BIAS_RES, BIAS_GELU = 1, 2

# tile configuration -> (M, N, K, epilogue): rows and columns that end inside a tile, K shorter than the ring and longer
TILES = {
    16: [(65, 2040, 64, BIAS_RES), (64, 1000, 256, BIAS_GELU), (160, 2832, 1024, BIAS_GELU)],   # 64x64
    18: [(33, 8192, 2048, BIAS_GELU), (64, 1000, 512, BIAS_GELU), (169, 80, 576, BIAS_RES),   # 64x32
         (177, 1272, 1024, BIAS_GELU)],
    17: [(129, 6136, 448, BIAS_GELU), (257, 5000, 1024, BIAS_RES), (156, 4288, 64, BIAS_RES),   # 128x64
         (66, 8312, 1024, BIAS_GELU), (65, 8216, 2048, BIAS_RES), (129, 4232, 2048, BIAS_GELU),
         (130, 4232, 128, BIAS_GELU)],
    40: [(151, 8376, 64, BIAS_RES), (758, 4512, 256, BIAS_GELU), (1281, 2040, 4096, BIAS_RES),   # 128x128
         (130, 8352, 128, BIAS_GELU), (130, 8408, 1024, BIAS_RES)],
    35: [(2299, 2040, 8192, BIAS_RES), (2241, 2048, 8192, BIAS_RES), (539, 6576, 1024, BIAS_GELU),   # 160x128
         (731, 6152, 2048, BIAS_GELU), (1159, 3400, 448, BIAS_RES)],
    34: [(770, 4648, 64, BIAS_RES), (731, 6144, 256, BIAS_GELU), (731, 7688, 1920, BIAS_GELU),   # 192x128
         (938, 5264, 320, BIAS_RES), (1154, 3488, 64, BIAS_RES), (1345, 8192, 128, BIAS_RES),
         (642, 5432, 1024, BIAS_GELU)],
    14: [(920, 8336, 64, BIAS_GELU), (925, 8416, 1024, BIAS_RES), (899, 8224, 128, BIAS_RES),   # 192x192
         (898, 8216, 192, BIAS_GELU), (1680, 4616, 64, BIAS_GELU), (1687, 4624, 128, BIAS_RES),
         (1153, 6744, 192, BIAS_GELU), (735, 8768, 1024, BIAS_RES)],
    13: [(1126, 8104, 1024, BIAS_RES), (1291, 7944, 256, BIAS_GELU)],   # 192x256
    36: [(577, 8200, 2048, BIAS_GELU), (579, 8264, 1024, BIAS_RES)],   # 224x128
    37: [(1732, 4816, 128, BIAS_GELU), (1553, 5384, 256, BIAS_RES), (1153, 6936, 1024, BIAS_GELU)],   # 224x192
    38: [(1537, 8192, 2048, BIAS_GELU), (1348, 8224, 1024, BIAS_GELU), (1540, 7568, 64, BIAS_RES),   # 224x256
         (1544, 7576, 128, BIAS_RES), (1409, 8224, 192, BIAS_GELU), (1546, 7216, 256, BIAS_GELU)],
    32: [(577, 8200, 256, BIAS_GELU), (1500, 4104, 64, BIAS_GELU), (772, 6648, 256, BIAS_RES),   # 256x128
         (1345, 8472, 64, BIAS_RES), (646, 8536, 64, BIAS_GELU), (645, 8496, 128, BIAS_RES),
         (2261, 5912, 128, BIAS_GELU)],
    12: [(2122, 4896, 192, BIAS_RES), (2115, 4872, 256, BIAS_GELU), (964, 8240, 1024, BIAS_RES),   # 256x192
         (1924, 5928, 64, BIAS_RES), (2025, 4816, 128, BIAS_GELU), (1155, 8208, 192, BIAS_RES),
         (962, 8272, 1024, BIAS_GELU)],
    11: [(2242, 5896, 192, BIAS_RES), (2244, 5904, 256, BIAS_GELU), (1573, 8224, 448, BIAS_RES)],   # 256x256
}

# ... and those of GELU on the widest tiles, whose workgroups walk several tiles: more than a round of 256, in numbers that eight XCDs do and
# do not share evenly, of K shorter than the ring, as long and longer
SEAMS = {
    11: [(2887, 10600, 192, BIAS_GELU), (2332, 11912, 448, BIAS_GELU), (5070, 6008, 1024, BIAS_GELU), (3516, 8632, 2048, BIAS_GELU)],
    38: [(2517, 10600, 64, BIAS_GELU), (2147, 11256, 128, BIAS_GELU), (5810, 4696, 192, BIAS_GELU), (3331, 8304, 448, BIAS_GELU)],
}

# tiles of QKV -> (D, dh, B, k): the one of its own, 64x64 with eight stages, and some of the wide ones, with at most a round of tiles and more
QKV_TILES = {15: (1152, 128, 1, 131), 37: (1344, 64, 2, 1283), 14: (1600, 64, 3, 1110), 13: (2368, 64, 3, 971)}
# ... with more than a round of tiles each, plain and with rotary positions
QKV_SEAMS = {11: (1152, 128, 2, 4315), 38: (1152, 64, 8, 911), 12: (1152, 64, 3, 2165), 37: (896, 128, 1, 7349), 14: (704, 64, 5, 1543),
             13: (1344, 64, 3, 1799), 32: (704, 64, 3, 2409)}
# ... and one of every other tile that rotary positions are turned on, within a round
ROPE_TILES = {35: (2048, 128, 1, 679), 36: (1536, 128, 2, 688), 34: (1024, 64, 1, 1529), 40: (448, 64, 3, 538), 17: (448, 64, 3, 283),
              16: (704, 64, 1, 237), 15: (1152, 128, 1, 135), 18: (448, 64, 3, 79)}

# blocks whose out-proj and FC2 are cut into slices, on every tile that takes them: (D, H, dh, F) and (B, h, w, k)
SLICED_DIMS = [(448, 7, 64, 2048), (1024, 16, 64, 4096), (1088, 17, 64, 8192), (4224, 33, 128, 4352)]
SLICED_ROWS = [(1, 1, 17, 17), (1, 9, 9, 63), (1, 9, 9, 65), (3, 6, 8, 43), (1, 16, 17, 257), (2, 16, 16, 193), (1, 25, 25, 577)]
SLICED_ALONE = ((1472, 23, 64, 4096), (1, 18, 18, 321))   # 192x128
