"""Host model of the projections' plans (gemm.hip: runs_whole, sk_plan, plan_cost, choose_tile and the launch
rule that leaves the fixup out), and the shapes with which the GPU tests reach each kind of plan.

A plan is (tile, tiles, pieces per tile, data-parallel units, stream-K units, workgroups sharing those), or
("small", tiles, turns) for the 64 x 32 tiles.  More workgroups than stream-K units means cut units."""
from paper_2606_13898_amd.inputs import BlockShape

WORKGROUPS = 256      # kGemmWorkgroups
NO_SPLIT_STEPS = 64   # kNoSplitSteps
MIN_STEPS = 12        # kSkMinSteps
# estimates of choose_tile in units of 10 ns: a K step, a tile, a tile that updates z, the partials of a tail, of K
# pieces in all, per tile, and in all without a tail
TILE_COSTS = {192: (91, 400, 1400, 2000, 2700, 20, 2500), 256: (146, 700, 3300, 3600, 4500, 35, 4500)}
SMALL_COSTS = (140, 265, 300)  # four K steps with one tile a workgroup, with two, a turn
LAUNCH_Z, LAUNCH = 300, 700  # a launch of whole tiles that update z or don't


def whole_tiles(T, P, nk):
    """runs_whole: every tile runs whole (no K pieces, no stream-K tail)."""
    whole_waves = T >= P and (T % P == 0 or 2 * (T % P) >= P)
    return (T < P and nk <= NO_SPLIT_STEPS) or whole_waves or (T < P and 8 * T >= 7 * P)


def plan(T, P, nk):
    """sk_plan: pieces s, units U, data-parallel units dp, steps of a stream-K unit, their steps, Pk."""
    if whole_tiles(T, P, nk):
        return 1, T, T, nk, 0, P
    return cut_plan(T, P, nk)


def cut_plan(T, P, nk):
    """The plan of a problem that does not run whole tiles."""
    s = 1 if (T >= P or T == 0) else min(-(-P // T), nk)
    U = T * s
    dp = U // P * P
    tail = U - dp
    pc = dp // T if tail > 0 else 0
    ln = (pc + 1) * nk // s - pc * nk // s
    I = tail * ln
    Pk = min(P, max(tail, -(-I // MIN_STEPS)))
    return s, U, dp, ln, I, Pk


def row_tiles(segments, tile):
    """Row tiles of [(image rows, text rows)] per sample."""
    return sum(-(-n // tile) for seg in segments for n in seg)


def cost(resid, T, nk, step, tile, tile_z, tail, piece, piece_t, even):
    """plan_cost, in units of 10 ns."""
    P = WORKGROUPS
    rounds, t = -(-T // P), tile_z if resid else tile
    if whole_tiles(T, P, nk):
        return rounds * (nk * step + t) + (LAUNCH_Z if resid else LAUNCH)
    steps = T * nk // P * step
    if T >= P:
        return steps + rounds * t + tail
    return steps + (even if T & (T - 1) == 0 else piece + piece_t * T)


def choose(segments, N, K, resid):
    """choose_tile: 192, 256 or "small"."""
    nk = K // 64
    c192, c256 = (cost(resid, row_tiles(segments, t) * -(-N // t), nk, *TILE_COSTS[t]) for t in (192, 256))
    best, tile = (c256, 256) if c256 < c192 else (c192, 192)
    tiles = row_tiles(segments, 64) * (N // 32)
    turns = -(-tiles // (2 * WORKGROUPS))
    one, two, turn = SMALL_COSTS
    if turns * (-(-nk // 4) * (one if tiles <= WORKGROUPS else two) + turn) < best:
        tile = "small"
    return tile


def describe(segments, N, K, resid, tile=None, kstep=64):
    """The plan of a projection: on `tile` (FP8: fixed, with kstep 128), or on the one the kernel chooses."""
    tile = tile or choose(segments, N, K, resid)
    if tile == "small":
        tiles = row_tiles(segments, 64) * (N // 32)
        return "small", tiles, -(-tiles // (2 * WORKGROUPS))
    T = row_tiles(segments, tile) * -(-N // tile)
    s, U, dp, _, _, Pk = plan(T, WORKGROUPS, K // kstep)
    return tile, T, s, dp, U - dp, Pk


def projections(segments, dim, mlp, fp8=False):
    """Plans of the four projections of a block."""
    roles = dict(qkv=(3 * dim, dim, False, 256), o=(dim, dim, True, 192), up=(mlp, dim, False, 192),
                 down=(dim, mlp, True, 192))
    return {k: describe(segments, N, K, r, tile if fp8 else None, 128 if fp8 else 64)
            for k, (N, K, r, tile) in roles.items()}


def fixup_skipped(max_img_rows, text, batch, N, K, tile=192, kstep=64):
    """The launch rule: no fixup when even the longest sequences make fewer tiles than workgroups and K is
    short."""
    tiles = batch * (-(-max_img_rows // tile) + -(-text // tile)) * -(-N // tile)
    return tiles < WORKGROUPS and K // kstep <= NO_SPLIT_STEPS


# (dim, mlp_dim, sample lengths, text rows), and the plans of MLP up and down
MLP_SHAPES = [
    # 64 x 32 tiles: K of one, three, five and fifteen steps over four waves, one turn; 192 x 192 of one K step
    ((64, 320, [193, 65], 31), dict(up=("small", 60, 1), down=("small", 12, 1))),
    ((192, 960, [705, 64, 1], 0), dict(up=("small", 420, 1), down=("small", 84, 1))),
    ((64, 1024, [1100, 901], 31), dict(up=(192, 78, 1, 78, 0, 256), down=("small", 66, 1))),
    # 64 x 32 tiles in two turns
    ((256, 1088, [2100], 40), dict(up=(192, 72, 1, 72, 0, 256), down=("small", 272, 1))),
    ((640, 1024, [1640], 40), dict(up=(192, 60, 1, 60, 0, 256), down=("small", 520, 2))),
    # 256 whole 256 x 256 tiles; 12 tiles of 192 x 192 in 22 pieces and a stream-K tail of 8 whole pieces
    ((512, 16384, [600], 40), dict(up=(256, 256, 1, 256, 0, 256), down=(192, 12, 22, 256, 8, 8))),
    # 192 x 192, one piece: tails of 4 tiles over 6 workgroups and (residual) 41 over 195; K pieces whose tail
    # is cut again
    ((1024, 8192, [2040], 40), dict(up=(192, 516, 1, 512, 4, 6), down=(192, 72, 4, 256, 32, 86))),
    ((2048, 3648, [5000], 0), dict(up=(192, 513, 1, 512, 1, 3), down=(192, 297, 1, 256, 41, 195))),
    # 192 x 192 in five waves of whole tiles; 19 pieces, their tail cut
    ((64, 16384, [2500], 0), dict(up=(192, 1204, 1, 1204, 0, 256), down=(192, 14, 19, 256, 10, 12))),
    # 256 x 256: a tail of 16 tiles over 32 workgroups; K pieces whose tail is cut (residual)
    ((1536, 13312, [5000], 0), dict(up=(256, 1040, 1, 1024, 16, 32), down=(256, 120, 3, 256, 104, 256))),
    # 256 x 256 residual in one wave of whole tiles, and in two
    ((2560, 8192, [5540], 40), dict(up=(256, 736, 1, 736, 0, 256), down=(256, 230, 1, 230, 0, 256))),
    ((2048, 4096, [15000], 0), dict(up=(256, 944, 1, 944, 0, 256), down=(256, 472, 1, 472, 0, 256))),
]

# Whole blocks, every patch kept fine so that the row counts are fixed: all four projections
BLOCK_SHAPES = {
    # QKV on 192 x 192: one wave and a tail of 8 tiles over 44 workgroups; the output in 3 pieces, their tail cut
    "sk_tail": (BlockShape(1, 1, 24, 24, 40, 4224, 33, 128, 1024, "bf16"),
                dict(qkv=(192, 264, 1, 256, 8, 44), o=(192, 88, 3, 256, 8, 15), up=(192, 24, 11, 256, 8, 8),
                     down=(192, 88, 1, 88, 0, 256))),
    # MLP up on 192 x 192 in two waves of whole tiles
    "whole_waves": (BlockShape(1, 1, 52, 52, 256, 256, 2, 128, 5760, "bf16"),
                    dict(qkv=(192, 68, 1, 68, 0, 256), o=("small", 376, 1), up=(192, 510, 1, 510, 0, 256),
                         down=(192, 34, 8, 256, 16, 16))),
    # QKV in 2 pieces, their tail of 40 over 124 workgroups; the output in 6
    "k_pieces": (BlockShape(1, 1, 12, 12, 40, 4736, 37, 128, 1024, "bf16"),
                 dict(qkv=(192, 148, 2, 256, 40, 124), o=(192, 50, 6, 256, 44, 48),
                      up=("small", 128, 1), down=("small", 592, 2))),
    # QKV on 256 x 256 in 5 pieces, their tail cut
    "k_pieces_256": (BlockShape(1, 1, 14, 14, 0, 5120, 40, 128, 1024, "bf16"),
                     dict(qkv=(256, 60, 5, 256, 44, 59), o=(192, 54, 5, 256, 14, 19), up=("small", 128, 1),
                          down=("small", 640, 2))),
}

# The MLP half with K pieces, every row compared
SPLIT_K_SHAPES = {
    # MLP down in 10 pieces plus a stream-K tail of 14 units over 16 workgroups; MLP up in two waves
    "pieces_and_tail": (BlockShape(3, 1, 16, 20, 40, 512, 4, 128, 8192, "bf16"),
                        dict(qkv=("small", 864, 2), o=("small", 288, 1), up=(192, 387, 1, 387, 0, 256),
                             down=(192, 27, 10, 256, 14, 16))),
    # a single 192 x 192 down-projection tile: every K piece is one step, the fixup sums 128 partial tiles
    "one_tile_128_pieces": (BlockShape(1, 1, 12, 12, 0, 192, 3, 64, 8192, "bf16"),
                            dict(qkv=("small", 54, 1), o=("small", 18, 1), up=("small", 768, 2),
                                 down=(192, 1, 128, 0, 128, 128))),
}

# FP8 (QKV on 256 x 256 tiles, the others on 192 x 192, K steps of 128), every patch kept fine
FP8_SHAPES = {
    # QKV: one wave plus an 8-tile tail over 11 workgroups; MLP up: one wave plus a 29-tile tail over 39
    "sk_tail": (BlockShape(1, 1, 48, 48, 512, 2048, 16, 128, 3584, "bf16"),
                dict(qkv=(256, 264, 1, 256, 8, 11), o=(192, 165, 1, 165, 0, 256), up=(192, 285, 1, 256, 29, 39),
                     down=(192, 165, 1, 165, 0, 256))),
    # MLP up: the last wave half full, so two waves of whole tiles
    "whole_waves": (BlockShape(1, 1, 64, 64, 256, 256, 2, 128, 3072, "bf16"),
                    dict(qkv=(256, 51, 1, 51, 0, 256), o=(192, 48, 1, 48, 0, 256), up=(192, 384, 1, 384, 0, 256),
                         down=(192, 48, 1, 48, 0, 256))),
    # K = 4608 in 36 steps, few tiles: whole tiles; MLP up N = 1152 ends in a 128-column tile; MLP down 9 steps
    "long_k": (BlockShape(1, 1, 16, 16, 0, 4608, 36, 128, 1152, "bf16"),
               dict(qkv=(256, 54, 1, 54, 0, 256), o=(192, 48, 1, 48, 0, 256), up=(192, 12, 1, 12, 0, 256),
                    down=(192, 48, 1, 48, 0, 256))),
    # MLP down, 128 steps: 10 pieces of 12 and 13 steps, a tail of 24 over 26 workgroups that cuts them again
    "k_pieces": (BlockShape(1, 1, 32, 32, 40, 768, 6, 128, 16384, "bf16"),
                 dict(qkv=(256, 45, 1, 45, 0, 256), o=(192, 28, 1, 28, 0, 256), up=(192, 602, 1, 512, 90, 90),
                      down=(192, 28, 10, 256, 24, 26))),
}


def segments(shape):
    """(image rows, text rows) of every sample with every patch kept fine."""
    return [(shape.images * shape.n_patches, shape.text_len)] * shape.batch
