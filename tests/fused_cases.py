"""Linears whose fused products (the 1-bit product with the rank-r branch as a second contraction) take each form that the
library has on 128x128 and 256x256 tiles: whole contraction steps or a partial last one, the second contraction in the ring of
the 256x256 loop (rank 64 or 128; it starts at the stage where the first one ends) or through registers, whole or split
contractions, and the unfused fall-back of a split 256x256 plan.  test_launch_rules.py checks without a GPU that each case still
takes the form it stands for; test_gpu_tile.py runs them."""

# (tokens, d_in, d_out, rank, INT8 branch) -> forward, input gradient
#   256x256: (256, "ring", steps, first stage), (256, "registers", steps), (256, "unfused", steps); steps: "whole" or "partial"
#   smaller tiles: (128 or 64, splits > 1)
CASES = {
    (5494, 384, 416, 72, 0): ((128, False), (128, False)),
    (5534, 352, 544, 200, 0): ((128, False), (128, False)),
    (2435, 3776, 416, 128, 0): ((128, True), (256, "ring", "partial", 3)),
    (4833, 416, 2144, 128, 0): ((256, "ring", "partial", 0), (128, True)),
    (3358, 608, 2400, 64, 0): ((256, "ring", "partial", 1), (256, "unfused", "partial")),
    (5458, 736, 1920, 128, 0): ((256, "ring", "partial", 2), (256, "unfused", "whole")),
    (5957, 800, 1312, 128, 0): ((256, "ring", "partial", 3), (128, False)),
    (5573, 512, 1472, 64, 0): ((256, "ring", "whole", 0), (128, False)),
    (5155, 640, 1568, 128, 0): ((256, "ring", "whole", 1), (128, False)),
    (5564, 768, 1536, 128, 0): ((256, "ring", "whole", 2), (128, False)),
    (4357, 896, 1824, 64, 0): ((256, "ring", "whole", 3), (128, False)),
    (1300, 6272, 224, 64, 0): ((64, True), (256, "ring", "partial", 0)),
    (2470, 3296, 288, 128, 0): ((64, False), (256, "ring", "partial", 1)),
    (1317, 6080, 352, 64, 0): ((64, True), (256, "ring", "partial", 2)),
    (1441, 5440, 256, 128, 0): ((64, True), (256, "ring", "whole", 0)),
    (2355, 3424, 384, 64, 0): ((64, False), (256, "ring", "whole", 2)),
    (5892, 1344, 96, 128, 0): ((64, False), (256, "registers", "partial")),
    (4215, 3648, 224, 200, 0): ((128, True), (256, "registers", "partial")),
    (2702, 2976, 128, 32, 0): ((64, False), (256, "registers", "whole")),
    (4407, 96, 1952, 128, 0): ((256, "registers", "partial"), (64, False)),
    (4249, 128, 2080, 200, 0): ((256, "registers", "whole"), (64, False)),
    # INT8 branch: its forward is not fused
    (657, 3168, 96, 32, 1): (None, (128, False)),
    (266, 3552, 1440, 96, 1): (None, (128, True)),
    (3612, 2208, 96, 96, 1): (None, (256, "registers", "partial")),
    (4399, 1856, 128, 64, 1): (None, (256, "registers", "whole")),
    (5493, 1472, 224, 128, 1): (None, (256, "ring", "partial", 0)),
    (2452, 3328, 256, 64, 1): (None, (256, "ring", "whole", 0)),
    (391, 4896, 2560, 128, 1): (None, (256, "unfused", "whole")),
}
