"""Shapes of the layer-step parity cases (pure data, importable without a GPU).

Every case is one linear layer [O, K] with T calibration tokens.  `chained` cases are stepped with an
upstream gradient and with dX requested (three GEMMs), the others with the locally derived dY (two GEMMs);
every case also runs faar_layer_prepare with a bf16 and with a float32 reference output.  The list is
chosen so that, together, the cases reach every GEMM kernel variant the library's planner can pick for any
layer shape (tests/test_plan_coverage.py proves that on the CPU from faar_gemm_plan), and so that the shapes
the benchmark times are compared with the oracle at their full size.
"""
from __future__ import annotations

import dataclasses


@dataclasses.dataclass(frozen=True)
class StepCase:
    name: str
    O: int
    K: int
    T: int
    seed: int
    quantised_acts: bool = False    # X_q = X with seeded relative noise (stand-in for low-precision activations)
    gated_input: bool = False       # silu(g) * u activations (input of a down projection)
    chained: bool = False           # dY_ext given and dX requested
    full_size: bool = False         # a benchmark shape at its real size: one beta, no repeated variants
    fp32_small: bool = False        # the 256x256 float32 parity configuration (own generator)
    on_boundary: bool = False       # an entry of W_q - W lies on a bf16 rounding boundary where a flip counts (Gram form)
    whole_device: bool = False      # stepped with FAAR_STEP_WHOLE_DEVICE: the token-major dW GEMM may take 192-wide tiles


STEP_CASES = [
    StepCase("config1", 256, 256, 64, 0, fp32_small=True),
    StepCase("ragged", 96, 80, 100, 21, quantised_acts=True, chained=True),   # nothing a multiple of a tile
    StepCase("kproj_slice", 512, 2048, 640, 22),
    StepCase("three_tiles", 320, 256, 300, 23, quantised_acts=True, chained=True),
    StepCase("wide_two_slices", 12288, 64, 2048, 24),             # one slice of 64
    StepCase("mid_k96", 3072, 96, 2048, 25, quantised_acts=True),
    # small shapes that exist to reach one kernel variant each
    StepCase("tall_k32", 14336, 32, 640, 26),                    # residual / C GEMMs on 256x256 tiles, half a slice
    StepCase("dx_o32_t640", 32, 12288, 640, 27, chained=True),   # dX GEMM: contraction 32, 256x256 tiles
    StepCase("dx_o32_t300", 32, 12288, 300, 28, chained=True),   # dX GEMM: contraction 32, 256x128 tiles
    StepCase("dx_o80", 80, 96, 100, 29, chained=True),           # dX GEMM: ragged contraction
    StepCase("dw_split_256x256", 288, 6144, 4096, 30),           # dW GEMM: 256x256 tiles, contraction split
    StepCase("dw_one_slice", 288, 12288, 33, 31),                # dW GEMM: 256x128 tiles, a single 64-token slice
    # dW GEMM on token-major operands (upstream gradient given): last tiles 8 rows / 16 columns wide, 32 slices split 11 + 11 + 10
    StepCase("dw_token_major_ragged", 3592, 1040, 2048, 32, chained=True),
    # ... with the device to itself: on 192 x 256 tiles (last tile 72 rows x 80 columns) and on 256 x 192 tiles (last 152 x 160),
    # whole and split in three
    StepCase("dw_token_major_192x256", 1032, 7248, 512, 34, chained=True, whole_device=True),
    StepCase("dw_token_major_256x192", 8088, 1312, 512, 35, chained=True, whole_device=True),
    StepCase("dw_token_major_192x256_split", 528, 6576, 2048, 36, whole_device=True),
    StepCase("dw_token_major_256x192_split", 6576, 528, 2048, 37, whole_device=True),
    StepCase("dw_token_major_256x192_split_long", 6576, 528, 4096, 38, whole_device=True),
    StepCase("dw_split_256x128", 6576, 272, 2048, 39),           # dW GEMM: 256x128 tiles, contraction split
    StepCase("dx_o16", 16, 3072, 4096, 48, chained=True),        # dX GEMM: contraction 16
    # token-major dY out of the residual GEMM (with H): contractions that end 32 into a slice, last tiles of 256 x 64 outputs
    StepCase("rows_k160_t6144", 14336, 160, 6144, 49),
    StepCase("rows_k544", 4416, 544, 8192, 50),
    # residual contractions that end inside a slice: 16 and 48 of 64 on 128x64 tiles, 16 on 128x128 (config-sized ones above: 32)
    StepCase("tail_16", 272, 80, 192, 45, chained=True),
    StepCase("tail_48", 136, 624, 520, 46, chained=True),
    StepCase("tail_128x128", 1000, 208, 3001, 47),
    # token-major dY out of the residual GEMM (with H) on 256x256 tiles, contraction ending 32 into a slice
    StepCase("rows_k160", 12288, 160, 4096, 33),
    # the shapes the benchmark times, at full size
    StepCase("llama_q_proj", 2048, 2048, 4096, 0, full_size=True),
    StepCase("llama_k_proj", 512, 2048, 4096, 8, full_size=True),
    StepCase("llama_gate_proj", 8192, 2048, 4096, 1, chained=True, full_size=True),
    StepCase("llama_down_proj", 2048, 8192, 4096, 2, gated_input=True, chained=True, full_size=True),
    StepCase("qwen_k_proj", 1024, 2048, 8192, 3, quantised_acts=True, chained=True, full_size=True),
    StepCase("qwen_q_proj", 2048, 2048, 8192, 5, full_size=True),                       # the default benchmark's q / o projection
    StepCase("qwen_down_proj", 2048, 6144, 8192, 6, gated_input=True, full_size=True, whole_device=True),   # ... its down projection
    StepCase("qwen_gate_proj", 6144, 2048, 8192, 7, full_size=True, whole_device=True),   # ... and its gate / up projection
    StepCase("qwen_gate_proj_T16384", 6144, 2048, 16384, 4, chained=True, full_size=True),
]

# Cases only the Gram-matrix form of the step runs (tests/test_gpu_gram.py, next to all of STEP_CASES): shapes whose
# O x K x K product takes a kernel variant none of the above reaches with that epilogue
GRAM_CASES = [
    StepCase("gram_256x128_split", 1024, 2112, 256, 41),          # 256x128 tiles, contraction split
    StepCase("gram_256x128_k64", 4096, 1088, 192, 42),            # 256x128 tiles, whole
    StepCase("gram_256x128_k32", 4096, 1056, 192, 43),            # 256x128 tiles, contraction ending 32 into a slice
    StepCase("gram_256x128_split_k3072", 656, 3072, 256, 44),
    StepCase("gram_o400_k6144", 400, 6144, 192, 51),              # contraction split, last tiles of 16 and of 176 rows
    StepCase("gram_o688_k6144", 688, 6144, 192, 53),
    StepCase("gram_o688_k6144_boundary", 688, 6144, 192, 52, on_boundary=True),   # see tests/boundary_flips.py
    # contraction split, the last split ending 16 and 48 into a slice: on 256x256, 256x128, 128x128 and 128x64 tiles
    StepCase("gram_256x256_split_k16", 272, 5584, 192, 60),
    StepCase("gram_256x256_split_k48", 272, 5616, 192, 61),
    StepCase("gram_256x128_split_k16", 160, 5392, 192, 62),
    StepCase("gram_256x128_split_k48", 160, 5424, 192, 63),
    StepCase("gram_128x128_split_k16", 16, 4112, 192, 64),
    StepCase("gram_128x128_split_k48", 16, 4144, 192, 65),
    StepCase("gram_128x64_split_k16", 16, 1040, 192, 66),
    StepCase("gram_128x64_split_k48", 16, 1072, 192, 67, on_boundary=True),
]

# (O, K, T) of layers that between them run every GEMM instantiation -- epilogue, tile, contraction whole or split, ending with a slice,
# in its first half or in its second, and with fewer slices than the ring of stages or more -- which the cases above do not
# (tests/test_gpu_variants.py runs all of a layer's products on them, tests/test_plan_coverage.py counts)
VARIANT_SHAPES = [
    (6144, 16, 300), (6144, 64, 300), (6144, 320, 300), (320, 272, 8192), (16, 1040, 2048), (64, 1040, 2048),        # 128-row tiles
    (12288, 16, 300), (12288, 48, 300), (12288, 64, 300), (12288, 240, 300), (14336, 272, 300), (14336, 304, 64),   # 256x128
    (48, 1040, 4096), (64, 1040, 4096), (272, 320, 16384), (432, 1040, 4096),
    (1040, 16, 8192), (1040, 48, 8192), (1040, 64, 8192), (1040, 144, 8192), (1040, 176, 8192), (12288, 192, 64),   # 256x256
    (12288, 192, 640), (14336, 560, 64), (48, 2064, 4096), (64, 2064, 4096), (160, 2064, 4096), (432, 2064, 4096),
    (14336, 640, 192), (14336, 528, 512), (14336, 560, 512), (14336, 560, 640),                                     # dY token-major
    (520, 4096, 16384), (4104, 1280, 8192),                                                                         # dX on W_q^T
    (8256, 1360, 64), (8256, 1392, 64), (8256, 1408, 64), (7552, 560, 64),            # Gram form: a pass over V of its own, 256x256, 256x128
    (3072, 5584, 64), (3072, 5584, 300), (6144, 4112, 64), (6144, 4112, 192),         # dW: likewise, whole, 256x128 and 256x256
]

BY_NAME = {c.name: c for c in STEP_CASES + GRAM_CASES}
