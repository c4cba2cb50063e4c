"""CPU-only: the layer-step parity cases together reach every GEMM kernel variant the library can pick.

faar_gemm_plan is a pure host function that reports the variant (tile shape, contraction split)
the library uses for each GEMM of a layer.  The set of (GEMM, variant, split or not) combinations that ANY layer
shape can produce is found by scanning a wide grid of shapes; the parity cases must cover all of it, so that no
kernel instantiation runs in the benchmark without having been compared with the oracle."""
import itertools

from paper_2603_22370_amd import binding as fb

from parity_cases import GRAM_CASES, STEP_CASES, VARIANT_SHAPES
from test_gpu_rounds import FORWARD as WALKED_FORWARD, STEP as WALKED_STEP
from test_gpu_small_step import SHAPES as SMALL_SHAPES
from test_gpu_update_in_product import DW as UPDATE_DW, GRAM as UPDATE_GRAM

GEMMS = {"residual": fb.K_GEMM_RESIDUAL, "dw": fb.K_GEMM_DW, "dx": fb.K_GEMM_DX, "c": fb.K_GEMM_C}
DIMS = [16, 32, 48, 64, 80, 96, 128, 160, 192, 224, 256, 288, 320, 384, 448, 512, 640, 768, 1024, 1280, 1536, 2048,
        2560, 3072, 4096, 6144, 8192, 12288, 14336, 16384]
TOKENS = [1, 3, 33, 64, 65, 100, 128, 256, 300, 512, 640, 1024, 1536, 2048, 3072, 4096, 8192, 16384, 65536]


# shapes (O, K, T) on which tests/test_gpu_block.py compares faar_linear_forward with the oracle
FORWARD_CASES = [(96, 80, 100), (640, 256, 300), (2048, 512, 1024), (6144, 2048, 2048), (640, 256, 300), (256, 640, 300)]


def _combos(O, K, T, chained):
    for g, which in GEMMS.items():
        if g == "dx" and not chained:
            continue
        kind, bm, bn, split = fb.faar_gemm_plan(which, O, K, T)
        yield (g, kind, (bm, bn), "split" if split > 1 else "whole")


def test_parity_cases_reach_every_gemm_variant():
    reachable = {}
    for O, K, T in itertools.product(DIMS, DIMS, TOKENS):
        if O * K * T > 2 ** 40:
            continue
        for combo in _combos(O, K, T, chained=(O % 8 == 0)):
            reachable.setdefault(combo, (O, K, T))
    covered = set()
    for c in STEP_CASES:
        covered.update(_combos(c.O, c.K, c.T, c.chained))
    missing = {k: v for k, v in reachable.items() if k not in covered}
    assert not missing, f"variants no parity case reaches (with an example shape): {missing}"
    # every variant name the library knows is reachable by some GEMM, so none is dead code
    assert {k[1] for k in reachable} == set(fb.GEMM_KINDS)


def test_tiles_192_wide_are_only_for_a_step_that_has_the_device_to_itself():
    """They fill compute units that 256-wide tiles leave idle, which are not idle where other streams share the device: only
    the token-major dW GEMM takes them, and only where the caller says it is alone (FAAR_STEP_WHOLE_DEVICE)."""
    dims = DIMS + [1152, 2304, 5120]
    for O, K, T in itertools.product(dims, dims, [64, 512, 2048, 4096, 8192, 16384]):
        if O * K * T <= 2 ** 40:
            for which in (*GEMMS.values(), fb.K_GEMM_FWD, fb.K_GEMM_GRAM):
                assert 192 not in fb.faar_gemm_plan(which, O, K, T)[1:3], (which, O, K, T)
            assert fb.faar_dw_token_major(O, K, T) in (0, 1)


def test_benchmark_shapes_are_parity_cases_at_full_size():
    """Every (variant, split) the Llama3-1B- and Qwen3-1.7B-shaped linears take at the benchmark's token counts is
    also taken by a full-size parity case (several contraction slices, ring wrap-around, all tiles)."""
    llama = [(2048, 2048), (512, 2048), (8192, 2048), (2048, 8192)]
    qwen = [(2048, 2048), (1024, 2048), (6144, 2048), (2048, 6144)]
    full = set()
    for c in STEP_CASES:
        if c.full_size:
            full.update(_combos(c.O, c.K, c.T, c.chained))
    for shapes, T, chained in ((llama, 4096, False), (qwen, 8192, False), (qwen, 16384, True)):
        for O, K in shapes:
            for combo in _combos(O, K, T, chained):
                assert combo in full, (O, K, T, combo)


def test_forward_gemm_of_the_joint_step_runs_kernels_that_parity_cases_cover():
    """faar_linear_forward uses the bf16-output GEMM (the dX GEMM's epilogue) on T x O x K: every variant it takes on the
    joint benchmark's shapes is a variant some parity case reaches with that epilogue (as dX GEMM or as forward GEMM)."""
    covered = set()
    for c in STEP_CASES:
        if c.chained:
            kind, bm, bn, _ = fb.faar_gemm_plan(fb.K_GEMM_DX, c.O, c.K, c.T)
            covered.add((kind, bm, bn))
    for O, K, T in FORWARD_CASES:
        kind, bm, bn, _ = fb.faar_gemm_plan(fb.K_GEMM_FWD, O, K, T)
        covered.add((kind, bm, bn))
    for O, K in ((6144, 2048), (2048, 6144)):
        kind, bm, bn, _ = fb.faar_gemm_plan(fb.K_GEMM_FWD, O, K, 16384)
        assert (kind, bm, bn) in covered, (O, K, kind)


def test_gram_form_product_runs_kernels_that_its_parity_cases_cover():
    """The O x K x K product of faar_layer_step_gram: every (variant, tile, split or not) any layer shape can take is taken
    by one of the cases tests/test_gpu_gram.py runs (all of STEP_CASES and GRAM_CASES), and the benchmark's layer shapes by full-size ones."""
    def combo(O, K):
        kind, bm, bn, split = fb.faar_gemm_plan(fb.K_GEMM_GRAM, O, K, 1)
        return (kind, (bm, bn), "split" if split > 1 else "whole")

    reachable = {}
    for O, K in itertools.product(DIMS, DIMS):
        if K % 16 == 0:
            reachable.setdefault(combo(O, K), (O, K))
    covered = {combo(c.O, c.K) for c in STEP_CASES + GRAM_CASES}
    missing = {k: v for k, v in reachable.items() if k not in covered}
    assert not missing, f"Gram-form variants no parity case reaches (with an example shape): {missing}"
    full = {combo(c.O, c.K) for c in STEP_CASES if c.full_size}
    for O, K in [(2048, 2048), (512, 2048), (8192, 2048), (2048, 8192), (1024, 2048), (6144, 2048), (2048, 6144)]:
        assert combo(O, K) in full, (O, K, combo(O, K))


def test_token_major_residual_gemm_runs_kernels_that_parity_cases_cover():
    """Where faar_dw_token_major holds, a step that carries the constant as H leaves dY token-major: its residual GEMM is the
    T x O x K product planned like the forward GEMM, with an epilogue of its own.  Every variant that product can take on such
    a shape is taken by a parity case (each runs once with H, no upstream gradient and no dX), and the benchmark's by
    full-size ones."""
    def combo(O, K, T):
        kind, bm, bn, _ = fb.faar_gemm_plan(fb.K_GEMM_FWD, O, K, T)
        return (kind, (bm, bn))

    reachable = {}
    for O, K, T in itertools.product(DIMS, DIMS, TOKENS):
        if O * K * T <= 2 ** 40 and fb.faar_dw_token_major(O, K, T):
            reachable.setdefault(combo(O, K, T), (O, K, T))
    covered = {combo(c.O, c.K, c.T) for c in STEP_CASES if fb.faar_dw_token_major(c.O, c.K, c.T)}
    missing = {k: v for k, v in reachable.items() if k not in covered}
    assert not missing, f"token-major residual variants no parity case reaches (with an example shape): {missing}"
    full = {combo(c.O, c.K, c.T) for c in STEP_CASES if c.full_size and fb.faar_dw_token_major(c.O, c.K, c.T)}
    for O, K in [(2048, 2048), (1024, 2048), (6144, 2048), (2048, 6144)]:
        assert not fb.faar_dw_token_major(O, K, 8192) or combo(O, K, 8192) in full, (O, K)
    assert fb.faar_dw_token_major(6144, 2048, 8192) and fb.faar_dw_token_major(2048, 6144, 8192)


def test_token_major_dw_gemm_tiles_are_all_reached_by_parity_cases():
    """The token-major dW GEMM has three tile shapes (two of them only for a step that has the device to itself), each whole or
    with the contraction split: every combination some layer shape takes is taken by a parity case (each runs it with H and
    its own gradient; chained ones also with an upstream one)."""
    def combo(O, K, T, whole_device):
        return (fb.faar_dw_token_major(O, K, T, whole_device), "split" if fb.faar_gemm_plan(fb.K_GEMM_DW, O, K, T)[3] > 1 else "whole")

    reachable = {}
    dims = DIMS + [528, 1032, 1312, 6576, 7248, 8088]
    for O, K, T in itertools.product(dims, dims, TOKENS):
        if O * K * T <= 2 ** 40 and fb.faar_dw_token_major(O, K, T):
            assert fb.faar_dw_token_major(O, K, T) == 1
            for whole_device in (False, True):
                reachable.setdefault(combo(O, K, T, whole_device), (O, K, T))
    assert {k[0] for k in reachable} == {1, 2, 3}
    token_major = [c for c in STEP_CASES if fb.faar_dw_token_major(c.O, c.K, c.T)]
    covered = {combo(c.O, c.K, c.T, c.whole_device) for c in token_major}
    missing = {k: v for k, v in reachable.items() if k not in covered}
    assert not missing, f"token-major dW variants no parity case reaches (with an example shape): {missing}"
    assert {combo(c.O, c.K, c.T, c.whole_device)[0] for c in token_major if c.chained} == {1, 2, 3}
    # alone on the device, the default benchmark's two large shapes take the 192-wide tiles, and full-size parity cases run them
    full = {combo(c.O, c.K, c.T, c.whole_device) for c in STEP_CASES if c.full_size}
    assert combo(6144, 2048, 8192, True) == (2, "whole") and combo(2048, 6144, 8192, True) == (3, "whole")
    assert combo(6144, 2048, 8192, True) in full and combo(2048, 6144, 8192, True) in full
    # ... and beside other streams 256 x 256 ones, split or not, which full-size cases run as well
    assert {(1, "whole"), (1, "split")} <= full


def test_products_that_update_v_have_a_slot_for_every_work_item():
    """A work item of a dW product that ends in the pass over V leaves one partial sum of the next step's losses, and a step has one slot
    for every 2048 weights, at most 2048: the tiles that a whole product is launched on are no more than that, whatever shape it takes."""
    bm_bn = {1: (256, 256), 2: (192, 256), 3: (256, 192)}
    rows = [96, 800, 2560, 5120, 6144, 6656, 8192, 10240, 14592, 16640, 17920, 18432, 20480, 24576, 65536]
    seen = set()
    for O, K, T in itertools.product(rows + [8 * n for n in range(600, 2600, 37)], [r // 16 * 16 for r in rows], [64, 512, 2048, 8192, 16384]):
        if O * K > 2 ** 28 or O * K * T > 2 ** 42 or not fb.faar_gemm_form(fb.K_GEMM_DW, O, K, T):
            continue
        slots = min(2048, -(-O * K // 2048))
        _, bm, bn, split = fb.faar_gemm_plan(fb.K_GEMM_DW, O, K, T)
        assert split == 1 and -(-O // bm) * -(-K // bn) <= slots, (O, K, T)
        for alone in (False, True):
            tiles = fb.faar_dw_token_major(O, K, T, alone)
            if tiles:
                bm, bn = bm_bn[tiles]
                assert -(-O // bm) * -(-K // bn) <= slots, (O, K, T, alone)
                seen.add((alone, tiles))
    assert seen == {(False, 1), (True, 1), (True, 2), (True, 3)}


def test_forms_are_taken_where_they_were_measured_to_be_faster():
    """On both sides of the lines that the rules draw: shapes that took longer in one launch, with the update inside a product, or
    with it on fewer compute units."""
    form = fb.faar_gemm_form
    for O, K in [(2048, 2112), (4352, 1024), (4096, 1088), (8192, 544), (3584, 3584), (7168, 1792), (5696, 2976), (8128, 5712), (8192, 8192),
                 (4096, 3072), (2048, 5120), (7168, 4736)]:
        assert form(fb.K_GEMM_GRAM, O, K, 1) == 0, (O, K)
    for O, K in [(2048, 2048), (2048, 6144), (6144, 2048), (2560, 2560), (3072, 3072), (4096, 4096), (2048, 8192), (2304, 5376), (2688, 4608),
                 (4608, 2688)]:
        assert form(fb.K_GEMM_GRAM, O, K, 1) == fb.FORM_UPDATES_V, (O, K)
    both = fb.FORM_UPDATES_V | fb.FORM_UPDATES_V_WITH_DX
    for O, K, T, want in [(4208, 7760, 1920, 0), (5440, 6576, 3136, 0), (5760, 7344, 704, 0), (2432, 4048, 3062, fb.FORM_UPDATES_V),
                          (2816, 5968, 324, 0), (4480, 4224, 1984, fb.FORM_UPDATES_V), (1728, 5952, 1234, both), (3072, 3072, 4096, both),
                          (6144, 2048, 8192, both), (2048, 8192, 4096, both), (4096, 6784, 704, both)]:
        assert form(fb.K_GEMM_DW, O, K, T) == want, (O, K, T)
    for O, K, T, want in [(64, 1024, 16, 0), (256, 512, 32, 0), (256, 384, 64, 0), (256, 320, 96, 0), (256, 256, 192, 0), (256, 256, 128, 4),
                          (1024, 128, 256, 4), (256, 320, 64, 4)]:
        assert form(fb.K_GEMM_RESIDUAL, O, K, T) == want, (O, K, T)


STAGES = {"L64": 2, "M64": 3, "S64": 4, "N64": 6}      # slices the ring of a tile shape holds


def _instantiation(epilogue, which, contraction, O, K, T):
    """(epilogue, tile, split, where the contraction ends in its last slice, whether a work item walks more slices than the ring
    holds).  Only the tiles of 256 rows treat the two halves of a slice differently."""
    kind, _, _, split = fb.faar_gemm_plan(which, O, K, T)
    slices, tail = (contraction + 63) // 64, contraction % 64
    ends = "whole" if tail == 0 else "tail" if kind in ("S64", "N64") else "half" if tail <= 32 else "more"
    return (epilogue, kind, "split" if split > 1 else "one", ends, "wraps" if -(-slices // split) > STAGES[kind] else "short")


def _widths(O, K):
    """The tile of a Gram-form product that ends in the pass over V, where the plan says 256x256: rounds of 256 units, by area, and
    192-wide ones up to the contraction that their limit is."""
    cost = {(bm, bn): -(-(-(-O // bm) * -(-K // bn)) // 256) * bm * bn for bm, bn in ((256, 256), (192, 256), (256, 192))}
    tile = min(cost, key=lambda t: (cost[t], t != (256, 256), t != (192, 256)))
    return tile if K <= {(256, 256): K, (192, 256): 4608, (256, 192): 2688}[tile] else (256, 256)


def _gram_instantiation(O, K):
    x = _instantiation("gram", fb.K_GEMM_GRAM, K, O, K, 1)
    if fb.faar_gemm_form(fb.K_GEMM_GRAM, O, K, 1) & fb.FORM_UPDATES_V:
        assert x[2] == "one"
        return ("gram, update", _widths(O, K) if x[1] == "L64" else x[1], x[3])
    return x


def _dw_instantiations(O, K, T, alone, nt=True, with_dx=False):
    """The dW product on transposed operands (nt: a step of the caller's takes them also where the token-major ones would do) and on the
    token-major ones, in a step that produces dX or in one that does not."""
    x = _instantiation("dw", fb.K_GEMM_DW, (T + 63) // 64 * 64, O, K, T)
    tiles = fb.faar_dw_token_major(O, K, T, alone)
    if fb.faar_gemm_form(fb.K_GEMM_DW, O, K, T) & (fb.FORM_UPDATES_V_WITH_DX if with_dx else fb.FORM_UPDATES_V):
        assert x[2] == "one"
        if nt or not tiles:
            yield ("update", x[1])
        if tiles:
            yield ("update", f"token-major {tiles}")
    elif nt or not tiles:
        yield x


def _walk(epilogue, which, contraction, O, K, T):
    if fb.faar_gemm_form(which, O, K, T) & fb.FORM_WALKS_TILES:
        assert fb.faar_gemm_plan(which, O, K, T)[0] == "L64" and contraction % 64 == 0
        return (epilogue + ", walked", "odd" if contraction // 64 % 2 else "even")
    return _instantiation(epilogue, which, contraction, O, K, T)


def _instantiations(O, K, T, chained=True, forward=True, alone=(False,), own_dx=True):
    """Everything a layer's set-up, steps (both forms; chained: also with an upstream gradient and dX; own_dx: with dX of their own
    gradient), Gram-form step and forward run."""
    small = fb.faar_gemm_form(fb.K_GEMM_RESIDUAL, O, K, T) & fb.FORM_WHOLE_STEP
    if small:
        yield ("small", "one group of columns" if K <= 256 else "more", "one group of tokens" if T <= 256 else "more")
    else:
        yield _walk("rows" if fb.faar_dw_token_major(O, K, T) else "perturbation", fb.K_GEMM_RESIDUAL_H, K, O, K, T)
    if not small or chained and own_dx:
        yield _instantiation("residual", fb.K_GEMM_RESIDUAL, K, O, K, T)
    for a in alone:
        if not small:
            yield from _dw_instantiations(O, K, T, a)
        if chained:
            yield from _dw_instantiations(O, K, T, a, own_dx, True)
    yield _instantiation("c", fb.K_GEMM_C, K, O, K, T)
    yield _gram_instantiation(O, K)
    if chained:
        yield _instantiation("loss", fb.K_GEMM_LOSS, K, O, K, T)
        yield _instantiation("loss_h", fb.K_GEMM_LOSS_H, K, O, K, T)
        # wide layers of many tokens, and products that fill less than three quarters of the chip with 256x256 tiles: on a transposed
        # copy of W_q, with the kernels of the forward
        on_copy = fb.faar_gemm_form(fb.K_GEMM_DX, O, K, T) & fb.FORM_ON_COPY
        yield _walk("forward" if on_copy else "dx", fb.K_GEMM_DX, O, O, K, T)
    if forward:
        yield _walk("forward", fb.K_GEMM_FWD, K, O, K, T)


def test_every_gemm_instantiation_is_compared_with_an_oracle():
    """Over layer shapes that end in every place of a slice, the epilogues that only some steps use among them: each instantiation that
    a shape reaches is run by a parity case, by tests/test_gpu_variants.py or by the tests of the products that update V, walk their
    tiles or are a whole step."""
    outs = [16, 48, 64, 96, 160, 256, 272, 320, 432, 640, 1000, 1040, 1280, 2048, 3072, 4096, 6144, 8192, 12288, 14336]
    ins = [16, 32, 48, 64, 80, 112, 144, 176, 192, 240, 256, 272, 304, 320, 432, 528, 560, 640, 1024, 1040, 1072, 2048, 2064, 2096,
           3072, 4112, 4144, 5584, 5616, 6144]
    tokens = [1, 33, 64, 65, 128, 192, 300, 512, 640, 1024, 2048, 4096, 8192, 16384]
    reachable = {}
    for O, K, T in itertools.product(outs, ins, tokens):
        if O * K * T <= 2 ** 38:
            for x in _instantiations(O, K, T, alone=(False, True)):
                reachable.setdefault(x, (O, K, T))
    covered = {_gram_instantiation(c.O, c.K) for c in GRAM_CASES}
    for c in STEP_CASES:
        covered.update(_instantiations(c.O, c.K, c.T, c.chained, False, (c.whole_device,), own_dx=False))
    for O, K, T in FORWARD_CASES:
        covered.add(_walk("forward", fb.K_GEMM_FWD, K, O, K, T))
    for shape in VARIANT_SHAPES:
        covered.update(_instantiations(*shape))
    for O, K, T, alone in UPDATE_DW:
        covered.update(_dw_instantiations(O, K, T, alone, False))
        covered.update(_dw_instantiations(O, K, T, alone, False, True))
    covered.update(_gram_instantiation(O, K) for O, K in UPDATE_GRAM)
    covered.update(x for O, K, T in SMALL_SHAPES for x in _instantiations(O, K, T, False, False) if x[0] == "small")
    covered.update(_walk("forward", fb.K_GEMM_FWD, K, O, K, T) for O, K, T in WALKED_FORWARD)
    covered.update(_walk("rows", fb.K_GEMM_RESIDUAL_H, K, O, K, T) for O, K, T in WALKED_STEP)
    missing = {k: v for k, v in reachable.items() if k not in covered}
    assert not missing, f"instantiations that no test compares (with an example shape): {missing}"
    assert {k[0] for k in reachable} == {"residual", "rows", "rows, walked", "perturbation", "dw", "update", "c", "gram", "gram, update",
                                         "loss", "loss_h", "dx", "forward", "forward, walked", "small"}
