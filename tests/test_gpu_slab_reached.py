"""The small tiles that are built are those that some shape reaches: a grid of shapes over all that decides between them."""
import pytest

pytestmark = pytest.mark.gpu


def built(fp8):
    """(waves, row blocks, vocabulary blocks): in one round of tiles 8 to 16 waves, except the smallest; in several 4."""
    tiles = {(4, mb, 1) for mb in range(1, 5)}
    tiles |= {(4 * nb, mb, nb) for nb in (2, 3) for mb in range(3 if fp8 else 2, 9)}
    if fp8:
        return (tiles - {(8, 6, 2)}) | {(4, mb, nb) for nb in (2, 3) for mb in range(1, 9)} | {(4, mb, 4) for mb in (1, 2, 3)}
    tiles |= {(16, mb, 4) for mb in range(1, 5)} | {(8, 5, 4), (8, 6, 4)}
    return tiles | {(4, mb, 4) for mb in range(1, 7)} | {(4, mb, 3) for mb in range(2, 9)} | {(4, mb, 2) for mb in (2, 3, 6, 7, 8)}


@pytest.mark.parametrize("fp8", [False, True])
def test_built_tiles_are_reached(fp8):
    import paper_2504_20039_amd as aj
    seen = set()
    for mb in (*range(1, 19), 20, 25, 29) if not fp8 else range(1, 18):
        for V in (*range(12289, 60000, 1017), *range(60001, 152064, 3067)):
            for d in (512, 4096) if fp8 else (328,):
                h = aj.aj_create(1, 16 * mb - 14, d, 0, V, aj.AJ_BF16, 1, 0, 0, aj.AJ_W_FP8_E4M3 if fp8 else aj.AJ_W_SAME)
                if "slab" in aj.aj_kernel_name(h):
                    waves, blocks, _ = aj.aj_debug_form(h)
                    seen.add((waves, aj.aj_debug_tile(h)[1] // 16, waves * blocks // 4))
                aj.aj_destroy(h)
    assert seen == built(fp8)
