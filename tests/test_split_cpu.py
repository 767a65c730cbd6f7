"""The host rules of wf_split.h (compiled for the host): how tiles are spread over the XCDs, and
the tile of a request-time product."""
import ctypes
import pathlib
import subprocess

import pytest

from test_gpu_products import BATCHED

SRC = pathlib.Path(__file__).parents[1] / "paper_2609_32869_amd" / "csrc"


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    folder = tmp_path_factory.mktemp("split")
    (folder / "split.cpp").write_text(
        f'#include "{SRC}/wf_split.h"\n'
        'extern "C" int row_parts(int m, int n, long b) { return wf::xcd_row_parts(m, n, b); }\n'
        'extern "C" int tile(int rows, int cols, int batch) { return wf::mm_tile(rows, cols, 128, batch).rows; }\n'
        'extern "C" int most(int m, int n, int rs) { return wf::xcd_most_blocks(m, n, rs); }\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", folder / "split.so", folder / "split.cpp"], check=True)
    lib = ctypes.CDLL(str(folder / "split.so"))
    lib.row_parts.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_long]
    return lib


def blocks_of_xcds(nmb, nnb, rs):
    """Tiles of each XCD, from the definition: row part x % rs of rs, column part x / rs of 8 / rs."""
    part = lambda n, parts, i: max(0, min(n, (i + 1) * -(-n // parts)) - i * -(-n // parts))  # noqa: E731
    return [part(nmb, rs, x % rs) * part(nnb, 8 // rs, x // rs) for x in range(8)]


def test_row_parts_keep_the_xcds_busy(lib):
    """No split for the L2's sake that costs the fullest XCD an eighth more blocks a step."""
    for nmb in range(1, 41):
        for nnb in (1, 2, 8, 12, 20, 40, 60, 80, 811):
            for nbytes in (1 << 16, 327680, 655360, 1638400, 1 << 23):
                rs = lib.row_parts(nmb, nnb, nbytes)
                assert rs in (1, 2, 4, 8) and sum(blocks_of_xcds(nmb, nnb, rs)) == nmb * nnb
                assert lib.most(nmb, nnb, rs) == max(blocks_of_xcds(nmb, nnb, rs))
                steps = [max(blocks_of_xcds(nmb, nnb, r)) for r in (1, 2, 4, 8)[:(1, 2, 4, 8).index(rs) + 1]]
                assert all(8 * b <= 9 * a for a, b in zip(steps, steps[1:])), (nmb, nnb, nbytes, rs)


@pytest.mark.parametrize("nmb,nnb,nbytes,want", [
    (9, 20, 1638400, 2), (14, 20, 1638400, 2), (26, 20, 655360, 4),  # uneven parts
    (1, 20, 16 << 20, 1),                                            # a single row block stays spread
    (28, 80, 327680, 4), (14, 80, 327680, 2), (3, 80, 327680, 1)])   # even ones: by bytes
def test_row_parts_measured(lib, nmb, nnb, nbytes, want):
    assert lib.row_parts(nmb, nnb, nbytes) == want


@pytest.mark.parametrize("n_ctx,d,d_ff,want", BATCHED)
def test_tiles_of_the_batched_encoder_test(lib, n_ctx, d, d_ff, want):
    pitch = -(-n_ctx // 64) * 64
    assert pitch % 128 != 0
    rows = {"qkv": (4 * pitch, 3 * d, 1), "o": (4 * pitch, d, 1), "w1": (4 * pitch, d_ff, 1), "w2": (4 * pitch, d, 1),
            "conv1": (4 * 2 * n_ctx, d, 1), "conv2": (n_ctx, d, 4)}
    assert {k: lib.tile(*v) for k, v in rows.items()} == want


def test_tiles_of_large_v3(lib):
    """One request and four: the tiles whose times stand at the rule."""
    assert [lib.tile(1536, n, 1) for n in (5120, 3840, 1280)] == [256, 256, 64]
    assert [lib.tile(6144, n, 1) for n in (5120, 3840, 1280)] == [256, 256, 256]
    assert lib.tile(1500, 1280, 4) == 128 and lib.tile(1536, 2560, 32) == 256
