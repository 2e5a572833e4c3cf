"""Which calls take which route, on both sides of the lines that were measured.  No GPU needed."""
import pytest

import routes


# members: one size, or (smallest, largest)
def nnz_of(G, members):
    return G * members if isinstance(members, int) else G * (members[0] + members[1]) // 2 + 1 - G % 2


@pytest.mark.parametrize("V,members,weighted,rows,csr", [
    (4100, 100, False, 5, True), (14000, 13, False, 9, True), (8192, 24, False, 18, True), (10000, 10, False, 48, False),
    (20011, 20, False, 60, False), (30000, 33, False, 9, False), (20000, 32, False, 64, False), (4096, 32, False, 1, False),
    # with weights: 8 lanes a group, two to four turns
    (17000, 20, True, 9, True), (7000, 18, True, 48, False), (7000, 20, True, 64, False), (5000, 28, True, 64, True),
    (7000, 28, True, 64, False), (20000, 32, True, 18, True), (20011, (1, 60), True, 18, False), (9000, (1, 60), True, 36, False),
    (4500, (1, 60), True, 1, True),
    # 16 lanes, four and five
    (20011, 33, True, 12, True), (14000, 33, True, 18, False), (26000, 56, True, 9, True), (4100, (1, 128), True, 64, False),
    (5000, (1, 128), True, 36, True)])
def test_rows_of_a_prepared_membership(V, members, weighted, rows, csr):
    assert routes.rows_from_csr(V, V, nnz_of(V, members), weighted, rows) == csr


@pytest.mark.parametrize("V,members,weighted,B,K,csr", [
    (20000, 32, False, 1, 8, True), (20011, 20, False, 12, 8, True), (20000, 8, False, 32, 8, False), (20000, 32, False, 16, 8, False),
    (65536, 32, False, 1, 8, True), (65536, 32, False, 3, 8, False), (50000, 140, False, 1, 8, False), (65536, 32, True, 1, 8, False),
    (20011, 32, True, 24, 8, True), (14000, (20, 40), True, 18, 8, False), (26000, 56, True, 9, 8, True)])
def test_steps_of_a_prepared_membership(V, members, weighted, B, K, csr):
    assert routes.step_from_csr(V, V, nnz_of(V, members), weighted, B, K) == csr


# of one chunk, slots without padding: one launch or two where that was measured to be ahead of the four from the CSR, and
# where those would take the prepared layout
@pytest.mark.parametrize("V,members,weighted,B,K,launches", [
    (16384, 4, False, 1, 8, 2), (12000, 32, False, 1, 8, 4), (8192, 64, False, 8, 8, 4), (16384, 100, False, 1, 8, 4),
    (16384, 100, True, 1, 8, 4), (16384, 100, True, 8, 8, 4), (6000, 32, True, 64, 8, 2), (12000, 64, False, 8, 8, 4),
    (8192, 64, False, 64, 8, 2), (16384, 100, False, 64, 8, 2), (4096, 100, True, 1, 8, 2), (1024, 8, False, 1, 4, 1),
    (16384, 100, False, 129, 8, 1), (16384, 100, False, 100, 8, 2)])
def test_launches_of_a_small_step(V, members, weighted, B, K, launches):
    assert routes.step_launches(V, V, V * members, weighted, B, K, 1, V * members) == launches


@pytest.mark.parametrize("V,members,B,launches", [(8192, 32, 1, 2), (12000, 16, 64, 4), (16384, 100, 8, 4), (8192, 64, 128, 2)])
def test_launches_where_there_are_chunks(V, members, B, launches):
    assert routes.step_launches(V, V, V * members, False, B, 8, (V + 4095) // 4096, V * members) == launches


# from the CSR: one workgroup a sequence, or four launches where that has too many trips
@pytest.mark.parametrize("V,members,weighted,B,K,launches", [
    (1000, 64, False, 16, 8, 1), (2048, 24, False, 16, 8, 1), (2048, 24, True, 64, 8, 1), (4096, 16, True, 16, 8, 2),
    (5000, 16, False, 1, 8, 2), (5000, 16, True, 1, 8, 4), (5000, 16, True, 64, 1, 1), (3000, 32, False, 16, 8, 4),
    (1000, 100, False, 1, 8, 4), (6000, 8, False, 1, 8, 4), (6144, 12, False, 80, 8, 2), (6144, 4, True, 80, 8, 4),
    (5120, 12, True, 80, 8, 2), (7168, 4, False, 80, 8, 4), (7168, 12, False, 128, 8, 2), (3072, 48, False, 128, 8, 2),
    (4096, 32, True, 128, 8, 2), (8192, 4, False, 128, 8, 4), (5120, 32, True, 128, 8, 4), (12000, 8, False, 130, 8, 1)])
def test_launches_of_a_small_step_from_the_csr(V, members, weighted, B, K, launches):
    assert routes.csr_step_launches(V, V, V * members, weighted, B, K) == launches


def test_the_calls_compared_on_the_gpu_take_both_routes():
    """The sizes of the GPU tests around the lines of few rows lie on the sides they were chosen for."""
    import test_gpu_edges as edges
    params = lambda f: next(m.args[1] for m in f.pytestmark if m.name == "parametrize")
    steps = [routes.step_from_csr(V, G, nnz_of(G, (1, size)), w, B, K) for V, G, size, B, K, _, w in params(edges.test_few_rows)]
    assert steps == [True] * 4 + [False, True, False, True, True, True, False, False, False, False]
    rows = [routes.rows_from_csr(V, V, V * size, False, n) for V, size, n in params(edges.test_few_rows_of_groups_of_one_size)]
    assert rows == [True, False, True, False, True]
    small = [routes.csr_step_launches(V, G, nnz_of(G, (1, size)), w, B, K) for V, G, size, B, K, _, w in params(edges.test_small_steps_from_the_csr)]
    assert small == [1, 1, 2, 2, 1, 2, 1]
    some = [routes.rows_from_csr(V, V, nnz_of(V, (1, 12)), w, n)
            for V, _, n, w in params(edges.test_rows_of_calls_of_different_sizes)]
    assert not any(some)


# chunks of groups and tiles of the vocabulary from the CSR: a few chunks more than run at once where they spare a tile
@pytest.mark.parametrize("V,members,rows,chunks,tiles", [
    (30592, 68, 70, 4, 1), (33720, 133, 55, 5, 1), (27744, 10, 93, 3, 1), (28980, 7, 101, 3, 1), (29706, 4, 127, 3, 1),
    (57588, 64, 49, 6, 2), (60411, 32, 44, 5, 3), (58163, 32, 46, 5, 3), (48852, 4, 85, 4, 2), (20000, 32, 12, 20, 1), (16384, 32, 32, 8, 1)])
def test_chunks_and_tiles_from_the_csr(V, members, rows, chunks, tiles):
    c = routes.csr_shape(V, V, V * members, rows, 256)
    assert (c.nchunks, c.ntiles) == (chunks, tiles)
    assert c.nchunks * c.chunk_groups >= V and c.ntiles * c.tile_len >= V and c.chunk_groups + c.tile_len + 64 <= 40704


def test_every_cut_of_the_csr_fits():
    """Chunks and tiles cover groups and tokens, and a chunk's sums and a tile fit the LDS together, at any number of rows."""
    for V in (1, 63, 64, 4097, 20000, 27000, 30592, 33720, 40576, 40640, 40704, 65536, 81000, 131072, 1000003):
        for G in (1, 33, 4097, 16384, 16385, 30000, V):
            for rows in list(range(1, 140)) + [200, 255, 256, 257, 4096]:
                for mean in (1, 40):
                    c = routes.csr_shape(V, G, G * mean, rows, 256)
                    assert c.nchunks * c.chunk_groups >= G > (c.nchunks - 1) * c.chunk_groups and c.chunk_groups % 16 == 0
                    assert c.ntiles * c.tile_len >= V and c.chunk_groups + c.tile_len + 64 <= 40704 and c.chunk_groups <= 16384


# the split over the XCDs of a gather over the prepared layout (slots without padding): as many parts of the rows
@pytest.mark.parametrize("V,members,weighted,rows,nchunks,parts", [
    (65536, 32, False, 64, 4, 8), (65536, 32, True, 16, 4, (1, 2)), (65536, 32, False, 8, 8, (1, 2, 4)), (32768, 64, False, 128, 2, 8),
    # not all at once: the split that leaves the least to the last turn, or saves bytes and leaves no more
    (50945, 64, True, 49, 5, 8), (50464, 94, False, 33, 7, 8), (50979, 123, False, 38, 7, 8), (35648, 117, False, 54, 5, 8),
    (36772, 115, False, 56, 5, 8), (25336, 24, False, 33, 7, 8), (51092, 128, False, 19, 13, 4), (65507, 32, True, 17, 16, (1, 2))])
def test_split_over_the_chip(V, members, weighted, rows, nchunks, parts):
    m = routes.gather_map(rows, nchunks, 4 * V, V * members * (6 if weighted else 2) // nchunks, False, weighted)
    assert (1 << m.row_shift) in (parts if isinstance(parts, tuple) else (parts,))


# the same from the CSR
@pytest.mark.parametrize("V,members,weighted,rows,parts", [
    (65536, 32, False, 1, 1), (30000, 100, False, 8, (1, 2)), (16384, 32, False, 32, 8), (14987, 8, True, 1, 8), (15569, 10, False, 1, 8),
    (28456, 111, True, 86, 4), (32524, 72, True, 56, 4), (29622, 39, False, 33, 8)])
def test_split_over_the_chip_from_the_csr(V, members, weighted, rows, parts):
    c = routes.csr_shape(V, V, V * members, rows, 256)
    m = routes.gather_map(rows, c.nchunks, 4 * V, V * members * (8 if weighted else 4) // c.nchunks, True, weighted)
    assert (1 << m.row_shift) in (parts if isinstance(parts, tuple) else (parts,))


def test_every_split_reaches_every_row_and_chunk():
    """The kernels' arithmetic on every workgroup of the grid: each (row, chunk) once."""
    for rows in list(range(1, 40)) + [63, 64, 65, 128, 257]:
        for nchunks in (1, 2, 3, 5, 7, 8, 9, 16, 33):
            for row_bytes, chunk_bytes in ((4096, 1 << 22), (262144, 1 << 20), (1 << 20, 64)):
                m = routes.gather_map(rows, nchunks, row_bytes, chunk_bytes, rows % 2 == 0, False)
                grid = 8 * -(-rows // (1 << m.row_shift)) * m.chunks_each
                seen = []
                for b in range(grid):
                    xcd, y = b & 7, b >> 3
                    turn = y // m.chunks_each
                    row = (xcd & ((1 << m.row_shift) - 1)) + (turn << m.row_shift)
                    chunk = (xcd >> m.row_shift) + ((y - turn * m.chunks_each) << (3 - m.row_shift))
                    if row < rows and chunk < nchunks:
                        seen.append((row, chunk))
                assert sorted(seen) == [(r, c) for r in range(rows) for c in range(nchunks)]
