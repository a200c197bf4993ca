"""Single kernels on the CPU build."""
import pytest

from host_library import host_run


@pytest.mark.parametrize("v,slot", [(2, 0), (17, 3), (2, 2 ** 27 - 1), (2, 2 ** 27), (9, 2 ** 22)])
def test_build_product_at_slot(host_library, v, slot):
    """Blocks whose elements lie below and above 2^32 in the window (a window of
    fewer than six times the occupied orbitals' blocks is not cut any smaller)."""
    host_run(host_library, "seg_slot", v, slot)


@pytest.mark.parametrize("seed", range(6))
def test_forms_of_plain_products(host_library, seed):
    """Two-level rows, columns and contractions with every remainder by four,
    operands in any order and with gaps, rows numbered the other way round and
    products taken transposed, complex factors, outputs added to, written over
    and shared by a batch: one by one and several in a launch."""
    host_run(host_library, "products", seed, 160)


@pytest.mark.parametrize("extents,batch,form,ksplit", [
    ((1, 17, 1, 17, 3, 5), 700, 0, 0), ((1, 17, 3, 11, 1, 9), 1030, 2, 0), ((1, 5, 1, 64, 2, 7), 2050, 36, 0),
    ((4, 16, 1, 7, 1, 10), 2050, 0, 0), ((1, 70, 1, 70, 3, 450), 4, 0, 0), ((1, 64, 1, 16, 5, 220), 64, 0, 0),
    ((1, 16, 1, 64, 1, 1100), 64, 32, 0), ((1, 40, 1, 40, 1, 403), 1, 0, 3), ((1, 40, 1, 40, 13, 31), 1, 0, 7),
    ((2, 9, 3, 6, 5, 24), 2, 1, 2)])
def test_tiles_of_plain_products(host_library, extents, batch, form, ksplit):
    """Enough entries or a contraction long enough for tiles of four blocks a
    wave, in each of their shapes and with k split over waves and workgroups."""
    host_run(host_library, "product", *extents, batch, form, ksplit)


@pytest.mark.parametrize("o,v", [(1, 1), (2, 3), (3, 6), (2, 17)])
@pytest.mark.parametrize("one_by_one", [0, 1])
def test_block_products(host_library, o, v, one_by_one):
    """All groups of columns in a launch, and one at a time as where their panels
    span more than 32-bit offsets reach."""
    host_run(host_library, "block", o, v, one_by_one)
