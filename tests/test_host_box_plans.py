"""Which elementwise calls go out in boxes of any extents, and what their boxes cover (no GPU needed)."""
import paper_1810_08723_amd as ocn

BASES = (0x10000000000, 0x20000000000, 0x30000000000)  # far apart: never dereferenced


def _tensor(dtype, es, sizes, strides, which):
    if strides is None:
        strides, acc = [], es
        for n in reversed(sizes):
            strides.insert(0, acc)
            acc *= n
    return ocn.Tensor(BASES[which], dtype, tuple(sizes), tuple(strides), 0, 0)


def _unary(dtype, es, sizes, sa, so=None):
    return ocn.plan_unary("neg", _tensor(dtype, es, sizes, sa, 1), _tensor(dtype, es, sizes, so, 0))


def _binary(dtype, es, sizes, sa, sb, so=None):
    broadcast = [1 if s == 0 else n for n, s in zip(sizes, sb)]
    return ocn.plan_binary("add", _tensor(dtype, es, sizes, sa, 1), _tensor(dtype, es, broadcast, sb, 2),
                           _tensor(dtype, es, sizes, so, 0))


def test_an_operand_cut_off_in_memory_does_not_take_the_box():
    # b is stepped: no extent makes its runs longer, and the output's axis has 14 elements to cover
    p = _binary("double", 8, (196528, 14), (8, 196528 * 8), (16, 0))
    assert p["tile_log2"][1] >= 3
    # a has two elements together and a gap, the output long runs
    p = _unary("double", 8, (4, 300, 500), (8, 64, 19200))
    assert p["tile_log2"][2] >= 4


def test_parts_of_whole_vectors():
    # five parts of 64 bytes, not of 58: the rest of a vector is stored byte by byte
    p = _unary("uint8", 1, (50001, 289), (1, 50001))
    assert p["vec"] == 16 and p["lds_bytes"] == 64 * (64 + 16) and p["grid"] == (50001 + 63) // 64 * 5


def test_no_boxes_of_a_few_elements():
    # five axes, of which a box covers four: the short ones
    sizes = (2, 5, 8668, 2, 3)
    p = _binary("float", 4, sizes, (1040160, 208032, 24, 12, 4), (4, 16, 240, 8, 80))
    assert 2 * 5 * 8668 * 2 * 3 >= p["grid"] * 64 * p["vec"]
    # thousands of boxes, each less than an element per lane
    p = ocn.plan_binary("gt", _tensor("double", 8, (16656, 4, 2, 8, 2), (1024, 256, 128, 16, 8), 1),
                        _tensor("double", 8, (16656, 4, 2, 8, 2), (256, 4263936, 8, 16, 128), 2),
                        _tensor("bool", 1, (16656, 4, 2, 8, 2), None, 0))
    assert 16656 * 128 >= p["grid"] * 256


def test_lanes_do_not_read_from_the_same_banks():
    # a run of 8 x 189 elements in LDS, read eight elements apart: tiles, whose rows are padded
    assert _unary("int32", 4, (8, 189, 4751), (4, 152032, 32))["tile_log2"] == (3, 9)


def test_no_staging_of_two_bytes_at_a_time():
    # six bytes from pair to pair: a vector of sixteen bytes would be loaded for each
    assert not _unary("int16", 2, (48, 157000, 2), (6, 288, 2), (2, 96, 15072000))["stage_a"]
    # vectors of sixteen outputs of which two lie together
    assert not _unary("uint8", 1, (4, 161832, 2), (1, 4, 647328), (970992, 6, 1))["stage_a"]


def test_few_boxes_of_bytes():
    # a few thousand bytes in three orders: vectors of sixteen leave most lanes without work
    p = _binary("uint8", 1, (9, 262), (1, 9), (1, 9))
    assert not p["stage_a"] and not p["stage_b"]
