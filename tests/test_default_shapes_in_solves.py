"""The coarsest product's default shape, held against whole solves timed with the
shape pinned: FP64 matrices that are too small to stage x in LDS."""
import pytest

from paper_2508_17517_amd import binding

COARSEST = 6

# rows, entries a row, the solve in ms by the lanes of the coarsest product (no mapping)
MEASURED = [
    (16193, 66, {16: 2.564, 32: 2.698, 64: 3.100}),
    (14252, 67, {16: 2.564, 32: 2.629, 64: 3.010}),
    (14490, 94, {16: 3.497, 32: 3.499, 64: 3.894}),
    (28455, 98, {16: 4.312, 32: 4.490, 64: 5.111}),
    (10794, 191, {16: 5.259, 32: 5.063, 64: 5.198}),
    (13007, 193, {16: 5.198, 32: 5.052, 64: 5.176}),
    (15514, 172, {16: 6.599, 32: 6.463, 64: 6.716}),
    (17421, 197, {16: 8.212, 32: 8.434, 64: 8.529}),
    (22842, 203, {16: 10.226, 32: 10.413, 64: 10.389}),
    (26063, 191, {16: 9.763, 32: 9.861, 64: 9.972}),
    (18750, 247, {16: 12.215, 32: 12.622, 64: 12.394}),
    (19704, 249, {16: 16.620, 32: 17.055, 64: 16.832}),
    (19966, 207, {16: 10.145, 32: 10.490, 64: 10.454}),
    (18228, 284, {16: 27.278, 32: 27.289, 64: 27.292}),
    (26974, 345, {16: 26.491, 32: 26.369, 64: 26.315}),
]


@pytest.mark.parametrize("rows,avg,ms", MEASURED)
def test_coarsest_lanes(rows, avg, ms):
    shape = binding.load_host_dense().airg_host_default_shape(COARSEST, rows, rows * avg, 8, 8, 1, 2600)
    assert not shape & ~255
    # two medians of one solve differ by up to 1%
    assert ms[shape] <= 1.01 * min(ms.values())


# rows, entries a row, bytes of a value and of a vector element, widest window, the
# solve in ms by the shape that stages x (+ 512; + 256 with the XCD mapping)
STAGED = [
    (13382, 197, 4, 4, 2154, {528: 5.122, 784: 5.088, 520: 5.448, 776: 5.409}),
    (15514, 172, 4, 4, 2154, {528: 5.839, 784: 5.729, 520: 6.256, 776: 6.028}),
    (28842, 208, 2, 4, 2500, {528: 9.393, 784: 9.144, 520: 9.997, 776: 9.351}),
    (25298, 133, 2, 4, 2201, {528: 10.872, 784: 10.814, 520: 10.994, 776: 10.947}),
    (28480, 98, 4, 4, 2069, {528: 3.735, 784: 3.644, 520: 3.882, 776: 3.657}),
    (36168, 75, 8, 8, 2256, {528: 6.919, 784: 6.716, 520: 6.651, 776: 6.537}),
    (38775, 190, 8, 8, 3136, {528: 14.874, 784: 14.872, 520: 14.374, 776: 14.358}),
    (42409, 74, 8, 8, 2069, {528: 5.775, 784: 6.024, 520: 5.445, 776: 5.602}),
    (61629, 144, 4, 4, 2167, {528: 17.240, 784: 17.522, 520: 17.252, 776: 17.432}),
    (47308, 294, 8, 8, 3439, {528: 53.031, 784: 53.107, 520: 52.544, 776: 52.511}),
]


@pytest.mark.parametrize("rows,avg,vb,xb,span,ms", STAGED)
def test_coarsest_staged_mapping(rows, avg, vb, xb, span, ms):
    shape = binding.load_host_dense().airg_host_default_shape(COARSEST, rows, rows * avg, vb, xb, 1, span)
    assert ms[shape] <= 1.01 * min(ms.values())
