"""Which kernel a grid takes (host plans, no GPU), on both sides of the rules."""
import pytest

from _plans import FUSED, is_route, route


# wide grids of few rows: single steps where both sides were measured and they won
# by more than the rule's 6 %, tiles where tiles won
@pytest.mark.parametrize("storage,shape,kernel", [
    ("f64", (5, 77792), "single"), ("f64", (8, 286424), "single"), ("f64", (5, 400000), "single"),
    ("f64", (12, 256080), "single"), ("f64", (17, 22144), "tile"), ("f64", (19, 147265), "tile"),
    ("f32", (7, 353696), "single"), ("f32", (6, 33184), "single"), ("f32", (12, 8809), "tile"),
    ("f32", (25, 164760), "tile"), ("f16dev", (5, 320184), "single"), ("f16dev", (17, 400000), "single"),
    ("f16dev", (30, 31016), "tile"), ("f16dev", (185, 55074), "tile"),
    # tall grids of few columns keep tiles: a single step fills 64 lanes per row
    ("f64", (18108, 5), "tile"), ("f16dev", (7346, 5), "tile"),
    # and grids of ordinary aspect
    ("f64", (64, 64), "tile"), ("f32", (2048, 2048), "tile"), ("f16dev", (3089, 2464), "tile")])
@pytest.mark.parametrize("basis", ["default", "geier"])
def test_flat_grids_take_the_faster_kernel(storage, shape, kernel, basis):
    assert route("d2q9", storage, shape, basis)[0] == kernel


@pytest.mark.parametrize("lattice,storage,shape,want", FUSED)
def test_the_compared_grids_take_the_kernels_they_are_listed_for(lattice, storage, shape, want):
    assert is_route(lattice, storage, shape, want), route(lattice, storage, shape)


def test_every_instance_is_compared():
    slides = {(la, s) for la, s, _, w in FUSED if w == "slide"}
    assert slides == {("d3q19", "f32"), ("d3q19", "f64"), ("d3q27", "f32"), ("d3q27", "f64")}
    chunks = [route(la, s, sh)[2] for la, s, sh, w in FUSED if w == "slide"]
    assert any(sh[0] % c for (_, _, sh, w), c in zip([f for f in FUSED if f[3] == "slide"], chunks))  # a short last chunk
    assert min(sh[0] for _, _, sh, w in FUSED if w == "slide") == 4                                    # the fewest planes
