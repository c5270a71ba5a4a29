"""Parameters as the binding takes them: whatever a program reads them from."""
import pytest

from paper_2008_11578_amd import orca

FIELDS = dict(dt=0.1, time_horizon=2.0, neighbor_dist=5.0, cell_size=0.0, max_neighbors=10,
              pref_is_goal=1, f=((0.5, 1.0), (0.0, 0.5)), par_eps=1e-5)


class Computed:
    """Fields that exist only through attribute look-up (a proxy, a config)."""

    def __getattr__(self, name):
        try:
            return FIELDS[name]
        except KeyError:
            raise AttributeError(name) from None


@pytest.mark.parametrize("given", [FIELDS, Computed()])
def test_params_from_dict_and_from_computed_attributes(given):
    p = orca.make_params(given)
    assert (p.max_neighbors, p.pref_is_goal) == (10, 1)
    assert [list(r) for r in p.f] == [[0.5, 1.0], [0.0, 0.5]]
    assert list(p.accel) == [0.0, 0.0] and list(p.turn) == [0.0, 0.0]


@pytest.mark.parametrize("f", [((0.5, 1.0),), ((0.5,), (0.0, 0.5)), ()])
def test_short_responsibility_table_is_refused(f):
    with pytest.raises(IndexError):
        orca.make_params(dict(FIELDS, f=f))
