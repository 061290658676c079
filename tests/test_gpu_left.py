"""Walks whose near-peak list overflows, so that a step leaves them to the table
evaluation: no matrix products where no step could use them."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    from paper_2107_09801_amd import libpsl
    c = libpsl.Context(0)
    yield c
    c.close()


def test_no_products_with_the_list_switched_off(ctx):
    """PSL_OPT_NEAR_LIMIT 0: the time of the products (events around them) is that
    of no launch; a launch over this walk takes more than 0.1 ms."""
    from paper_2107_09801_amd import libpsl
    ctx.set_option(libpsl.OPT_NEAR_LIMIT, 0)
    (w,) = ctx.init_walks(131071, 1, 3)
    ctx.step_batch([w], 2)
    ctx.timing_enable()
    ctx.step_batch([w], 5)
    t = ctx.timing_read()
    assert t["steps"] == 5 and t["lin_ms"] / 5 < 0.05
