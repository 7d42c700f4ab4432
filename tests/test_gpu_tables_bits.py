"""The emission tables' bits.  The FP64 emission tables are made from the Bessel
sums with two shortcuts (terms that are 1e-28 of a sum are left out, halvings of
the search whose outcome the interpolated integrand shows are not evaluated), and
FP64 records of an emission step follow from their bits.  The digests are those
of the tables built without either, every sum in full and every halving
evaluated, one thread per entry; they hold for the math functions of ROCm 7.2."""
import hashlib

import pytest

from gpu_util import need_gpu

pytestmark = pytest.mark.gpu
WIDE = dict(rad_chi_min=1e-6, rad_chi_max=1e6, rad_x_min=-20.0, rad_x_max=30.0, rad_rows=24, f64_refine=2,
            rate_chi_min=1e-9, rate_chi_max=1e7)


@pytest.mark.parametrize("cfg, digests", [
    ({}, dict(cheb_rad="53ba9986cfe91dc1be1a74334ff0c7de", herm_rad="c7a4947fe945d41fe323797eee3684d9",
              cdf32_rad="7f5f1353f31764cbfccf773bd03bd088", cdf64_rad="f7d3ae9c1c1fabfdb52cafd1acdcc0be")),
    (WIDE, dict(cheb_rad="cbe10002a17d45f3367147d9110f988a", herm_rad="9eb4159eb949cb3689a907e6c19a2ba9",
                cdf32_rad="18a03c7ad38fbf3bed5617572c99b023", cdf64_rad="f46831614d625453ece5909c72186ad5")),
])
def test_emission_tables(cfg, digests):
    _, sf = need_gpu()
    tabs = sf.Tables(sf.default_table_cfg(**cfg))
    for part, want in digests.items():
        assert hashlib.sha256(tabs.export(part).tobytes()).hexdigest()[:32] == want, part
