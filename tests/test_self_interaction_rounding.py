"""Rounding of one application of the self-interaction, measured on the host build of the kernels'
arithmetic (no GPU): the state passes through it with at most four roundings of its full magnitude."""
import os
import subprocess

import pytest

from paper_1907_12834_amd.build import CSRC, hipcc

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def measured(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "u_rounding")
    subprocess.run([hipcc(), "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-mfma", "-ffp-contract=fast",
                    "-I", CSRC, os.path.join(HERE, "host", "u_rounding.cpp"), "-o", exe], check=True)
    rows = [line.split() for line in subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()]
    return {(r[0], float(r[1])): (float(r[2]), float(r[3])) for r in rows}


@pytest.mark.parametrize("dtype,unit", [("c128", 2.0 ** -53), ("c64", 2.0 ** -24)])
@pytest.mark.parametrize("amp", [0.05, 0.3, 1.0])
def test_state_is_rounded_a_few_times(measured, dtype, unit, amp):
    # One rounding to nearest errs by unit/sqrt(3) RMS in the last place of a mantissa of 1, and a
    # mantissa in [1, 2) is 1.47 RMS (logarithmic distribution): 0.39 unit of the value.  Four
    # independent ones: 0.79 unit; 5 % more for the corrections, a few hundredths of the state.
    # The norm's relative change is twice the mean of 20 such errors' projections on the state:
    # below the error itself.
    err, norm = measured[dtype, amp]
    bound = 1.05 * 2 * unit / 3 ** 0.5 / 1.47
    assert err <= bound and norm <= bound, (err / unit, norm / unit)
