"""Resources of the built kernels, from the metadata of the library's code
objects (no GPU needed): a kernel's scratch memory holds spilled registers
and nothing else.  An array or a struct that ends up there (a select between
two of its entries becomes one between their addresses) is read back through
memory at every use."""
import re

import pytest

import device_code

pytestmark = pytest.mark.skipif(not device_code.available(), reason="library or LLVM tools not there")


def _kernels(tmp):
    out = {}
    for obj in device_code.code_objects(tmp):
        for part in device_code.metadata(obj).split("- .agpr_count:")[1:]:
            get = lambda key: re.search(r"\.%s:\s+(\S+)" % key, part).group(1)
            out[get("symbol")] = (int(get("private_segment_fixed_size")), int(get("vgpr_spill_count")),
                                  int(get("sgpr_spill_count")))
    return out


# kernels for boxes and bands without a bound on their size
GENERAL = re.compile(r"\d(k_basis|k_particular|k_smooth|k_bandlu_blocked)E")


def test_scratch_holds_spills_only(tmp_path):
    ks = _kernels(tmp_path)
    assert len(ks) > 60
    # four bytes per spilled register, rounded up to 16 bytes
    bad = {k: v for k, v in ks.items() if v[0] > 4 * v[1] + 15 and not GENERAL.search(k)}
    assert not bad, bad
