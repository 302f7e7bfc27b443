"""How many compute units a device has is asked of the runtime in one place, once per device: a launch whose grid
depends on it does not ask again (0.11 us a call)."""
import glob
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_unit_count_is_looked_up_in_one_place():
    sources = [p for ext in ("hip", "h") for p in glob.glob(os.path.join(ROOT, "paper_2203_09044_amd", "csrc", "*." + ext))]
    asks = [os.path.basename(p) for p in sources for line in open(p) if "hipDeviceAttributeMultiprocessorCount" in line]
    assert asks == ["api.hip"]
