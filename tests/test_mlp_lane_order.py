"""The gradient kernel hands dL/da1 from lane to lane of one wavefront through LDS,
without a barrier.  The hardware keeps such accesses in order; the compiler has to be
told, and whether it was cannot be seen in the results, so this looks at the source."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "paper_2002_05024_amd", "csrc", "mlp.hip")


def test_fence_between_store_and_load():
    text = re.sub(r"//[^\n]*", "", open(SOURCE).read())
    store = text.index("d1[4 * lg + r][col] = ")
    load = text.index("d1[s][col]", store)
    assert re.search(r"wave_fence\(\)|__syncthreads\(\)", text[store:load])
