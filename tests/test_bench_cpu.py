"""The benchmark's own timing: what needs no GPU."""
import gc

import bench


def test_settled_interpreter_has_no_old_objects_to_collect():
    """After settling, a collection inside a timed window looks at new objects only."""
    try:
        keep = [[k] for k in range(100000)]
        bench.settle_interpreter()
        assert gc.get_freeze_count() >= len(keep)
        assert len(gc.get_objects()) < 5000
    finally:
        gc.unfreeze()
