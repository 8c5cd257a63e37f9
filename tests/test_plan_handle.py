"""The sizes a plan handle carries are its own plan's (no GPU): they are asked
for again once the handle, or a bare pointer, holds another plan."""
import ctypes

from paper_1810_06250_amd import rmsynth as B


def test_sizes_follow_the_pointer(monkeypatch):
    asked = []
    monkeypatch.setattr(B, "rmsynth_plan_info",
                        lambda plan: asked.append(plan.value) or dict(nchan=10 * plan.value, nphi=plan.value))
    h = B.PlanHandle(7)
    h.dims = 7, 16, 9
    assert B._plan_dims(h) == (16, 9) and not asked
    h.value = 8
    assert B._plan_dims(h) == (80, 8) and asked == [8]
    assert B._plan_dims(ctypes.c_void_p(3)) == (30, 3)
    assert B._plan_dims(B.PlanHandle(4)) == (40, 4)
