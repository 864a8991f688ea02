"""The timed region of bench.py: no full collection of the interpreter that was due before falls into it (CPU)."""
import gc


def test_a_due_collection_is_taken_before_the_clock_starts():
    import bench
    order, made = [], []

    def note(phase, info):
        if phase == "start" and info["generation"] == 2:
            order.append("collection")

    def one():
        made.extend([i] for i in range(2000))     # objects that live on, as the records of a step do
        order.append("step")
        return len(made)

    before, due = gc.get_threshold(), []
    gc.collect()
    try:
        gc.disable()
        n = len(gc.get_objects())
        due.extend([i] for i in range(n))         # far more than a quarter of all objects: a full collection is due
        gc.set_threshold(700, 10, 1)
        gc.callbacks.append(note)
        gc.enable()
        res, seconds, issue = bench.timed_steps(one, 5, lambda: order.append("sync"))
    finally:
        gc.callbacks.remove(note)
        gc.set_threshold(*before)
        gc.enable()
    assert res == 10000 and 0 <= issue <= seconds
    at = order.index("sync")
    assert order[:at] and set(order[:at]) == {"collection"}
    assert order[at:] == ["sync"] + ["step"] * 5 + ["sync"]
