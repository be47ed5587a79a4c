"""What the library's host code asks of the HIP runtime: streams, events and launches counted on a runtime without a
GPU."""
import fake_hip


def test_static_calls_keep_one_set_of_streams(tmp_path):
    """A ragged batch has a chain per width class, forked over side streams: burgers_run_static makes those once, not
    on every call."""
    fake_hip.run("""
batch = W.random_batch(5, 300, 3, 8000, scheme=W.BTCS)
mixed = W.random_batch(6, 300, 3, 30000)
for p in batch.problems + mixed.problems:
    p.dt = 1e-4
for b in (batch, mixed):
    ps, u = problems(b.problems), state(b.problems)
    for call in range(200):
        assert lib.burgers_run_static(ps, i64(len(ps)), B.F64, MAIN, vp(u.ctypes.data), i64(50)) == 0
    assert fake.fake_streams_used() > 1
    assert fake.fake_streams_made() <= 3 and fake.fake_events_made() <= 7, (fake.fake_streams_made(), fake.fake_events_made())
# a context's own are given back with it
made, events = fake.fake_streams_live(), fake.fake_events_live()
ctx = create(batch.problems)
u = state(batch.problems)
assert lib.burgers_run(ctx, vp(u.ctypes.data), i64(50)) == 0
assert fake.fake_streams_live() > made
lib.burgers_destroy(ctx)
assert fake.fake_streams_live() == made and fake.fake_events_live() == events
""", tmp_path)


def test_serial_gradients_keep_to_the_callers_stream(tmp_path):
    """plan.serial = 1: every launch of a gradient goes to the context's stream, with one checkpoint segment and with
    several; without it the chains fork."""
    fake_hip.run("""
batch = W.random_batch(7, 12, 3, 20000)
for p in batch.problems:
    p.dt = 1e-4
ctx = create(batch.problems)
u, lam, g, gn = (state(batch.problems) for _ in range(4))
at = lambda a: vp(a.ctypes.data)
def gradient(ckpt):
    fake.fake_reset()
    assert lib.burgers_adjoint(ctx, at(u), at(lam), i64(40), i64(ckpt), at(g), at(gn)) == 0
    assert fake.fake_launches() > 0
    return fake.fake_streams_used()
assert gradient(10) > 1
assert lib.burgers_set_plan(ctx, ctypes.byref(B.CPlan(0, 0, 0, 0, 0, 0, 1, 0))) == 0
for ckpt in (40, 10, 1):
    assert gradient(ckpt) == 1 and fake.fake_stream_used(MAIN), ckpt
lib.burgers_destroy(ctx)
""", tmp_path)
