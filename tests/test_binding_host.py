"""The binding's hand-over between the caller's stream and the model's, on stand-ins for torch's streams and
events (no GPU needed)."""
import threading

from paper_2512_21571_amd import binding


class FakeTorch:
    """Streams are names; an event remembers the stream it was last recorded on; `waits` lists (stream, awaited)."""

    def __init__(self):
        self.current, self.waits = threading.local(), []
        outer = self

        class Event:
            on = None

            def record(self, stream):
                self.on = stream.name

        class Stream:
            def __init__(self, name):
                self.name = name

            def wait_event(self, event):
                outer.waits.append((self.name, event.on))

        class cuda:
            pass

        cuda.Event, cuda.Stream = Event, Stream
        cuda.current_stream = staticmethod(lambda device=None: outer.current.stream)
        self.cuda = cuda


def _model():
    fake = FakeTorch()
    m = object.__new__(binding.Model)
    m.torch, m.device, m.stream = fake, "cuda:0", fake.cuda.Stream("model")
    m._local = threading.local()
    return m, fake


def test_hand_over_of_one_caller():
    m, fake = _model()
    for name in ("a", "b"):
        fake.current.stream = fake.cuda.Stream(name)
        m._before()
        m._after()
    assert fake.waits == [("model", "a"), ("a", "model"), ("model", "b"), ("b", "model")]


def test_calls_of_two_threads_hand_over_their_own_streams():
    """One thread's call begins and ends inside another's: each stream waits for the model, and the model for each."""
    m, fake = _model()
    began, ended = threading.Event(), threading.Event()

    def inner():
        fake.current.stream = fake.cuda.Stream("inner")
        assert began.wait(10)
        m._before()
        m._after()
        ended.set()

    t = threading.Thread(target=inner)
    t.start()
    fake.current.stream = fake.cuda.Stream("outer")
    m._before()
    began.set()
    assert ended.wait(10)
    m._after()
    t.join()
    assert fake.waits == [("model", "outer"), ("model", "inner"), ("inner", "model"), ("outer", "model")]
