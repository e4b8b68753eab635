"""Exchanges with a batch from two threads at once: each thread's stream is
waited for, whatever the other records in between (fake streams and events)."""
import threading

import torch

from paper_2112_13930_amd.batch import Batch


class Stream:
    def __init__(self):
        self.waited = []

    def wait_event(self, event):
        self.waited.append(event.at)


def test_a_record_of_another_thread_does_not_replace_ours(monkeypatch):
    first, second, own = Stream(), Stream(), Stream()
    recorded, done = threading.Event(), threading.Event()

    class Event:
        def record(self, stream):
            self.at = stream
            if stream is first:  # the other thread's exchange comes in between
                recorded.set()
                assert done.wait(10)

    monkeypatch.setattr(torch.cuda, "Event", Event)

    class Exchange(Batch):
        def __init__(self):
            self.stream, self._kept = own, threading.local()

        def __del__(self):
            pass

    b = Exchange()

    def other():
        assert recorded.wait(10)
        b._enter(second)
        done.set()

    t = threading.Thread(target=other)
    t.start()
    b._enter(first)
    t.join()
    assert own.waited == [second, first]
    pair = b._events()
    assert b._events() is pair  # kept within a thread
