"""A library call that blocks (a launch on a full queue) leaves the program's other Python threads running."""
import ctypes
import threading
import time

import pytest
import torch


class Stream:
    cuda_stream = 0


@pytest.mark.parametrize("call", ["visual_pool", "node_argmax"])
def test_other_threads_run_during_a_call(call):
    import paper_2509_11815_amd as sv
    lib = sv.load_library()
    # every entry point replaced by sleep(): the first argument, the data type's code of float32, is one second
    sleep = ctypes.cast(ctypes.CDLL(None).sleep, ctypes.c_void_p).value
    native = sv.binding._native
    stop, gaps = threading.Event(), []

    def tick():
        last = time.monotonic()
        while not stop.is_set():
            time.sleep(0.01)
            now = time.monotonic()
            gaps.append(now - last)
            last = now

    thread = threading.Thread(target=tick)
    try:
        native.bind({name: sleep for name in sv.binding.EXPORTS}, sv.binding.SpecvlmError)
        thread.start()
        begin = time.monotonic()
        x = torch.zeros(1, 2, 4)
        if call == "visual_pool":
            sv.specvlm_visual_pool(x, 1, out=torch.zeros(1, 2, 4), stream=Stream())
        else:
            sv.specvlm_node_argmax(x, stream=Stream())
        took = time.monotonic() - begin
    finally:
        stop.set()
        thread.join()
        sv.binding._load_native(lib)
    assert took >= 0.9 and max(gaps) < 0.5
