"""The side streams of the stage call (csrc/side_streams.h), compiled for the host from the lines the library uses, on a runtime
whose streams are only told to be busy or idle.  CPU only."""
import os
import subprocess
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_19131_amd", "csrc")

RUNTIME = textwrap.dedent(r'''
    #pragma once
    #include <set>
    struct FakeStream { bool busy = false; };
    typedef FakeStream* hipStream_t;
    typedef int* hipEvent_t;
    enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorNotReady = 600 };
    enum { hipEventDisableTiming = 2, hipStreamNonBlocking = 1 };
    enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal, hipStreamCaptureModeRelaxed };
    #define hipStreamPerThread ((hipStream_t)2)
    inline bool creation_fails = false;
    inline int recorded = 0, waited = 0, synchronized = 0, record_fails_at = 0, wait_fails_at = 0;   // the n-th one from here on
    inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { ++recorded; return record_fails_at && !--record_fails_at ? hipErrorOutOfMemory : hipSuccess; }
    inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { ++waited; return wait_fails_at && !--wait_fails_at ? hipErrorOutOfMemory : hipSuccess; }
    inline hipError_t hipStreamSynchronize(hipStream_t) { ++synchronized; return hipSuccess; }
    inline std::set<FakeStream*> streams;
    inline std::set<int*> events;
    inline hipStreamCaptureMode mode_now = hipStreamCaptureModeGlobal;
    inline int calls_outside_relaxed = 0;
    // a thread may not ask for the state of a stream while another one captures in the global mode, unless it says that it knows
    inline void unsafe() { calls_outside_relaxed += mode_now != hipStreamCaptureModeRelaxed; }
    inline hipError_t hipGetLastError() { return hipSuccess; }
    inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { events.insert(*e = new int); return hipSuccess; }
    inline hipError_t hipEventDestroy(hipEvent_t e) { events.erase(e); delete e; return hipSuccess; }
    inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
    {
        if (creation_fails) return hipErrorOutOfMemory;
        streams.insert(*s = new FakeStream);
        return hipSuccess;
    }
    inline hipError_t hipStreamDestroy(hipStream_t s) { streams.erase(s); delete s; return hipSuccess; }
    inline hipError_t hipStreamQuery(hipStream_t s) { unsafe(); return s->busy ? hipErrorNotReady : hipSuccess; }
    inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { const auto t = mode_now; mode_now = *m; *m = t; return hipSuccess; }
''')

PROGRAM = textwrap.dedent(r'''
    #include <cstdio>
    #include <cstring>
    #include "side_streams.h"
    using namespace mixaq;
    static FakeStream users[6];
    int main(int argc, char** argv)
    {
        SideStreams& pool = SideStreams::of(0);
        auto is = [&](const char* name) { return argc > 1 && !std::strcmp(argv[1], name); };
        bool ok = true;
        SideStreams::Side* side[6] = {};
        if (is("creation_while_all_are_in_use")) {
            // a block is created on a fifth stream while four others are inside a stage call: it is, and its stage runs as one chain
            for (int i = 0; i < 4; ++i) { pool.retain(&users[i]); side[i] = pool.begin(&users[i]); ok = ok && side[i]; }
            pool.retain(&users[4]);
            ok = ok && !pool.begin(&users[4]);
            for (int i = 0; i < 4; ++i) { ok = ok && side[i]->caller == &users[i]; pool.done(side[i]); }
            for (int i = 0; i < 5; ++i) { ok = ok && !streams.empty(); pool.release(); }
            ok = ok && streams.empty() && events.empty();
        }
        if (is("creation_without_a_stream")) {
            // the side stream is an option: a block exists without one, and gets one as soon as there are some
            creation_fails = true;
            pool.retain(&users[0]);
            ok = ok && !pool.begin(&users[0]);
            creation_fails = false;
            side[0] = pool.begin(&users[0]);
            ok = ok && side[0] && side[0]->stream;
            if (side[0]) pool.done(side[0]);
            pool.release();
            ok = ok && streams.empty() && events.empty();
        }
        if (is("creation_takes_no_stream_over")) {
            // a block created on a fifth stream leaves the callers theirs
            for (int i = 0; i < 4; ++i) { pool.retain(&users[i]); side[i] = pool.begin(&users[i]); pool.done(side[i]); }
            pool.retain(&users[4]);
            for (int i = 0; i < 4; ++i) ok = ok && side[i]->caller == &users[i];
            ok = ok && streams.size() == 4;
            for (int i = 0; i < 5; ++i) pool.release();
            ok = ok && streams.empty() && events.empty();
        }
        if (is("taken_over_when_idle")) {
            // four callers' second chains are queued and wait for their callers; a fifth caller's would wait behind one of them for a
            // stream that may itself wait for the fifth: it gets the one that is idle, the least used where there are more, or none
            for (int i = 0; i < 4; ++i) { pool.retain(&users[i]); side[i] = pool.begin(&users[i]); pool.done(side[i]); side[i]->stream->busy = true; }
            pool.retain(&users[4]);
            ok = ok && !pool.begin(&users[4]);
            for (int i = 0; i < 4; ++i) ok = ok && side[i]->caller == &users[i] && side[i]->calls == 0;
            for (int i : {3, 1, 2}) side[i]->stream->busy = false;
            side[4] = pool.begin(&users[4]);
            ok = ok && side[4] == side[1] && side[1]->caller == &users[4];
            side[5] = pool.begin(&users[1]);                     // and the one that lost it takes the next
            ok = ok && side[5] == side[2] && side[2]->caller == &users[1];
            ok = ok && pool.begin(&users[0]) == side[0];         // a busy stream goes on serving its own caller
            ok = ok && calls_outside_relaxed == 0 && mode_now == hipStreamCaptureModeGlobal;
            for (int i = 0; i < 5; ++i) pool.release();
        }
        if (is("join_that_fails")) {
            // the caller's stream cannot be made to wait for the second chain: the call says so, and does not return before the chain's end
            pool.retain(&users[0]);
            side[0] = pool.begin(&users[0]);
            ok = ok && side[0]->fork_from(&users[0]) == hipSuccess && side[0]->join_to(&users[0]) == hipSuccess && !synchronized;
            ok = ok && recorded == 2 && waited == 2;
            record_fails_at = 2;
            ok = ok && side[0]->fork_from(&users[0]) == hipSuccess && side[0]->join_to(&users[0]) != hipSuccess && synchronized == 1;
            wait_fails_at = 2;
            ok = ok && side[0]->fork_from(&users[0]) == hipSuccess && side[0]->join_to(&users[0]) != hipSuccess && synchronized == 2;
            record_fails_at = 1;
            ok = ok && side[0]->fork_from(&users[0]) != hipSuccess;
            wait_fails_at = 1;
            ok = ok && side[0]->fork_from(&users[0]) != hipSuccess;
            pool.done(side[0]);
            pool.release();
        }
        std::printf(ok ? "ok\n" : "bad\n");
        return 0;
    }
''')


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("side_streams")
    os.makedirs(d / "hip")
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "main.cpp").write_text(PROGRAM)
    exe = str(d / "side_streams")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", str(d), "-I", CSRC, "-o", exe, str(d / "main.cpp"), "-lpthread"], check=True)
    return exe


@pytest.mark.parametrize("case", ["creation_while_all_are_in_use", "creation_without_a_stream", "creation_takes_no_stream_over"])
def test_a_block_can_always_be_created(program, case):
    assert subprocess.run([program, case], capture_output=True, text=True, check=True, timeout=20).stdout == "ok\n"


def test_a_side_stream_with_queued_work_is_not_taken_over(program):
    assert subprocess.run([program, "taken_over_when_idle"], capture_output=True, text=True, check=True, timeout=20).stdout == "ok\n"


def test_a_join_that_fails_is_an_error_and_leaves_no_chain_behind(program):
    assert subprocess.run([program, "join_that_fails"], capture_output=True, text=True, check=True, timeout=20).stdout == "ok\n"
