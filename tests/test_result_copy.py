"""The host side of copying results out (csrc/result_copy.h) by itself: it calls no HIP, so small programs around it run on the CPU, with
memory copies in the place of the device's."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, body, top=""):
    """Compiles and runs int main() { body }; CHECK(condition) ends it with the line's number."""
    if not shutil.which("g++"):
        pytest.skip("no g++")
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text("#include <chrono>\n#include <cstdio>\n#include <cstdlib>\n#include <cstring>\n#include <future>\n#include <new>\n"
                   '#include <thread>\n#include <vector>\n#include "result_copy.h"\n'
                   "#define CHECK(x) do { if (!(x)) { std::printf(\"line %d: %s\\n\", __LINE__, #x); std::fflush(stdout); std::_Exit(1); } } while (0)\n"
                   "using namespace hydra;\n" + top + "\nint main() {\n" + body + "\n  return 0;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "paper_2107_06469_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)


STAGE = """
static int made = 0, given = 0;
static bool none = false;
static Stage st([](size_t n) -> void* { if (none) return nullptr; ++made; return std::malloc(n); },
                [](void* p) { ++given; std::free(p); });
"""


def test_contexts_come_and_go_while_another_reads(tmp_path):
    """A reader keeps the buffer for the length of its copies, seconds for large models: contexts of other threads attach and detach
    meanwhile."""
    _run(tmp_path, """
  st.attach();
  StageLease held(st);
  CHECK(held.p);
  auto other = std::async(std::launch::async, [] { st.attach(); { StageLease l(st); CHECK(!l.p); } st.detach(); });
  CHECK(other.wait_for(std::chrono::seconds(10)) == std::future_status::ready);
  CHECK(made == 1 && given == 0);
""", STAGE)


def test_the_buffer_has_one_reader_and_goes_with_the_last_context(tmp_path):
    _run(tmp_path, """
  { StageLease l(st); CHECK(!l.p); }
  st.attach();
  st.attach();
  { StageLease a(st); StageLease b(st); CHECK(a.p && !b.p); }
  { StageLease a(st); CHECK(a.p); }
  st.detach();
  CHECK(made == 1 && given == 0);
  {
    StageLease a(st);
    st.detach();
    CHECK(given == 0);
    a.p[0] = 1.f;
  }
  CHECK(given == 1);
  none = true;
  st.attach();
  { StageLease l(st); CHECK(!l.p); }
  none = false;
  st.attach();
  { StageLease l(st); CHECK(l.p); }
  st.detach();
  st.detach();
  CHECK(made == 2 && given == 2);
""", STAGE)


@pytest.mark.parametrize("left", [0, 1, 2, 3, 5])
def test_threads_that_cannot_be_made_leave_their_work_to_the_others(tmp_path, left):
    """Memory for a thread's state runs out after `left` allocations: the threads made so far are waited for, no exception leaves."""
    _run(tmp_path, f"""
  std::atomic<int> next{{0}}, done{{0}};
  auto work = [&](unsigned) {{
    while (next.fetch_add(1) < 100) {{
      std::this_thread::sleep_for(std::chrono::microseconds(200));
      ++done;
    }}
  }};
  left = {left};
  on_threads(4, work);
  left = -1;
  CHECK(done == 100);
""", """
#include <atomic>
static std::atomic<int> left{-1};  // allocations that still succeed; negative: all do
void* operator new(std::size_t n) {
  if (left >= 0 && left-- == 0) { left = 0; throw std::bad_alloc(); }
  if (void* p = std::malloc(n)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
""")


def test_copies_under_way_are_waited_for_where_one_could_not_be_requested(tmp_path):
    """The third of five copies into the leased buffer fails to start: the first two have landed before the lease can end."""
    _run(tmp_path, """
  int asked = 0, waits = 0;
  CHECK(request_all(5, [&](int i) { ++asked; return i == 2 ? 7 : 0; }, [&] { ++waits; return 0; }) == 7);
  CHECK(asked == 3 && waits == 1);
  CHECK(request_all(5, [&](int i) { return 0; }, [&] { ++waits; return 9; }) == 9);
  CHECK(request_all(5, [&](int i) { return i == 4 ? 3 : 0; }, [&] { ++waits; return 9; }) == 3);
  CHECK(request_all(0, [&](int i) { return 1; }, [&] { ++waits; return 0; }) == 0 && waits == 4);
""")


# Tensors of a model as they lie in its block (each padded to 64 floats): what is left out of a run, and runs on either side of 1 MB (262144
# floats); one tensor; tensors that do not rise.
BLOCKS = {"small": [40 * 24, 24, 24 * 24, 24, 7 * 24, 7], "around_1_mb": [512 * 512, 512, 512 * 520, 520, 130000, 131000, 1000, 11],
          "exactly_1_mb": [262144 - 64, 64, 262144, 1, 262143, 1], "large": [776 * 776, 776] * 3 + [13 * 776, 13], "one": [5]}


@pytest.mark.parametrize("block,first", [(b, f) for b in sorted(BLOCKS) for f in (0, 1) if f < len(BLOCKS[b])])
def test_tensors_arrive_whole_with_and_without_the_buffer(tmp_path, block, first):
    """Every tensor at its place and nothing beside it, straight and through the buffer by one thread and by four (a buffer of 4 MB and one of
    a few hundred floats, so that parts end inside tensors); a copy that fails is reported; the number of direct copies is that of the runs."""
    sizes = BLOCKS[block]
    _run(tmp_path, """
  const std::vector<size_t> sizes = {%s};
  std::vector<Piece> ps;
  size_t off = 64, to = 0;
  for (size_t j = 0; j < sizes.size(); ++j) {
    if (j >= %d) { ps.push_back({off, sizes[j], to}); to += sizes[j]; }
    off += (sizes[j] + 63) / 64 * 64;
  }
  std::vector<float> src(off + 64), want(to);
  for (size_t i = 0; i < src.size(); ++i) src[i] = (float)(i %% 16777213);
  for (const Piece& p : ps) std::memcpy(&want[p.to], &src[p.off], p.n * 4);
  auto same = [&](const std::vector<float>& got) {
    return got.size() == to + 2 && got[0] == -1.f && got.back() == -1.f && std::memcmp(&got[1], want.data(), to * 4) == 0;
  };
  auto fresh = [&] { return std::vector<float>(to + 2, -1.f); };

  int copies = 0;
  auto plain = [&](float* d, const float* s, size_t n) { ++copies; std::memcpy(d, s, n * 4); return 0; };
  std::vector<float> got = fresh();
  CHECK(copy_direct(ps, true, src.data(), &got[1], plain) == 0 && same(got));
  int runs = 0;
  for (size_t j = 0; j < ps.size(); ++runs) {
    const size_t end = ps[j].off + 262144;
    for (++j; j < ps.size() && ps[j].off + ps[j].n <= end;) ++j;
  }
  CHECK(copies == runs);
  copies = 0;
  got = fresh();
  CHECK(copy_direct(ps, false, src.data(), &got[1], plain) == 0 && same(got) && copies == (int)ps.size());
  CHECK(copy_direct(ps, true, src.data(), &got[1], [](float*, const float*, size_t) { return 5; }) == 5);

  for (const size_t room : {Stage::BYTES / 4, (size_t)1000}) {
    std::vector<float> stage(room);
    for (const unsigned T : {1u, 4u}) {
      got = fresh();
      auto part = [&](unsigned k, float* d, const float* s, size_t n) {
        CHECK(k < T && n <= room / T && d == stage.data() + k * (room / T));
        std::memcpy(d, s, n * 4);
        return 0;
      };
      CHECK(copy_staged(ps, src.data(), &got[1], stage.data(), room, T, part) == 0 && same(got));
      CHECK(copy_staged(ps, src.data(), &got[1], stage.data(), room, T, [](unsigned, float*, const float*, size_t) { return 3; }) == 3);
    }
  }
""" % (", ".join(map(str, sizes)), first))
