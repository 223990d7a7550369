// The C ABI's host side on the model of HIP (see hip/hip_runtime.h): what it
// keeps, hands out and releases over many contexts and batches.  Kernels are
// stand-ins that leave what the host reads back; an NRMSE of (J mod 5 + 1)/k
// after k iterations makes members stop at different times.
#include "../../paper_2111_14240_amd/csrc/pmace_api.hip"

#include <atomic>
#include <thread>

// Memory that runs out: the allocation from which on every one fails.
static std::atomic<long> g_allocs_left{-1};
static bool exhausted() {
  long n = g_allocs_left.load();
  if (n < 0 || model::inside > 0) return false;
  if (n > 0) g_allocs_left = n - 1;
  return n == 0;
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return exhausted() ? nullptr : std::malloc(n ? n : 1); }
void* operator new(size_t n) {
  if (exhausted()) throw std::bad_alloc();
  void* p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

namespace pmace {
static double figure(const Recon& r, double k) { return (r.J % 5 + 1) / (k > 0 ? k : 1); }
static void finish(const Recon* recs, const int* items, int nf, int update_stop, float tol, int min_iter, int max_iter,
                   double* host, int word) {
  for (int i = 0; i < nf; ++i) {
    const Recon& r = recs[items[i]];
    if (update_stop && *r.done) continue;
    if (update_stop) r.track[3] += 1;
    const double e = figure(r, r.track[3]), prev = r.track[word];
    r.track[update_stop ? word : word == 4 ? 6 : word] = e;
    if (host) *host = e;
    if (update_stop && (r.track[3] >= max_iter || (r.track[3] >= min_iter && std::fabs(e - prev) < tol))) *r.done = 1;
  }
}
int max_ppw(int np) { return np <= 64 ? 2 : np <= 128 ? 1 : 0; }
int default_ppw(int) { return 1; }
int cr_round(int) { return 16; }
hipError_t launch_setup_inputs(const Recon& h, const SetupInputs& in, int* fitem, hipStream_t st) {
  const Recon r = h;
  const int2* pos = in.pos;
  model::launch(st, [=] {
    *r.status = 0;
    *r.done = *fitem = 0;
    r.track[3] = 0;
    std::memcpy(r.pos, pos, r.J * sizeof(int2));
  });
  return hipSuccess;
}
hipError_t launch_setup_states(const Recon&, const SetupInputs&, hipStream_t) { return hipSuccess; }
hipError_t launch_setup_lists(const Recon& h, const SetupChunk& k, int tiles_c, int, int, hipStream_t st) {
  const Recon r = h;
  const SetupChunk c = k;
  model::launch(st, [=] {  // as the kernel: every place once
    for (int t = 0; t < c.tiles_r * tiles_c; ++t) {
      const int slot = c.slots ? c.slots[t] : t;
      if (slot >= 0) r.tiles[c.tile0 + slot] = make_int4(0, 1, 0, 0);
    }
    for (int i = 0; i < c.nitems; ++i)
      if (c.rows) r.citems[c.item0 + i] = make_int4(0, 1, c.rows[i].x, c.rows[i].y);
  });
  return hipSuccess;
}
hipError_t launch_setup_images(const Recon& h, Recon* rec, int2*, hipStream_t st) {
  const Recon r = h;
  model::launch(st, [=] { *rec = r; });
  return hipSuccess;
}
static hipError_t nothing(hipStream_t st) { return model::launch(st, [] {}), hipSuccess; }
hipError_t launch_small_iteration(int, const Recon&, int, hipStream_t st) { return nothing(st); }
hipError_t launch_small_batch(int, const Recon*, const int2*, int, const int2*, int, int, bool, hipStream_t st) {
  return nothing(st);
}
hipError_t launch_large_iteration(const Recon&, const Recon*, const int2*, const int2*, hipStream_t st) {
  return nothing(st);
}
hipError_t launch_get_state(const Recon&, const Recon*, float2*, hipStream_t st) { return nothing(st); }
hipError_t launch_set_state(const Recon&, const Recon*, const float2*, const int2*, hipStream_t st) { return nothing(st); }
hipError_t launch_nrmse(const Recon* recs, const int2*, int, const int* fitems, int nf, int update_stop, float tol,
                        int min_iter, int max_iter, double* host, hipStream_t st) {
  model::launch(st, [=] { finish(recs, fitems, nf, update_stop, tol, min_iter, max_iter, host, 1); });
  return hipSuccess;
}
hipError_t launch_fit_member(const Recon&, const Recon*, int, hipStream_t st) { return nothing(st); }
hipError_t launch_fit_batch(int, const Recon*, const int2*, int, hipStream_t st) { return nothing(st); }
hipError_t launch_fit_finish(const Recon* recs, const int* fitems, int nf, int update_stop, float tol, int min_iter,
                             int max_iter, double* host, hipStream_t st) {
  model::launch(st, [=] { finish(recs, fitems, nf, update_stop, tol, min_iter, max_iter, host, 4); });
  return hipSuccess;
}
hipError_t launch_tick(const Recon* recs, const int* items, int n, int max_iter, hipStream_t st) {
  model::launch(st, [=] {
    for (int i = 0; i < n; ++i) {
      const Recon& r = recs[items[i]];
      if (!*r.done && ++r.track[3] >= max_iter) *r.done = 1;
    }
  });
  return hipSuccess;
}
hipError_t launch_poll(const Recon* recs, int n, PollItem* out, hipStream_t st) {
  model::launch(st, [=] {
    for (int i = 0; i < n; ++i) out[i] = {recs[i].track[1], recs[i].track[3], recs[i].track[4], *recs[i].done, 0};
  });
  return hipSuccess;
}
hipError_t launch_fft2(int, int, const float2*, float2*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_split_iteration(const Recon&, int, hipStream_t st) { return nothing(st); }
}  // namespace pmace

#define CHECK(x) \
  if (!(x)) model::fault(std::string("line ") + std::to_string(__LINE__) + ": " #x)

struct Rec {  // a small reconstruction: np, J
  std::vector<char> ws;
  pmace_ctx* c = nullptr;
  int J;
  Rec(int np, int J, hipStream_t st = nullptr) : J(J) {
    pmace_params p{};
    p.n1 = p.n2 = np + 8;
    p.np = np;
    p.num_pos = J;
    p.alpha = 0.5f;
    p.kappa = 1.25f;
    p.rho = 0.5f;
    ws.resize(pmace_footprint(&p));
    CHECK(!ws.empty());
    std::vector<int> pos(2 * J);
    for (int j = 0; j < J; ++j) pos[2 * j] = pos[2 * j + 1] = j % 9;
    std::vector<float> any(16);
    CHECK(pmace_init(&p, any.data(), pos.data(), any.data(), nullptr, ws.data(), ws.size(), st, &c) == PMACE_OK);
    CHECK(pmace_set_reference(c, any.data(), nullptr) == PMACE_OK);  // never read by the stand-ins
  }
  ~Rec() { pmace_destroy(c); }
  void figures() {
    double e = -1, f = -1;
    CHECK(pmace_nrmse(c, &e) == PMACE_OK && e == J % 5 + 1);
    CHECK(pmace_data_fit(c, &f) == PMACE_OK && f == J % 5 + 1);
    CHECK(pmace_sync(c) == PMACE_OK);
  }
};

struct Bat {
  std::vector<char> ws;
  pmace_batch* b = nullptr;
  int n;
  std::vector<int> done, it;
  std::vector<double> e;
  Bat(const std::vector<Rec*>& rs, pmace_stop_rule rule) : n((int)rs.size()), done(n), it(n), e(n) {
    std::vector<pmace_ctx*> cs;
    for (auto* r : rs) cs.push_back(r->c);
    ws.resize(pmace_batch_footprint(cs.data(), n));
    CHECK(pmace_batch_create(cs.data(), n, &rule, ws.data(), ws.size(), &b) == PMACE_OK);
  }
  ~Bat() { pmace_batch_destroy(b); }
  void step(int k) { CHECK(pmace_batch_step(b, k) == PMACE_OK); }
  int poll() {
    const long before = model::destroys;
    CHECK(pmace_batch_poll(b, done.data(), e.data(), it.data()) == PMACE_OK);
    CHECK(model::destroys == before);  // nothing is released next to work that has only just ended
    int k = 0;
    for (int d : done) k += d != 0;
    return k;
  }
};

static const int kSides[] = {32, 64, 256, 48, 128, 160, 96, 256};

// Read-back memory: more contexts and batches alive than it has slots, used by
// several threads, and none to be had.
static void slots() {
  std::vector<Rec*> rs;
  for (int i = 0; i < 100; ++i) rs.push_back(new Rec(kSides[i % 8], 1 + i % 7));
  {
    Bat a(rs, {1e-3f, 2, 50, PMACE_STOP_NRMSE, 1}), b({rs[3], rs[5]}, {1e-3f, 2, 50, PMACE_STOP_DATA_FIT, 2});
    for (auto* r : rs) r->figures();
    CHECK(a.poll() == 0 && b.poll() == 0);
  }
  for (auto* r : rs) delete r;
  std::vector<std::thread> ts;
  for (int t = 0; t < 6; ++t)
    ts.emplace_back([t] {
      hipStream_t st = nullptr;
      CHECK(hipStreamCreateWithFlags(&st, 0) == hipSuccess);
      for (int i = 0; i < 30; ++i) {
        Rec r(kSides[(i + t) % 8], 2 + t, st);
        r.figures();
      }
      CHECK(hipStreamDestroy(st) == hipSuccess);
    });
  for (auto& t : ts) t.join();
  CHECK(model::host_frees == 0);
  CHECK(model::host_mallocs <= (long)pmace::kHostSlots);
  const long had = model::host_mallocs;
  model::host_malloc_fails = true;
  std::vector<void*> taken;
  while (void* p = pmace::take_host_slot()) taken.push_back(p);
  CHECK((long)taken.size() == had);
  {
    Rec r(64, 3), q(256, 4);
    r.figures();
    Bat b({&r, &q}, {0.f, 2, 3, PMACE_STOP_NRMSE, 1});
    b.step(5);
    CHECK(b.poll() == 2 && b.it[0] == 3 && b.it[1] == 3);
  }
  for (void* p : taken) pmace::give_host_slot(p);
}

// Batches: members that stop one after the other, are started again, polls
// between; many batches one after the other, and several at a time.
static void batches() {
  for (int criterion : {PMACE_STOP_NRMSE, PMACE_STOP_DATA_FIT})
    for (int every : {1, 3}) {
      std::vector<Rec*> rs;
      for (int i = 0; i < 64; ++i) rs.push_back(new Rec(kSides[i % 8], 1 + i % 7));
      {
        Bat b(rs, {0.02f, 2, 40, criterion, every});
        int last = 0;
        for (int k = 0; k < 12 && last < 64; ++k) {
          b.step(4);
          const int now = b.poll();
          CHECK(now >= last);
          last = now;
        }
        CHECK(last == 64);
        for (int i = 0; i < 64; ++i) {
          // |e_k - e_(k-1)| = c/(k (k - every)) < tol first, k a multiple of every
          const double c = rs[i]->J % 5 + 1;
          int k = every;
          while (!(k >= 2 && k > every && c / (k - every) - c / k < 0.02 - 1e-12)) k += every;
          CHECK(b.it[i] == k);
        }
        CHECK(pmace_set_reference(rs[2]->c, rs[2]->ws.data(), nullptr) == PMACE_OK);  // runs again
        CHECK(pmace_iterate(rs[7]->c, 1) == PMACE_OK);
        b.step(1);
        CHECK(b.poll() <= 63 && !b.done[2] && b.it[2] == 1);
      }
      for (auto* r : rs) delete r;
    }
  const long made = model::streams_made;
  for (int i = 0; i < 100; ++i) {
    Rec a(256, 3), b(64, 2), c(160, 5);
    Bat x({&a, &b, &c}, {0.f, 2, 9, PMACE_STOP_NRMSE, 1});
    x.step(10);
    CHECK(x.poll() == 3);
  }
  CHECK(model::streams_made - made <= 8);
  {
    std::vector<Rec*> rs;
    std::vector<Bat*> bs;
    for (int i = 0; i < 40; ++i) {
      rs.push_back(new Rec(256, 3));
      rs.push_back(new Rec(160, 4));
      bs.push_back(new Bat({rs[2 * i], rs[2 * i + 1]}, {0.f, 2, 5, PMACE_STOP_NRMSE, 1}));
      bs.back()->step(6);
    }
    for (auto* b : bs) CHECK(b->poll() == 2);
    for (auto* b : bs) delete b;
    for (auto* r : rs) delete r;
  }
  CHECK(model::streams_live <= 64);
  CHECK(model::execs_live == 0);
}

// The places of gather tiles without the empty ones, against a count of what
// each rectangle meets: every kept tile has one place, in its row's range, and
// a full row's are the kernel's own.
static void cover() {
  unsigned seed = 1;
  const auto rnd = [&](int n) { return (int)((seed = seed * 1664525u + 1013904223u) >> 8) % n; };
  for (int trial = 0; trial < 2000; ++trial) {
    const int nr = 1 + rnd(6), nc = 1 + rnd(40), rects = rnd(8);
    Cover c(nr, nc);
    std::vector<int> ref(nr * nc, 0);
    for (int k = 0; k < rects; ++k) {
      const int r0 = rnd(nr), r1 = r0 + rnd(nr - r0), c0 = rnd(nc), c1 = c0 + rnd(nc - c0);
      const bool all = rnd(6) == 0;  // a rectangle over everything
      c.add(all ? 0 : r0, all ? nr - 1 : r1, all ? 0 : c0, all ? nc - 1 : c1);
      for (int r = all ? 0 : r0; r <= (all ? nr - 1 : r1); ++r)
        for (int q = all ? 0 : c0; q <= (all ? nc - 1 : c1); ++q) ++ref[r * nc + q];
    }
    int met = 0;
    for (int v : ref) met += v > 0;
    CHECK(c.close() == met);
    for (bool xcd : {false, true}) {
      const std::vector<int> slots = tile_slots(c, xcd);
      std::vector<int> seen(met, 0);
      int first = 0;
      for (int r = 0; r < nr; ++r) {
        int n = 0;
        for (int q = 0; q < nc; ++q) n += ref[r * nc + q] > 0;
        for (int q = 0; q < nc; ++q) {
          const int s = slots[r * nc + q];
          CHECK(c.at(r, q) == (ref[r * nc + q] > 0) && (s >= 0) == c.at(r, q));
          if (s < 0) continue;
          CHECK(s >= first && s < first + n && !seen[s]++);
          if (n == nc && first == r * nc) {
            const int e = nc / 8;
            int own = xcd && q < 8 * e ? (q % e) * 8 + q / e : q;
            if (!xcd && nc % 8 == 0) own = (q + r) % nc;
            CHECK(s == r * nc + own);
          }
        }
        first += n;
      }
    }
  }
  // through pmace_init, whose tables must hold the kept ones: sparse, and in chunks
  for (int np : {32, 128, 160, 256})
    for (int chunk : {0, 3}) {
      pmace_params p{};
      p.n1 = np > 128 ? 2200 : 700;
      p.n2 = 2500;
      p.np = np;
      p.num_pos = 14;
      p.alpha = 0.5f;
      p.kappa = 1.25f;
      p.rho = 0.5f;
      p.chunk = chunk;
      p.flags = np > 128 ? PMACE_ROWSPEC_AGENT : 0;
      std::vector<char> ws(pmace_footprint(&p));
      std::vector<int> pos(28);
      for (int j = 0; j < 14; ++j) {
        pos[2 * j] = rnd(p.n1 - np + 1);
        pos[2 * j + 1] = rnd(2500 - np + 1);
      }
      std::vector<float> any(16);
      pmace_ctx* x = nullptr;
      CHECK(pmace_init(&p, any.data(), pos.data(), any.data(), nullptr, ws.data(), ws.size(), nullptr, &x) == PMACE_OK);
      int items = 0;
      for (const int2& r : x->chunk_rows) items += r.y;
      if (np <= 128) CHECK(x->ngitems > 0 && x->ngitems < (int)max_tiles(p) - kEmptyTiles && items == 0);
      if (np > 128 && chunk == 0) CHECK(items > 0 && items < (int)cr_items(p) - kEmptyItems);
      for (int t = 0; t < x->ngitems; ++t) CHECK(x->h.tiles[t].y == 1);
      for (int t = 0; np > 128 && chunk == 0 && t < items; ++t) CHECK(x->h.citems[t].y == 1);
      pmace_destroy(x);
    }
}

// pmace_iterate under a caller's capture: launches only, whatever came before
// (membership of a batch, a captured graph of its own).
static void captured() {
  for (int np : {64, 256}) {
    hipStream_t st = nullptr;
    CHECK(hipStreamCreateWithFlags(&st, 0) == hipSuccess);
    {
      Rec a(np, 3, st), b(160, 2, st);
      {
        Bat x({&a, &b}, {0.f, 2, 4, PMACE_STOP_NRMSE, 1});
        x.step(5);
        CHECK(x.poll() == 2);
      }
      for (int before : {0, 300}) {
        CHECK(pmace_iterate(a.c, before) == PMACE_OK);
        CHECK(pmace_sync(a.c) == PMACE_OK);
        const long mine = model::graph_calls;
        hipGraph_t g = nullptr;
        CHECK(hipStreamBeginCapture(st, hipStreamCaptureModeThreadLocal) == hipSuccess);
        CHECK(pmace_iterate(a.c, 40) == PMACE_OK);
        CHECK(hipStreamEndCapture(st, &g) == hipSuccess);
        CHECK(model::graph_calls == mine + 1);
        CHECK(model::memsets_captured == 0);
        CHECK((int)g->nodes.size() >= 40);
        CHECK(hipGraphDestroy(g) == hipSuccess);
        CHECK(pmace_sync(a.c) == PMACE_OK);
      }
      CHECK(pmace_iterate(a.c, 300) == PMACE_OK);
    }
    CHECK(hipStreamDestroy(st) == hipSuccess);
  }
}

// Host memory that runs out at any allocation of a call: ENOMEM, nothing left
// behind, and the same call succeeds once there is memory.
static void no_memory() {
  const std::vector<float> any(64);
  for (int np : {64, 160}) {
    pmace_params p{};
    p.n1 = 500;
    p.n2 = 1900;
    p.np = np;
    p.num_pos = 5000;  // (more than a slot holds)
    p.alpha = 0.5f;
    p.kappa = 1.25f;
    p.rho = 0.5f;
    p.chunk = np > 128 ? 2000 : 0;
    p.flags = np > 128 ? PMACE_ROWSPEC_AGENT : 0;
    std::vector<char> ws(pmace_footprint(&p)), first;
    std::vector<int> pos(2 * p.num_pos);
    for (int j = 0; j < p.num_pos; ++j) {
      pos[2 * j] = j % 200;
      pos[2 * j + 1] = 7 * j % 300;  // the right of the object lists nothing
    }
    pmace_ctx* c[2] = {nullptr, nullptr};
    for (int k = 0; k < 2; ++k) {
      pmace_status s = PMACE_ENOMEM;
      for (long n = 0; s != PMACE_OK; ++n) {
        CHECK(n < 2000 && s == PMACE_ENOMEM && !c[k]);
        g_allocs_left = n;
        s = pmace_init(&p, any.data(), pos.data(), any.data(), nullptr, ws.data(), ws.size(), nullptr, &c[k]);
        g_allocs_left = -1;
      }
      if (k == 0) {  // the first keeps its own
        first.swap(ws);
        ws.resize(first.size());
      }
    }
    const pmace_stop_rule rule{0.f, 2, 4, PMACE_STOP_DATA_FIT, 1};
    std::vector<char> bws(pmace_batch_footprint(c, 2));
    pmace_batch* b = nullptr;
    pmace_status s = PMACE_ENOMEM;
    for (long n = 0; s != PMACE_OK; ++n) {
      CHECK(n < 2000 && (s == PMACE_ENOMEM || s == PMACE_EDEVICE) && !b && c[0]->holders.empty() && c[1]->holders.empty());
      g_allocs_left = n;
      s = pmace_batch_create(c, 2, &rule, bws.data(), bws.size(), &b);
      g_allocs_left = -1;
    }
    CHECK(pmace_batch_step(b, 5) == PMACE_OK);
    model::host_malloc_fails = true;
    std::vector<void*> taken;
    while (void* q = pmace::take_host_slot()) taken.push_back(q);
    int done[2];
    g_allocs_left = 0;
    s = pmace_batch_poll(b, done, nullptr, nullptr);
    g_allocs_left = -1;
    CHECK(s == PMACE_ENOMEM);
    CHECK(pmace_batch_poll(b, done, nullptr, nullptr) == PMACE_OK && done[0] && done[1]);
    for (void* q : taken) pmace::give_host_slot(q);
    model::host_malloc_fails = false;
    pmace_batch_destroy(b);
    pmace_destroy(c[0]);
    pmace_destroy(c[1]);
  }
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "slots") slots();
  else if (what == "batches") batches();
  else if (what == "cover") cover();
  else if (what == "captured") captured();
  else if (what == "no_memory") no_memory();
  else return 2;
  std::printf("ok\n");
}
