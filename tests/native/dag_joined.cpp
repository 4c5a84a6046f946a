// The joined task lists of the persistent launch (dag.hpp, join) with the
// emulator of dag_emulate.cpp: no task lost, every value a task waits for is set
// by an earlier one, workers that take tasks in order never all wait, tasks
// runnable together never conflict on a tile, and the tasks compute the same
// inverse.  Prints "ok ..." per case.
#define main emulate_main
#include "dag_emulate.cpp"
#undef main

static std::vector<Task> parts(const Task& t) {
  std::vector<Task> p;
  for (int q = 0; q < t.n; ++q) p.push_back(Task{t.type, t.i, t.k, t.j + q});
  return p;
}

static void foot(const Task& t, std::vector<Acc>& rd, std::vector<Acc>& wr, int phase) {
  std::vector<Acc> r, w, ra, wa;
  for (const Task& p : parts(t)) {
    footprint(p, r, w, phase);
    ra.insert(ra.end(), r.begin(), r.end());
    wa.insert(wa.end(), w.begin(), w.end());
  }
  rd = ra;
  wr = wa;
}

static int check_joined(const std::vector<int>& nbks, const std::vector<char>& inv, int most,
                        int TS, unsigned seed, int workers) {
  const std::vector<uint64_t> plain = launch_list(nbks, inv), list = join(plain, most);
  size_t total = 0;
  for (uint64_t w : list) {
    int b = 0;
    const Task t = unpack(w, &b);
    if (t.n < 1 || t.n > most) return fail("length", nbks[0], total);
    total += t.n;
  }
  if (total != plain.size()) return fail("tasks lost", nbks[0], total);
  std::vector<std::vector<int>> ctr(nbks.size());
  for (size_t b = 0; b < nbks.size(); ++b) ctr[b].assign(counters_per_block(nbks[b]), 0);
  std::vector<Block> blocks(nbks.size());
  std::vector<std::vector<double>> A0(nbks.size());
  std::mt19937_64 rng(seed);
  for (size_t b = 0; b < nbks.size(); ++b) {
    Block& B = blocks[b];
    B.nbk = nbks[b];
    B.TS = TS;
    B.n = B.nbk * TS;
    B.A.assign((size_t)B.n * B.n, 0.0);
    for (int r = 0; r < B.n; ++r)
      for (int c = 0; c <= r; ++c)
        B.a(r, c) = B.a(c, r) = r == c ? 4.0 : 0.3 * std::cos(1.0 + r * 0.7 + c * 1.3) / B.n;
    A0[b] = B.A;
    B.L.assign((size_t)B.n * B.n, 0.0);
    B.St.assign((size_t)B.nbk * B.nbk * TS * TS, 0.0);
  }
  size_t next = 0, done = 0;
  std::vector<size_t> held;
  std::vector<int> phase;
  while ((int)held.size() < workers && next < list.size()) {
    held.push_back(next++);
    phase.push_back(0);
  }
  std::vector<Acc> r1, w1, r2, w2;
  while (done < list.size()) {
    std::vector<size_t> ready;
    for (size_t h = 0; h < held.size(); ++h) {
      int b = 0;
      const Task t = unpack(list[held[h]], &b);
      Wait w[4], st;
      const int nw = waits_of(nbks[b], t, w, &st);
      bool ok = true;
      for (int e = 0; e < nw && phase[h] == 0; ++e) ok = ok && ctr[b][w[e].ctr] >= w[e].value;
      if (ok) ready.push_back(h);
    }
    if (ready.empty()) return fail("deadlock: every worker waits", nbks[0], done);
    for (size_t x = 0; x < ready.size(); ++x)
      for (size_t y = x + 1; y < ready.size(); ++y) {
        int b1 = 0, b2 = 0;
        const Task t1 = unpack(list[held[ready[x]]], &b1), t2 = unpack(list[held[ready[y]]], &b2);
        if (b1 != b2) continue;
        foot(t1, r1, w1, phase[ready[x]]);
        foot(t2, r2, w2, phase[ready[y]]);
        if (overlap(w1, r2) || overlap(w1, w2) || overlap(r1, w2))
          return fail("conflicting runnable tasks", nbks[b1], held[ready[x]]);
      }
    const size_t h = ready[(size_t)(rng() % ready.size())];
    int b = 0;
    const Task t = unpack(list[held[h]], &b);
    Wait w[4], st, md;
    waits_of(nbks[b], t, w, &st);
    if (t.type == T_C && phase[h] == 0) {
      run_task(blocks[b], t, 0);
      mid_set(t, &md);
      if (ctr[b][md.ctr] + 1 != md.value) return fail("counter step", nbks[b], held[h]);
      ctr[b][md.ctr] = md.value;
      phase[h] = 1;
      continue;
    }
    for (const Task& p : parts(t)) run_task(blocks[b], p, phase[h]);
    if (ctr[b][st.ctr] + (t.type == T_C ? 2 : t.n) != st.value)
      return fail("counter step", nbks[b], held[h]);
    ctr[b][st.ctr] = st.value;
    ++done;
    if (next < list.size()) {
      held[h] = next++;
      phase[h] = 0;
    } else {
      held.erase(held.begin() + h);
      phase.erase(phase.begin() + h);
    }
  }
  for (size_t b = 0; b < nbks.size(); ++b) {
    Block& B = blocks[b];
    std::vector<double> M = A0[b], G;
    if (!chol(M, B.n)) return fail("reference not SPD", B.nbk, 0);
    trinv(M, G, B.n);
    double ld = 0.0;
    for (int i = 0; i < B.n; ++i) ld += 2.0 * std::log(M[(size_t)i * B.n + i]);
    if (!(std::fabs(ld - B.logdet) <= 1e-12 * std::fabs(ld))) return fail("logdet", B.nbk, 0);
    for (int c = 0; inv[b] && c < B.n; ++c)
      for (int r = c; r < B.n; ++r)
        if (!(std::fabs(G[(size_t)c * B.n + r] - B.a(r, c)) <= 1e-12)) return fail("inverse", B.nbk, 0);
  }
  std::printf("ok joined %d blocks=%zu workers=%d words=%zu of %zu\n", most, nbks.size(), workers,
              list.size(), plain.size());
  return 0;
}

int main() {
  // one tile to two full groups and a remainder, blocks with and without inverse
  const std::vector<std::vector<int>> cases = {{1}, {2}, {3}, {5}, {6}, {9}, {13}, {18}, {7, 10, 3}};
  for (size_t c = 0; c < cases.size(); ++c)
    for (int most : {1, 4, 8})
      for (int w : {1, 17, 256})
        for (int inverse = 0; inverse < 2; ++inverse) {
          std::vector<char> inv(cases[c].size(), (char)inverse);
          if (cases[c].size() > 1) inv[0] = 1;
          if (check_joined(cases[c], inv, most, 3, 5 + (unsigned)c, w)) return 1;
        }
  return 0;
}
