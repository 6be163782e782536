// Deferred shrinks (csrc/fd_defer_plan.h): streams cut into calls at random, with every half's rows followed by their numbers. What is
// written and what is left unwritten must together be the stream, no half may be stored to while it holds rows that are still
// needed, and no more blocks may come together than the buffers are made for. The buffers of the coefficients are followed too, by the
// numbers of the shrinks that are in them: what the side stream does between the mark and the join is done before or after what the
// context stream does there, at random, and must find what it was enqueued for either way.
// Arguments: "planted", the same with the rows of a full set of blocks not written first; "two", with two buffers for the M's;
// "forgets", with shrinks deferred after a captured call as before it. All must fail.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

#include "fd_defer_plan.h"

using sage::DeferPlan;
typedef std::vector<int> Rows;

static bool planted = false, two = false, forgets = false;
static int failures = 0;
#define REQUIRE(cond, what)                                                                      \
    do {                                                                                         \
        if (!(cond) && ++failures <= 5) printf("max = %d, ell = %d: %s\n", p.max, ell, what);     \
    } while (0)

struct Stream {
    DeferPlan p;
    int ell, fill_top = 0, fill_new = 0, rows = 0;
    bool pending = false, stored = false, shrunk = false, ready = false;
    Rows top, half[16];
    int shrinks = 0;
    Rows coef[5], due;                       // shrinks whose coefficients a buffer holds; those whose rows are not written
    std::vector<std::function<void()>> side;  // enqueued there, not done yet
    bool on_side = false;

    static void add(Rows& a, const Rows& b) { a.insert(a.end(), b.begin(), b.end()); }
    void enqueue(std::function<void()> f) {
        if (on_side) side.push_back(f);
        else f();
    }
    void join() {
        for (auto& f : side) f();
        side.clear();
    }
    void holds(int buffer, const Rows& want, const char* what) {
        enqueue([=] { REQUIRE(coef[buffer] == want, what); });
    }
    void fold() {
        REQUIRE(p.count >= 1 && p.count <= p.max, "blocks beyond what W is made for");
        const DeferPlan::Fold f = p.fold();
        const int m = p.m;
        if (f.out < 0) return;
        holds(f.from, Rows(due.begin(), due.end() - 1), "W is not that of the shrinks before the last");
        holds(m, Rows(1, due.back()), "M is not the last shrink's");
        enqueue([=] {
            Rows w = coef[f.from];
            add(w, coef[m]);
            coef[f.out] = w;
        });
    }
    void write() {
        if (!p.folded) fold();
        REQUIRE(p.count >= 1 && p.count <= p.max, "blocks beyond what W is made for");
        holds(p.w, due, "rows are written with another W than theirs");
        due.clear();
        for (int b = 0; b < p.count; ++b) add(top, half[p.slots >> (4 * b) & 15]);
        p.written();
    }
    void shrink(const int* next, int64_t n, bool captured) {
        const bool ahead = n >= ell;
        if (captured) p.captured = true;
        DeferPlan::Step s = p.step(ahead, true, n, ell);
        if (planted) s.write_first = false;
        REQUIRE((int)half[p.cur].size() == ell, "a shrink of a half that is not full");
        REQUIRE(p.count == 0 || (ready && !captured), "the products of unwritten rows are not there");
        ready = false;
        const bool write_now = !s.defer && p.count == 0, last = rand() & 1;  // last: the side stream comes late
        if (ahead) {
            if (s.defer && p.beside) {
                on_side = true;
                if (p.count > 0 && !p.folded) fold();
                if (s.write_first) write();
                if (p.count > 0) holds(p.w, due, "the rectangle is taken through another W than the rows'");
                on_side = false;
            }
            REQUIRE(s.defer || p.count == 0, "stored ahead for a shrink that comes after unwritten ones");
            const int o = p.next = p.free_half();
            REQUIRE(o >= 0 && o < p.halves() && o != p.cur, "no such half");
            for (int b = 0; b < p.count; ++b) REQUIRE(o != (int)(p.slots >> (4 * b) & 15), "the half holds a block");
            if (s.defer && (p.beside || !s.last)) REQUIRE(p.count + 2 <= p.max + 1, "more products than there is room for");
            half[o].assign(next, next + ell);
        } else if (s.write_first) {
            write();
        } else if (p.count > 0 && !p.folded) {
            fold();
        }
        if (!last) join();
        if (!write_now) coef[p.next_m()] = Rows(1, shrinks);  // the eigensolve
        join();
        if (write_now) {
            add(top, half[p.cur]);
        } else {
            p.push();
            p.made_m();
            due.push_back(shrinks);
            if (s.defer && !p.beside) {
                fold();
                holds(p.w, due, "the rectangle is taken through another W than the rows'");
            } else if (s.defer) {
                holds(p.m, Rows(1, shrinks), "the rectangle is taken through another M than the last shrink's");
            }
            ready = s.defer && (p.beside || !s.last);
            if (!s.defer || s.last) write();
        }
        p.advance(ahead);
        REQUIRE(p.cur < p.halves(), "no such half");
        if (!ahead) half[p.cur].clear();
        fill_top = ell;
        fill_new = 0;
        stored = ahead;
        shrunk = true;
        ++shrinks;
    }
    void update(int n, bool captured) {
        Rows r(n);
        for (int& x : r) x = rows++;
        const int* g = r.data();
        if (pending) {
            pending = false;
            shrink(g, n, captured);
        }
        while (n > 0) {
            int take = ell - fill_new < n ? ell - fill_new : n;
            if (fill_top < ell) {
                take = ell - fill_top < n ? ell - fill_top : n;
                top.insert(top.end(), g, g + take);
                fill_top += take;
            } else if (stored) {
                REQUIRE(take == ell && half[p.cur] == Rows(g, g + ell), "not the rows that were stored ahead");
                stored = false;
                fill_new = ell;
            } else {
                if (fill_new == 0) half[p.cur].clear();
                half[p.cur].insert(half[p.cur].end(), g, g + take);
                fill_new += take;
            }
            g += take;
            n -= take;
            if (fill_new == ell) {
                if (n == 0 && shrunk) pending = true;
                else shrink(g, n, captured);
            }
        }
        REQUIRE(p.count == 0, "a call that ends with rows unwritten");
    }
    void look() {
        if (pending) {
            pending = false;
            shrink(nullptr, 0, false);
        }
        Rows all = top;
        all.insert(all.end(), half[p.cur].begin(), half[p.cur].begin() + (fill_top == ell ? fill_new : 0));
        bool same = (int)all.size() == rows;
        for (int i = 0; same && i < rows; ++i) same = all[i] == i;
        REQUIRE(same, "the buffer is not the stream");
    }
};

int main(int argc, char** argv) {
    planted = argc > 1 && !strcmp(argv[1], "planted");
    two = argc > 1 && !strcmp(argv[1], "two");
    forgets = argc > 1 && !strcmp(argv[1], "forgets");
    srand(1);
    for (int trial = 0; trial < 40000; ++trial) {
        Stream s;
        s.ell = 2 + rand() % 4;
        s.p.max = rand() % 5;
        s.p.beside = rand() & 1;
        if (two) s.p.MS = 2;
        for (int calls = 1 + rand() % 9; calls > 0; --calls) {
            s.update(rand() % 5 < 3 ? 1 + rand() % (6 * s.ell) : s.ell * (1 + rand() % 5), false);
            if (rand() % 6 == 0) s.look();
            if (rand() % 12 == 0) {  // memory is short: the next smaller plan
                s.half[0] = s.half[s.p.cur];
                for (int i = 1; i < 16; ++i) s.half[i].clear();
                s.p.give_up();
            }
        }
        // two cycles of a captured call end where they began, and so does an even number of cycles after it
        while (!s.pending || s.shrunk == false) s.update(s.ell - s.fill_new % s.ell, false);
        const int cur = s.p.cur;
        s.ready = false;
        s.update(2 * s.ell, true);
        DeferPlan& p = s.p;
        const int ell = s.ell;
        REQUIRE(p.cur == cur, "a captured call of two cycles ends on another half");
        for (int calls = rand() % 4; calls > 0; --calls) {
            if (forgets) p.captured = false;
            s.update(2 * s.ell * (1 + rand() % 3), false);
            REQUIRE(p.cur == cur, "later calls of whole pairs of cycles end on another half than the captured one");
        }
        s.look();
    }
    if (failures) printf("%d failures\n", failures);
    else printf("defer_check ok\n");
    return failures ? 1 : 0;
}
